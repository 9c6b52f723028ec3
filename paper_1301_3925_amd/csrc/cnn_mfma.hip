// Fused inference kernel of the learned preconditioner in 2D:
//   z = r / diag(K) + N(r),  N = C1^T g1 C2^T g2 C2 g1 C1 applied as four
//   gated 3x3 convolutions 1->16->16->16->1 (expanded weights).
//
// One block computes a 16x16 tile of z.  The four layers run back to back
// in LDS with shrinking halos (r on 24x24, layer outputs on 22x22, 20x20,
// 18x18, 16x16), so r and z cross HBM once per tile and the gates once per
// tile plus halo.  Every layer runs on the matrix cores as an implicit GEMM
// with v_mfma_f32_16x16x16_bf16 (BF16 operands, FP32 accumulation), one
// 16-pixel group per instruction:
//   layer 1 (1 -> 16):  D[co][16 px] = W1[co][16 k = taps 0..8, zero-padded] X[k][px]
//   layers 2, 3:        sum over the 9 taps of W_t[co][16 ci] X_t[ci][16 px]
//   layer 4 (16 -> 1):  the same with only row co = 0 of W_t non-zero.
// The weight operands come pre-packed per lane from adlbr_net_gates.  The gates
// g1, g2 are 8-bit fixed point (g = q / 255, so they stay >= 0 and N stays
// positive semi-definite), staged in LDS once per tile.  Activations are
// stored as BF16 with a 40-byte pixel stride, which makes the 8-byte
// A-operand reads of 16 consecutive pixels bank-conflict free; layer 3
// writes over layer 1's buffer.  Zero padding: every layer's input is 0
// outside the grid.
#include <algorithm>

#include "common.h"

namespace adlbr {
namespace {

typedef short bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kT = 16;        // output tile edge
constexpr int kStride = 20;   // shorts per pixel in LDS (16 channels + pad)
constexpr int kR0 = kT + 8;   // r region edge (24)
constexpr int kR1 = kT + 6;   // layer-1 output edge (22), also the g1 region
constexpr int kR2 = kT + 4;   // layer-2 output edge (20), also the g2 region
constexpr int kR3 = kT + 2;   // layer-3 output edge (18)
constexpr int kG = 32;        // gate bytes per point (g1, g2)

// packed weight operands: [layer 1: 64 lanes][layer 2: 9 x 64][layer 3: 9 x 64][layer 4: 9 x 64]
constexpr int kPack1 = 0, kPack2 = 64, kPack3 = 64 + 9 * 64, kPack4 = 64 + 18 * 64;
constexpr int kPackEntries = 64 + 27 * 64;

// round to nearest even BF16 (one v_cvt_pk_bf16_f32 on gfx950)
__device__ __forceinline__ short bfbits(float f) { return __builtin_bit_cast(short, (__bf16)f); }
__device__ __forceinline__ float q8(uint32_t v) { return (float)v * (1.f / 255.f); }

// Pixel (py, px) of region index p of an R x R region, and the next pixel.
template <int R> struct Px {
    int y, x;
    __device__ __forceinline__ explicit Px(int p) : y(p / R), x(p % R) {}
    __device__ __forceinline__ void next() {
        if (++x == R) {
            x = 0;
            ++y;
        }
    }
};

// Store four channels c0 .. c0 + 3 of one pixel, each times its 8-bit
// gate (g4 holds the four gate bytes), as BF16 (one 8-byte LDS write).
__device__ __forceinline__ void store4(short *dst, f32x4 d, uint32_t g4, bool zero) {
    float v[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) v[c] = zero ? 0.f : d[c] * q8((g4 >> (8 * c)) & 0xffu);
    const uint32_t lo = (uint16_t)bfbits(v[0]) | ((uint32_t)(uint16_t)bfbits(v[1]) << 16);
    const uint32_t hi = (uint16_t)bfbits(v[2]) | ((uint32_t)(uint16_t)bfbits(v[3]) << 16);
    *(uint2 *)dst = make_uint2(lo, hi);
}

// One MFMA layer 16 -> 16: input region edge RI (LDS in), output edge RO;
// output gates from sg (LDS, pixel-major [GR * GR][16]; the output region
// sits at offset GO inside the gate region).  The product is taken as
// D[co][px] = W[co][ci] X[ci][px] (weights as the A operand, activations as
// B), so each lane ends with four consecutive channels of one pixel: one
// 4-byte gate read and one 8-byte store.  EDGE: the tile touches the grid
// boundary, so outputs outside the grid are set to 0.
template <int RI, int RO, int GR, int GO, bool EDGE>
__device__ __forceinline__ void mfma_layer(const short *__restrict__ sin, short *__restrict__ sout,
                                           const bf16x4 *wb, int gx0, int gy0, int nx, int ny,
                                           const uint8_t *__restrict__ sg) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    constexpr int npx = RO * RO;
    constexpr int ngroups = (npx + 15) / 16;
    const int n = lane & 15;            // B column / D column: the pixel in the group
    const int kq = (lane >> 4) * 4;     // channel quad of B (ci) and of D (co)
    for (int grp = wave; grp < ngroups; grp += 4) {
        const int pa = grp * 16 + n;    // this lane's pixel
        const bool va = pa < npx;
        const Px<RO> pxa(va ? pa : 0);
        const short *base = sin + (pxa.y * RI + pxa.x) * kStride + kq;
        f32x4 d = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int t = 0; t < 9; ++t) {
            bf16x4 b = *(const bf16x4 *)(base + ((t / 3) * RI + (t % 3)) * kStride);
            if (!va) b = bf16x4{0, 0, 0, 0};
            d = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(wb[t], b, d, 0, 0, 0);
        }
        if (!va) continue;
        const uint32_t g4 = *(const uint32_t *)(sg + ((pxa.y + GO) * GR + (pxa.x + GO)) * 16 + kq);
        bool zero = false;
        if (EDGE) {
            const int gx = gx0 + pxa.x, gy = gy0 + pxa.y;
            zero = gx < 0 || gx >= nx || gy < 0 || gy >= ny;
        }
        store4(sout + pa * kStride + kq, d, g4, zero);
    }
}

// Inputs of one tile, fetched into registers ahead of time: r on the 24x24
// region (0 outside the grid), g1 on 22x22 and g2 on 20x20 (16 bytes each).
constexpr int kRPer = (kR0 * kR0 + 255) / 256;                  // r values per thread
constexpr int kGPer = (kR1 * kR1 + kR2 * kR2 + 255) / 256;      // gate vectors per thread
struct TileIn {
    float r[kRPer];
    uint4 g[kGPer];
    float rp;  // r_prev at this thread's pixel of the 16x16 tile (fused dots)
};

__device__ __forceinline__ void fetch_tile(int x0, int y0, int nx, int ny,
                                           const float *__restrict__ r,
                                           const uint8_t *__restrict__ G8,
                                           const float *__restrict__ rp, TileIn &in) {
    const int tid = threadIdx.x;
    {
        const int gx = x0 + tid % kT, gy = y0 + tid / kT;
        in.rp = (rp && gx < nx && gy < ny) ? rp[gy * nx + gx] : 0.f;
    }
#pragma unroll
    for (int j = 0; j < kRPer; ++j) {
        const int k = tid + 256 * j;
        const int gx = x0 - 4 + k % kR0, gy = y0 - 4 + k / kR0;
        in.r[j] = (k < kR0 * kR0 && gx >= 0 && gx < nx && gy >= 0 && gy < ny) ? r[gy * nx + gx]
                                                                              : 0.f;
    }
#pragma unroll
    for (int j = 0; j < kGPer; ++j) {
        const int k = tid + 256 * j;
        const bool first = k < kR1 * kR1;
        const int kk = first ? k : k - kR1 * kR1;
        const int R = first ? kR1 : kR2, h = first ? 3 : 2;
        const int gx = x0 - h + kk % R, gy = y0 - h + kk / R;
        uint4 v = make_uint4(0u, 0u, 0u, 0u);
        if (k < kR1 * kR1 + kR2 * kR2 && gx >= 0 && gx < nx && gy >= 0 && gy < ny)
            v = ((const uint4 *)(G8 + (gy * nx + gx) * kG))[first ? 0 : 1];
        in.g[j] = v;
    }
}

__device__ __forceinline__ void stage_tile(const TileIn &in, float *sr, uint8_t *sg1, uint8_t *sg2,
                                           float *srp) {
    const int tid = threadIdx.x;
    srp[tid] = in.rp;
#pragma unroll
    for (int j = 0; j < kRPer; ++j) {
        const int k = tid + 256 * j;
        if (k < kR0 * kR0) sr[k] = in.r[j];
    }
#pragma unroll
    for (int j = 0; j < kGPer; ++j) {
        const int k = tid + 256 * j;
        if (k < kR1 * kR1) ((uint4 *)sg1)[k] = in.g[j];
        else if (k < kR1 * kR1 + kR2 * kR2) ((uint4 *)sg2)[k - kR1 * kR1] = in.g[j];
    }
}

// The four layers of one staged tile at (x0, y0).  EDGE: the tile's input
// region leaves the grid, so outputs outside the grid are zeroed.
template <bool EDGE>
__device__ __forceinline__ void net_tile(int x0, int y0, int nx, int ny,
                                         const float *__restrict__ F0, float *__restrict__ z,
                                         const float *__restrict__ rp, double &zr, double &zrp,
                                         const bf16x4 &wb1, const bf16x4 *wb2, const bf16x4 *wb3,
                                         const bf16x4 *wb4, const float *sr, const uint8_t *sg1,
                                         const uint8_t *sg2, short *s13, short *s2,
                                         const float *srp) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    auto inside = [&](int gx, int gy) {
        return !EDGE || (gx >= 0 && gx < nx && gy >= 0 && gy < ny);
    };
    // 1 / diag K at the output pixels of this lane in layer 4 (tile rows
    // wave, wave + 4, ...; lanes 0..15), loaded now so the load overlaps
    // layers 1-3
    float f0v[kT / 4];
#pragma unroll
    for (int j = 0; j < kT / 4; ++j) {
        const int gx = x0 + (lane & 15), gy = y0 + wave + 4 * j;
        f0v[j] = (lane < 16 && (!EDGE || (gx < nx && gy < ny))) ? F0[gy * nx + gx] : 0.f;
    }

    // layer 1 (1 -> 16) on 22x22: D[co][px] = W1[co][tap] X[tap][px], the
    // taps (4 per lane quad, 9..15 zero) as the K dimension
    {
        constexpr int npx = kR1 * kR1;
        const int n = lane & 15, kq = (lane >> 4) * 4;
        for (int grp = wave; grp < (npx + 15) / 16; grp += 4) {
            const int pa = grp * 16 + n;
            const bool va = pa < npx;
            const Px<kR1> pxa(va ? pa : 0);
            const float *rb = sr + pxa.y * kR0 + pxa.x;
            bf16x4 b;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const int t = kq + c;
                b[c] = (va && t < 9) ? bfbits(rb[(t / 3) * kR0 + (t % 3)]) : (short)0;
            }
            f32x4 d = {0.f, 0.f, 0.f, 0.f};
            d = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(wb1, b, d, 0, 0, 0);
            if (!va) continue;
            const uint32_t g4 = *(const uint32_t *)(sg1 + pa * 16 + kq);
            store4(s13 + pa * kStride + kq, d, g4, !inside(x0 - 3 + pxa.x, y0 - 3 + pxa.y));
        }
    }
    __syncthreads();
    mfma_layer<kR1, kR2, kR2, 0, EDGE>(s13, s2, wb2, x0 - 2, y0 - 2, nx, ny, sg2);
    __syncthreads();
    mfma_layer<kR2, kR3, kR1, 2, EDGE>(s2, s13, wb3, x0 - 1, y0 - 1, nx, ny, sg1);
    __syncthreads();

    // layer 4 (16 -> 1, no gate) on the 16x16 tile: D[co][px] with only row
    // co = 0 of the weights non-zero, so lanes 0..15 (c = 0) hold the 16
    // pixels of a tile row; then z = r / diag K + N(r)
    {
        const int n = lane & 15, kq = (lane >> 4) * 4;
#pragma unroll
        for (int j = 0; j < kT / 4; ++j) {
            const int grp = wave + 4 * j;  // group grp = one tile row: pixels (grp, 0..15)
            const short *base = s13 + (grp * kR3 + n) * kStride + kq;
            f32x4 d = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int t = 0; t < 9; ++t) {
                const bf16x4 b = *(const bf16x4 *)(base + ((t / 3) * kR3 + (t % 3)) * kStride);
                d = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(wb4[t], b, d, 0, 0, 0);
            }
            if (lane < 16) {
                const int gx = x0 + n, gy = y0 + grp;
                if (!EDGE || (gx < nx && gy < ny)) {
                    const int gi = gy * nx + gx;
                    const float rv = sr[(grp + 4) * kR0 + (n + 4)];
                    const float zv = rv * f0v[j] + d[0];
                    z[gi] = zv;
                    zr += (double)zv * (double)rv;
                    if (rp) zrp += (double)zv * (double)srp[grp * kT + n];
                }
            }
        }
    }
}

// Persistent over tiles: every block loads the packed weights once, and
// while it computes one tile the next tile's inputs are already in flight
// into registers (fetch_tile), then staged into LDS (stage_tile).
// With part given, the kernel also leaves the flexible-CG dot products
// <z, r> and <z, rp> (rp may be null) as per-block FP64 partials:
// part[blockIdx.x] and part[gridDim.x + blockIdx.x].
__global__ __launch_bounds__(256) void k_net2d_fused(int nx, int ny, const float *__restrict__ r,
                                                     const float *__restrict__ F0,
                                                     const uint8_t *__restrict__ G8,
                                                     const bf16x4 *__restrict__ wpack,
                                                     float *__restrict__ z,
                                                     const float *__restrict__ rp,
                                                     double *__restrict__ part,
                                                     const CgState *__restrict__ st) {
    if (st && (st->done || st->bad)) return;  // the solve has stopped: nothing reads z
    __shared__ __attribute__((aligned(16))) float sr[kR0 * kR0];
    __shared__ __attribute__((aligned(16))) uint8_t sg1[kR1 * kR1 * 16];
    __shared__ __attribute__((aligned(16))) uint8_t sg2[kR2 * kR2 * 16];
    // layer 1 output, later layer 3 output (s1 is dead once layer 2 has run)
    __shared__ __attribute__((aligned(16))) short s13[kR1 * kR1 * kStride];
    __shared__ __attribute__((aligned(16))) short s2[kR2 * kR2 * kStride];
    __shared__ float srp[kT * kT];
    const int lane = threadIdx.x & 63;
    const int ntx = (nx + kT - 1) / kT, ntiles = ntx * ((ny + kT - 1) / kT);
    // weight operands, packed per lane
    const bf16x4 wb1 = wpack[kPack1 + lane];
    bf16x4 wb2[9], wb3[9], wb4[9];
#pragma unroll
    for (int t = 0; t < 9; ++t) {
        wb2[t] = wpack[kPack2 + t * 64 + lane];
        wb3[t] = wpack[kPack3 + t * 64 + lane];
        wb4[t] = wpack[kPack4 + t * 64 + lane];
    }
    TileIn in;
    double zr = 0.0, zrp = 0.0;
    int tile = blockIdx.x;
    if (tile < ntiles) fetch_tile((tile % ntx) * kT, (tile / ntx) * kT, nx, ny, r, G8, rp, in);
    for (; tile < ntiles; tile += gridDim.x) {
        const int x0 = (tile % ntx) * kT, y0 = (tile / ntx) * kT;
        __syncthreads();  // the previous tile is done with the LDS buffers
        stage_tile(in, sr, sg1, sg2, srp);
        const int next = tile + gridDim.x;
        if (next < ntiles) fetch_tile((next % ntx) * kT, (next / ntx) * kT, nx, ny, r, G8, rp, in);
        __syncthreads();
        // interior tiles (the 24x24 input region inside the grid) skip every
        // bounds check; the branch is uniform over the block
        if (x0 >= 4 && y0 >= 4 && x0 + kT + 4 <= nx && y0 + kT + 4 <= ny)
            net_tile<false>(x0, y0, nx, ny, F0, z, rp, zr, zrp, wb1, wb2, wb3, wb4, sr, sg1, sg2,
                            s13, s2, srp);
        else
            net_tile<true>(x0, y0, nx, ny, F0, z, rp, zr, zrp, wb1, wb2, wb3, wb4, sr, sg1, sg2,
                           s13, s2, srp);
    }
    if (part) {  // block sums of the dots, in sr's storage (fixed order)
        double *red = (double *)sr;  // 256 doubles fit in the 24 x 24 floats
        for (int k = 0; k < 2; ++k) {
            __syncthreads();
            red[threadIdx.x] = k ? zrp : zr;
            __syncthreads();
            for (int st = 128; st > 0; st >>= 1) {
                if ((int)threadIdx.x < st) red[threadIdx.x] += red[threadIdx.x + st];
                __syncthreads();
            }
            if (threadIdx.x == 0) part[k * gridDim.x + blockIdx.x] = red[0];
        }
    }
}

// Pack the weight operands (expanded weights L1..L4, the A operands of
// D = W X) as BF16 in lane order: for layers 2 and 3 lane holds
// W[co = lane & 15][ci = 4 (lane >> 4) + c][t]; for layer 1
// W1[co = lane & 15][tap = 4 (lane >> 4) + c] (taps >= 9 are 0); for layer 4
// W4[ci = 4 (lane >> 4) + c][t] in row co = 0 only.
__global__ void k_pack_mfma(const float *__restrict__ L1, const float *__restrict__ L2,
                            const float *__restrict__ L3, const float *__restrict__ L4,
                            bf16x4 *__restrict__ out) {
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= kPackEntries) return;
    const int lane = e % 64;
    const int co = lane & 15, k0 = (lane >> 4) * 4;
    bf16x4 v;
    if (e < kPack2) {
#pragma unroll
        for (int c = 0; c < 4; ++c) v[c] = k0 + c < 9 ? bfbits(L1[co * 9 + k0 + c]) : (short)0;
    } else if (e < kPack4) {
        const bool second = e >= kPack3;
        const int t = ((e - (second ? kPack3 : kPack2)) / 64);
        const float *W = second ? L3 : L2;
#pragma unroll
        for (int c = 0; c < 4; ++c) v[c] = bfbits(W[(co * 16 + k0 + c) * 9 + t]);
    } else {  // A[co = lane & 15][ci = 4 (lane >> 4) + c], only row co = 0 non-zero
        const int t = (e - kPack4) / 64;
#pragma unroll
        for (int c = 0; c < 4; ++c) v[c] = co == 0 ? bfbits(L4[(k0 + c) * 9 + t]) : (short)0;
    }
    out[e] = v;
}


// ------------------------------------------------------------------ 3D --
// The 3D inference runs in three kernels: layers 1 and 2 together, layer 3,
// layer 4.  Activations cross HBM between them as BF16 [N][16] (32 bytes a
// point), gates as the 8-bit g1, g2 of every point.
//
// The 16 -> 16 layers walk the planes of a 16 x 8 column, a wave a row of 16
// points: an input plane and its halo, double buffered in LDS as 32 bytes a
// point (16 points of a row are 512 contiguous bytes, read without bank
// conflicts), feeds the three output planes that it neighbours, whose sums
// a wave holds, so that five LDS reads serve 15 matrix instructions, the 27
// taps of a row.  The next plane is on its way meanwhile, the
// weights stay in registers for the whole column, and only the column's own
// halo (180 points for 128) is read twice.
constexpr int k3X = 16, k3Y = 8;                         // output column
constexpr int k3HX = k3X + 2, k3HY = k3Y + 2, k3Plane = k3HX * k3HY;  // 180 staged points
constexpr int k3T = 27;
constexpr int k3BS = 64 * k3Y;                           // a wave per row

// Column c of the grid: its halo's origin and its planes [z0, z1).
struct Column {
    int x0, y0, z0, z1;
    __device__ __forceinline__ Column(const GridInfo &g, long long b, int chunk) {
        const int ntx = (g.nx + k3X - 1) / k3X, nty = (g.ny + k3Y - 1) / k3Y;
        x0 = (int)(b % ntx) * k3X - 1;
        y0 = (int)((b / ntx) % nty) * k3Y - 1;
        z0 = (int)(b / ((long long)ntx * nty)) * chunk;
        z1 = min(z0 + chunk, g.nz);
    }
    // in-plane index of a point of the halo grown by R, -1 outside the grid
    template <int R> __device__ __forceinline__ int at(const GridInfo &g, int h) const {
        const int x = x0 - R + h % (k3HX + 2 * R), y = y0 - R + h / (k3HX + 2 * R);
        return x >= 0 && x < g.nx && y >= 0 && y < g.ny ? x + g.nx * y : -1;
    }
};

// The A operands of a layer, per lane (row co = lane & 15): of each dz, four
// pairs of (dy, dx) taps (2 q, 2 q + 1) for v_mfma_f32_16x16x32_bf16, whose
// first 16 k are the first tap's channels, and the ninth tap's for
// v_mfma_f32_16x16x16_bf16.  A pair gives the bits that its two taps one
// after the other give, in the time of one.
typedef short bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8v __attribute__((ext_vector_type(8)));
constexpr int k3PackLayer = k3T * 64, k3PackPairs = 3 * 4 * 64 * 2;  // in bf16x4
struct Weights16 {
    bf16x8v w2[3][4];
    const bf16x4 *w1;  // the ninth taps' in LDS, [dz][lane]: layer 1 needs the registers
    __device__ __forceinline__ void load(const bf16x4 *__restrict__ pk, bf16x4 *lds) {
        const int lane = threadIdx.x & 63;
#pragma unroll
        for (int dz = 0; dz < 3; ++dz) {
#pragma unroll
            for (int q = 0; q < 4; ++q)
                w2[dz][q] = __builtin_bit_cast(bf16x8v, ((const bf16x8 *)pk)[(4 * dz + q) * 64 + lane]);
        }
        if (threadIdx.x < 3 * 64) lds[threadIdx.x] = pk[k3PackPairs + threadIdx.x];
        w1 = lds + lane;
    }
};

// Four gated channels as BF16.
__device__ __forceinline__ uint2 gated4(f32x4 d, uint32_t g4) {
    float v[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) v[c] = d[c] * q8((g4 >> (8 * c)) & 0xffu);
    return make_uint2((uint16_t)bfbits(v[0]) | ((uint32_t)(uint16_t)bfbits(v[1]) << 16),
                      (uint16_t)bfbits(v[2]) | ((uint32_t)(uint16_t)bfbits(v[3]) << 16));
}

// One wave's row of a 16 -> 16 layer along its column.  A lane holds four
// channels (4 (lane >> 4) + c) of point lane & 15.
struct Row16 {
    Weights16 W;
    f32x4 d0, d1, d2;  // output planes z - 1, z, z + 1 of input plane z
    int i;           // in-plane index of the lane's point, -1 outside
    uint32_t gate;   // its gates in plane z - 1
    __device__ __forceinline__ void init(const GridInfo &g, const Column &C, const bf16x4 *__restrict__ pk,
                                         bf16x4 *lds) {
        W.load(pk, lds);
        d0 = d1 = (f32x4){0.f, 0.f, 0.f, 0.f};
        gate = 0u;
        i = C.at<0>(g, (1 + (int)(threadIdx.x >> 6)) * k3HX + 1 + (int)(threadIdx.x & 15));
    }
    // requests the gates of plane z, for the next plane's end
    __device__ __forceinline__ void gates(const GridInfo &g, int z, const uint8_t *__restrict__ G8, int goff) {
        const long long nxy = (long long)g.nx * g.ny;
        gate = *(const uint32_t *)(G8 + 32 * (nxy * min(max(z, 0), g.nz - 1) + max(i, 0)) + goff +
                                   4 * ((threadIdx.x & 63) >> 4));
    }
    // input plane z (in sx; skipped outside the grid), its LDS reads all
    // requested before the first is waited for
    __device__ __forceinline__ void plane(const GridInfo &g, int z, const short *sx) {
        const int lane = threadIdx.x & 63, kg = lane >> 4;
        d2 = (f32x4){0.f, 0.f, 0.f, 0.f};
        if (z >= 0 && z < g.nz) {
            // a lane's tap of a pair: one point on, or from the end of a
            // halo row to the start of the next
            const short *row = sx + ((int)(threadIdx.x >> 6) * k3HX + (lane & 15)) * 16;
            const short *src = row + 8 * (kg & 1) + (kg & 2 ? 16 : 0);
            const short *wrap = row + 8 * (kg & 1) + (kg & 2 ? 16 * (k3HX - 2) : 0);
            bf16x8v x[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int t = 2 * q, o = (t / 3 * k3HX + t % 3) * 16;
                x[q] = __builtin_bit_cast(bf16x8v, *(const bf16x8 *)((t % 3 == 2 ? wrap : src) + o));
            }
            const bf16x4 x8 = *(const bf16x4 *)(row + 4 * kg + (2 * k3HX + 2) * 16);
            __builtin_amdgcn_sched_barrier(0);
            // every sum takes its taps in the order dz, dy, dx
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                d0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(W.w2[2][q], x[q], d0, 0, 0, 0);
                d1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(W.w2[1][q], x[q], d1, 0, 0, 0);
                d2 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(W.w2[0][q], x[q], d2, 0, 0, 0);
            }
            d0 = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(W.w1[64 * 2], x8, d0, 0, 0, 0);
            d1 = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(W.w1[64 * 1], x8, d1, 0, 0, 0);
            d2 = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(W.w1[64 * 0], x8, d2, 0, 0, 0);
        }
    }
    // output plane z - 1, complete with input plane z
    __device__ __forceinline__ void output(const GridInfo &g, const Column &C, int z, uint2 *__restrict__ out) {
        const long long nxy = (long long)g.nx * g.ny;
        if (z - 1 >= C.z0 && i >= 0)
            out[4 * (nxy * (z - 1) + i) + ((threadIdx.x & 63) >> 4)] = gated4(d0, gate);
        d0 = d1;
        d1 = d2;
    }
};

// Layers 1 and 2.  Layer 1 (1 -> 16, a1[p][co] = g1[p][co] sum_t W1[co][t]
// r(p + off_t), r = 0 outside the grid, tap t = (dz + 1) 9 + (dy + 1) 3 +
// (dx + 1)) runs in FP32 on v_mfma_f32_16x16x4_f32, seven for the 27 taps of
// 16 points, a plane ahead of layer 2 and straight into the LDS that layer 2
// reads: a1 does not cross HBM, at the price of taking 180 points for 128.
// r passes through a ring of four planes.
// 128^3: 45 + 77 us as two kernels in 8^3 tiles, 83 in columns.
constexpr int k3RX = k3HX + 2, k3RPlane = k3RX * (k3HY + 2);  // 240 points
__global__ __launch_bounds__(k3BS, 4) void k_net3d_l12(GridInfo g, int chunk,
                                                       const float *__restrict__ r,
                                                       const float *__restrict__ W1,
                                                       const bf16x4 *__restrict__ pk,
                                                       const uint8_t *__restrict__ G8,
                                                       uint2 *__restrict__ out,
                                                       const CgState *__restrict__ st) {
    if (st && (st->done || st->bad)) return;
    __shared__ float sr[4 * k3RPlane];
    __shared__ __attribute__((aligned(16))) short sx[2][k3Plane * 16];
    const Column C(g, xcd_block(blockIdx.x, gridDim.x), chunk);
    const long long nxy = (long long)g.nx * g.ny;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, n = lane & 15, kg = lane >> 4;
    __shared__ bf16x4 s1[3 * 64];
    Row16 R;
    R.init(g, C, pk, s1);
    // r: one point of a plane per thread
    const bool rt = threadIdx.x < k3RPlane;
    const int ri = rt ? C.at<1>(g, threadIdx.x) : -1;
    auto inr = [&](int z) { return ri >= 0 && z >= 0 && z < g.nz; };
    auto loadr = [&](int z) { return r[inr(z) ? nxy * z + ri : 0]; };  // dropped by inr where it is stored
    // layer 1: taps t = 4 j + kg of this lane, its weights in LDS (the
    // registers are layer 2's); twelve groups of 16 points, two to waves
    // 0 .. 3, so that each SIMD has three
    constexpr int kJ = (k3T + 3) / 4;
    __shared__ float sw[kJ * 64];
    for (int k = threadIdx.x; k < kJ * 64; k += k3BS) {
        const int t = 4 * (k / 64) + (k % 64 >> 4);
        const float v = W1[(k & 15) * k3T + min(t, k3T - 1)];
        sw[k] = t < k3T ? v : 0.f;
    }
    int off[kJ];
#pragma unroll
    for (int j = 0; j < kJ; ++j) {
        const int u = min(4 * j + kg, k3T - 1);
        off[j] = (u / 3 % 3) * k3RX + u % 3;
    }
    int hi[2], hs[2];  // in-plane index, point in sr
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int h = 16 * (wave + 8 * q) + n;
        hi[q] = h < k3Plane ? C.at<0>(g, h) : -1;
        hs[q] = h < k3Plane ? h / k3HX * k3RX + h % k3HX : 0;
    }
    auto loadg = [&](int z, int q) {
        return *(const uint32_t *)(G8 + 32 * (nxy * min(max(z, 0), g.nz - 1) + max(hi[q], 0)) + 4 * kg);
    };
    uint32_t g0 = loadg(C.z0 - 1, 0), g1 = loadg(C.z0 - 1, 1);
    auto layer1 = [&](int z) {  // plane z into sx[z & 1]
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            if (q == 1 && wave >= 4) break;
            // not the same value to the compiler, which would keep the sum
            // with every tap's offset in a register of its own
            asm volatile("" : "+v"(hs[q]));
            float x[kJ], w[kJ];
#pragma unroll
            for (int j = 0; j < kJ; ++j) {
                const int t = 4 * j + kg;
                x[j] = sr[((z - 1 + min(t, k3T - 1) / 9) & 3) * k3RPlane + hs[q] + off[j]];
                if (4 * j + 3 >= k3T) x[j] = t < k3T ? x[j] : 0.f;  // no tap: 0, whatever r holds
                w[j] = sw[64 * j + lane];
            }
            __builtin_amdgcn_sched_barrier(0);
            f32x4 d = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int j = 0; j < kJ; ++j) d = __builtin_amdgcn_mfma_f32_16x16x4f32(w[j], x[j], d, 0, 0, 0);
            uint2 v = gated4(d, q ? g1 : g0);
            if (hi[q] < 0) v = make_uint2(0u, 0u);  // layer 2's zero padding
            const int h = 16 * (wave + 8 * q) + n;
            if (h < k3Plane) *(uint2 *)(&sx[z & 1][h * 16 + 4 * kg]) = v;
        }
    };
    {
        float v[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = loadr(C.z0 - 2 + k);
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (rt) sr[((C.z0 - 2 + k) & 3) * k3RPlane + threadIdx.x] = inr(C.z0 - 2 + k) ? v[k] : 0.f;
    }
    float rv = loadr(C.z0 + 2);
    __syncthreads();
    if (C.z0 > 0) layer1(C.z0 - 1);
    g0 = loadg(C.z0, 0);
    g1 = loadg(C.z0, 1);
    __syncthreads();
    __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0): the weights, once
#pragma unroll 1
    for (int z = C.z0 - 1; z <= C.z1; ++z) {
        R.plane(g, z, sx[z & 1]);
        // what the last step has requested, then the next requests: nothing
        // waits for a load of its own step
        if (z + 1 <= C.z1 && z + 1 < g.nz) layer1(z + 1);
        if (rt) sr[((z + 3) & 3) * k3RPlane + threadIdx.x] = inr(z + 3) ? rv : 0.f;
        R.output(g, C, z, out);
        rv = loadr(z + 4);
        g0 = loadg(z + 2, 0);
        g1 = loadg(z + 2, 1);
        R.gates(g, z, G8, 16);
        __syncthreads();
    }
}

// Layer 3: out[p][co] = g1[p][co] sum_t sum_ci W_t[co][ci] in(p + off_t)[ci].
// 128^3: 77 us in 8^3 tiles, 46 in columns (5.0 TB/s of what it has to move).
__global__ __launch_bounds__(k3BS, 4) void k_net3d_l3(GridInfo g, int chunk, const uint4 *__restrict__ in,
                                                      const bf16x4 *__restrict__ pk,
                                                      const uint8_t *__restrict__ G8,
                                                      uint2 *__restrict__ out,
                                                      const CgState *__restrict__ st) {
    if (st && (st->done || st->bad)) return;
    __shared__ __attribute__((aligned(16))) short sx[2][k3Plane * 16];
    const Column C(g, xcd_block(blockIdx.x, gridDim.x), chunk);
    const long long nxy = (long long)g.nx * g.ny;
    __shared__ bf16x4 s1[3 * 64];
    Row16 R;
    R.init(g, C, pk, s1);
    // one 16-byte item of a plane per thread, two a point, 0 outside the grid
    static_assert(2 * k3Plane <= k3BS, "a plane in one item per thread");
    const bool it = threadIdx.x < 2 * k3Plane;
    const int hi = it ? C.at<0>(g, threadIdx.x >> 1) : -1;
    auto load = [&](int z) {
        return in[hi >= 0 && z >= 0 && z < g.nz ? 2 * (nxy * z + hi) + (threadIdx.x & 1) : 0];
    };
    auto store = [&](int z, uint4 q) {  // planes outside the grid are not read
        const bool ok = hi >= 0;
        if (it)
            *(uint4 *)(&sx[z & 1][8 * threadIdx.x]) =
                make_uint4(ok ? q.x : 0u, ok ? q.y : 0u, ok ? q.z : 0u, ok ? q.w : 0u);
    };
    store(C.z0 - 1, load(C.z0 - 1));
    uint4 v = load(C.z0);
    __syncthreads();
    __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0): the weights, once
#pragma unroll 1
    for (int z = C.z0 - 1; z <= C.z1; ++z) {
        R.plane(g, z, sx[z & 1]);
        store(z + 1, v);
        R.output(g, C, z, out);
        v = load(z + 2);
        R.gates(g, z, G8, 0);
        __syncthreads();
    }
}

// Layer 4 (16 -> 1) and the output: z = F0 r + sum_t sum_ci W4[ci][t]
// a3(p + off_t)[ci].  As an implicit GEMM it would use one row in 16 of the
// matrix instruction; taken the other way round it fills them: the 27 taps
// are the rows, P[t][p] = sum_ci W4[ci][t] a3(p)[ci] is two instructions for
// 16 points, and z sums P[t](p + off_t).  A block walks the planes of a
// 16 x 16 column of points, P of one plane and its halo in LDS (FP32),
// each thread one point of the plane with the sums of the three output
// planes that the input plane reaches; the next plane's a3 is in flight
// meanwhile.  With part, the block's FP64 partials of <z, r> in
// part[blockIdx] and of <z, rp> in part[gridDim + blockIdx].
// 128^3: 66 us as dot products over taps per point, 32 this way.
constexpr int k4X = 16, k4Y = 16, k4HX = k4X + 2, k4Halo = k4HX * (k4Y + 2);
constexpr int k4Groups = (k4Halo + 15) / 16, k4Per = (k4Groups + 3) / 4;
constexpr int k4P = 16 * k4Groups;  // 336 = 5 * 64 + 16: taps four apart in different banks
static_assert(k4P % 64 == 16, "tap planes staggered over the banks");
struct OutTile {
    int x0, y0, z0;  // halo origin = tile origin - 1
    __device__ __forceinline__ OutTile(const GridInfo &g, long long b, int chunk) {
        const int ntx = (g.nx + k4X - 1) / k4X, nty = (g.ny + k4Y - 1) / k4Y;
        x0 = (int)(b % ntx) * k4X - 1;
        y0 = (int)((b / ntx) % nty) * k4Y - 1;
        z0 = (int)(b / ((long long)ntx * nty)) * chunk - 1;
    }
};
__global__ __launch_bounds__(256) void k_net3d_l4(GridInfo g, int chunk, const uint2 *__restrict__ a3,
                                                  const bf16x4 *__restrict__ pk4,
                                                  const float *__restrict__ r,
                                                  const float *__restrict__ F0,
                                                  float *__restrict__ zout,
                                                  const float *__restrict__ rp,
                                                  double *__restrict__ part,
                                                  const CgState *__restrict__ st) {
    if (st && (st->done || st->bad)) return;
    __shared__ float P[k3T * k4P];
    const OutTile T(g, blockIdx.x, chunk);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, n = lane & 15, kg = lane >> 4;
    const bf16x4 wa = pk4[lane], wb = pk4[64 + lane];
    int hi[k4Per];  // in-plane index of this lane's halo points, -1 outside
#pragma unroll
    for (int j = 0; j < k4Per; ++j) {
        const int h = 16 * (wave + 4 * j) + n, x = T.x0 + h % k4HX, y = T.y0 + h / k4HX;
        hi[j] = h < k4Halo && x >= 0 && x < g.nx && y >= 0 && y < g.ny ? x + g.nx * y : -1;
    }
    const int nxy = g.nx * g.ny;
    const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
    const int px = T.x0 + 1 + tx, py = T.y0 + 1 + ty;
    const bool live = px < g.nx && py < g.ny;
    const int pi = live ? px + g.nx * py : 0;
    const int z1 = T.z0 + 1, zend = min(z1 + chunk, g.nz);  // output planes
    const int zlast = min(zend, g.nz - 1);                // last input plane
    bf16x4 x[k4Per];
    auto load = [&](int z) {
#pragma unroll
        for (int j = 0; j < k4Per; ++j) {
            const uint2 q = a3[4 * (long long)((long long)nxy * z + max(hi[j], 0)) + kg];
            x[j] = __builtin_bit_cast(bf16x4, hi[j] >= 0 ? q : make_uint2(0u, 0u));
        }
    };
    int z = max(T.z0, 0);
    load(z);
    float acc0 = 0.f, acc1 = 0.f;  // output planes z - 1, z
    float r0 = 0.f, f0 = 0.f, p0 = 0.f;  // of output plane z - 1
    double zr = 0.0, zrp = 0.0;
    const float *src = P + ty * k4HX + tx;
#pragma unroll 1
    for (;; ++z) {
        const bool out = z - 1 >= z1;  // plane z - 1 ends with this one
        const long long in = (long long)nxy * min(z, g.nz - 1) + pi;
        const float r1 = r[in], f1 = F0[in], p1 = (rp ? rp : r)[in];
        if (z <= zlast) {
#pragma unroll
            for (int j = 0; j < k4Per; ++j) {
                const int grp = wave + 4 * j;
                if (grp >= k4Groups) break;
                const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
                const f32x4 da = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(wa, x[j], zero, 0, 0, 0);
                const f32x4 db = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(wb, x[j], zero, 0, 0, 0);
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    P[(4 * kg + c) * k4P + 16 * grp + n] = da[c];
                    if (16 + 4 * kg + c < k3T) P[(16 + 4 * kg + c) * k4P + 16 * grp + n] = db[c];
                }
            }
            if (z < zlast) load(z + 1);
            __syncthreads();
        }
        float s0 = 0.f, s1 = 0.f, s2 = 0.f;  // to output planes z + 1, z, z - 1
        if (z <= zlast) {
#pragma unroll
            for (int t = 0; t < 9; ++t) {
                const float *q = src + t * k4P + (t / 3) * k4HX + t % 3;
                s0 += q[0];
                s1 += q[9 * k4P];
                s2 += q[18 * k4P];
            }
            __syncthreads();
        }
        if (out && live) {
            const float zi = f0 * r0 + (acc0 + s2);
            zout[(long long)nxy * (z - 1) + pi] = zi;
            zr += (double)zi * (double)r0;
            zrp += rp ? (double)zi * (double)p0 : 0.0;
        }
        if (z >= zend) break;
        acc0 = acc1 + s1;
        acc1 = s0;
        r0 = r1;
        f0 = f1;
        p0 = p1;
    }
    if (part) block_partial_sum2(zr, zrp, part, part + gridDim.x);
}

// The A operands of layers 2 and 3 (3D), then layer 4's: two of 16 taps.
constexpr int k3Pack4 = 2 * k3PackLayer, k3PackEntries = k3Pack4 + 2 * 64;
__global__ void k_pack_mfma3d(const float *__restrict__ L2, const float *__restrict__ L3,
                              const float *__restrict__ L4, bf16x4 *__restrict__ out) {
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= k3PackEntries) return;
    const bool last = e >= k3Pack4;
    const float *W = e >= k3PackLayer ? L3 : L2;
    const int k = e % k3PackLayer;
    int lane = e % 64, ci = 4 * (lane >> 4), t;
    if (last) {
        t = (e - k3Pack4) / 64 * 16 + (lane & 15);
    } else if (k < k3PackPairs) {  // two entries a lane
        lane = (k / 2) % 64;
        ci = 8 * ((lane >> 4) & 1) + 4 * (k & 1);
        t = k / 512 * 9 + 2 * (k / 128 % 4) + (lane >> 5);
    } else {
        t = (k - k3PackPairs) / 64 * 9 + 8;
    }
    bf16x4 v;
#pragma unroll
    for (int c = 0; c < 4; ++c)
        v[c] = !last ? bfbits(W[((lane & 15) * 16 + ci + c) * k3T + t])
               : t < k3T ? bfbits(L4[(ci + c) * k3T + t]) : (short)0;
    out[e] = v;
}

}  // namespace

// Offset (in floats) of the packed MFMA operands inside net->layers (2D).
constexpr size_t kPackOffset = 2 * 16 * 17 * 9;

int net_pack_mfma(const adlbr_net *net, hipStream_t s) {
    const float *L = net->layers;
    const size_t l2 = 16 * 9, l3 = l2 + 16 * 16 * 9, l4 = l3 + 16 * 16 * 9;
    hipLaunchKernelGGL(k_pack_mfma, dim3((kPackEntries + 255) / 256), dim3(256), 0, s, L, L + l2,
                       L + l3, L + l4, (bf16x4 *)(net->layers + kPackOffset));
    ADLBR_LAUNCH_CHECK();
    return ADLBR_OK;
}

// Planes a block of a 3D kernel walks: as many as leave `blocks` blocks.  Two
// more are read for its ends, and every plane is a wait of its own when the
// data are cold, so a grid that leaves CUs idle is cut into single planes
// (a first pass of 64^3 and less).
static int net3d_chunk(long long cols, int nz, long long blocks) {
    return (int)((cols * nz + blocks - 1) / blocks);
}
// The last kernel's: up to eight; 384 blocks and one more a column.
static int net3d_out_chunk(const GridInfo &g) {
    const long long cols = (long long)((g.nx + k4X - 1) / k4X) * ((g.ny + k4Y - 1) / k4Y);
    return cols >= 384 ? 8 : std::min(8, net3d_chunk(cols, g.nz, 384));
}
// Blocks of the last kernel, so partials of each dot.
long long net3d_tiles(const GridInfo &g) {
    const int chunk = net3d_out_chunk(g);
    return (long long)((g.nx + k4X - 1) / k4X) * ((g.ny + k4Y - 1) / k4Y) * ((g.nz + chunk - 1) / chunk);
}

// Packed 3D operands sit after the expanded 3D weights (T = 27).
constexpr size_t kPackOffset3 = 2 * 16 * 17 * 27;

int net_pack_mfma3d(const adlbr_net *net, hipStream_t s) {
    const float *L = net->layers;
    const size_t l2 = 16 * 27, l3 = l2 + 16 * 16 * 27, l4 = l3 + 16 * 16 * 27;
    static_assert(k3PackEntries * 2 <= 7168, "the packed operands fit the layers' reserve");
    hipLaunchKernelGGL(k_pack_mfma3d, dim3((k3PackEntries + 255) / 256), dim3(256), 0, s, L + l2,
                       L + l3, L + l4, (bf16x4 *)(net->layers + kPackOffset3));
    ADLBR_LAUNCH_CHECK();
    return ADLBR_OK;
}

int net_apply_mfma3d(const adlbr_net *net, const adlbr_operator *op, const float *r, float *z,
                     const float *rp, double *part, const CgState *st, hipStream_t s) {
    const GridInfo &g = operator_grid(op);
    const long long N = g.N;
    const float *L = net->layers;  // layer 1's weights come first
    const bf16x4 *pk = (const bf16x4 *)(net->layers + kPackOffset3);
    // activations as BF16 [N][16] in the two halves of the FP32 scratch
    uint4 *A = (uint4 *)net->scratch, *B = (uint4 *)(net->scratch + 8 * N);
    const long long cols = (long long)((g.nx + k3X - 1) / k3X) * ((g.ny + k3Y - 1) / k3Y);
    const int chunk = net3d_chunk(cols, g.nz, 512);  // two blocks a CU
    const unsigned nt = (unsigned)(cols * ((g.nz + chunk - 1) / chunk));
    hipLaunchKernelGGL(k_net3d_l12, dim3(nt), dim3(k3BS), 0, s, g, chunk, r, L, pk, net->gates8,
                       (uint2 *)B, st);
    hipLaunchKernelGGL(k_net3d_l3, dim3(nt), dim3(k3BS), 0, s, g, chunk, (const uint4 *)B,
                       pk + k3PackLayer, net->gates8, (uint2 *)A, st);
    hipLaunchKernelGGL(k_net3d_l4, dim3((unsigned)net3d_tiles(g)), dim3(256), 0, s, g,
                       net3d_out_chunk(g), (const uint2 *)A, pk + k3Pack4, r, net->features, z, rp, part, st);
    ADLBR_LAUNCH_CHECK();
    return ADLBR_OK;
}

// Blocks of the persistent inference grid for a grid of nx x ny points.
int net_mfma_blocks(int nx, int ny) {
    const int ntiles = ((nx + kT - 1) / kT) * ((ny + kT - 1) / kT);
    // three 51 KB blocks fit one CU's LDS: a persistent grid of 3 per CU
    return ntiles < 3 * 256 ? ntiles : 3 * 256;
}

int net_apply_mfma(const adlbr_net *net, const adlbr_operator *op, const float *r, float *z,
                   const float *rp, double *part, const CgState *st, hipStream_t s) {
    const GridInfo &g = operator_grid(op);
    hipLaunchKernelGGL(k_net2d_fused, dim3(net_mfma_blocks(g.nx, g.ny)), dim3(256), 0, s, g.nx,
                       g.ny, r, net->features, (const uint8_t *)net->gates8,
                       (const bf16x4 *)(net->layers + kPackOffset), z, rp, part, st);
    ADLBR_LAUNCH_CHECK();
    return ADLBR_OK;
}

}  // namespace adlbr
