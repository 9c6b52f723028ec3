// Learned preconditioner z = r / diag(K) + N(r) for K = I + dt A with
// N = B^T diag(g2) B, B = C2 diag(g1) C1 (symmetric positive semi-definite):
// features, gate net, the convolution stack on r, its backward pass, the
// energy loss and Adam -- everything the network needs to be trained and
// applied on the GPU.  These kernels are FP32 throughout (the convolutions and
// weight gradients on FP32 matrix instructions); the inference path used
// inside flexible CG has BF16 MFMA kernels in cnn_mfma.hip.
//
// N runs as a plain four-layer gated stack: the gate net writes expanded
// gates [g1, g2, g1, 1] and adlbr_net_gates expands the weights to
// [W1, W2, flip(W2)^T, flip(W1)^T] (the correlation adjoint is the
// correlation with channel-transposed, spatially flipped taps).  The
// backward pass runs on the expanded stack and folds the gradients of tied
// weights and repeated gates back onto the parameters.
//
// Layout: activations are [channels][N] FP32 planes; convolutions are 3^d
// taps with zero padding outside the grid; tap t = ((tz*3)+ty)*3+tx over
// offsets -1, 0, +1.
#include "common.h"

namespace adlbr {

int apply_K(const adlbr_operator *op, const void *u, void *out, double dt, hipStream_t s);
int apply_K_loss(const adlbr_operator *op, const void *u, void *out, double dt, hipStream_t s);
int net_apply_mfma(const adlbr_net *net, const adlbr_operator *op, const float *r, float *z,
                   const float *rp, double *part, const CgState *st, hipStream_t s);
int net_mfma_blocks(int nx, int ny);
int net_pack_mfma(const adlbr_net *net, hipStream_t s);
int net_pack_mfma3d(const adlbr_net *net, hipStream_t s);
int net_apply_mfma3d(const adlbr_net *net, const adlbr_operator *op, const float *r, float *z,
                     const float *rp, double *part, const CgState *st, hipStream_t s);
long long net3d_tiles(const GridInfo &g);

namespace {

constexpr int kBS = 256;

struct NetDims {
    int dim, W, H, nf, G, GX, T;
    // parameter offsets; expanded layer offsets (net->layers)
    size_t oWA, obA, oWB, obB, oW1, oW2, count;
    size_t l1, l2, l3, l4, lcount;
};

NetDims net_dims(int dim, int W, int H) {
    NetDims d;
    d.dim = dim;
    d.W = W;
    d.H = H;
    d.T = dim == 2 ? 9 : 27;
    d.nf = dim == 2 ? 7 : 13;
    d.G = 2 * W;       // gate-net outputs g1, g2
    d.GX = 3 * W + 1;  // expanded gates of the four-layer stack
    size_t o = 0;
    d.oWA = o; o += (size_t)H * d.nf * d.T;
    d.obA = o; o += H;
    d.oWB = o; o += (size_t)d.G * H;
    d.obB = o; o += d.G;
    d.oW1 = o; o += (size_t)W * d.T;
    d.oW2 = o; o += (size_t)W * W * d.T;
    d.count = o;
    o = 0;
    d.l1 = o; o += (size_t)W * d.T;
    d.l2 = o; o += (size_t)W * W * d.T;
    d.l3 = o; o += (size_t)W * W * d.T;
    d.l4 = o; o += (size_t)W * d.T;
    d.lcount = o;
    return d;
}

int check_net(const adlbr_operator *op, const adlbr_net *net, NetDims *d) {
    if (!op || !net || !net->params || !net->layers) {
        set_error("net: null argument (params and layers are required)");
        return ADLBR_E_INVALID;
    }
    const GridInfo &g = operator_grid(op);
    if (net->dim != g.dim || net->width != 16 || net->hidden != 16 ||
        net->nfeat != (g.dim == 2 ? 7 : 13)) {
        set_error("net: need dim = grid dim, width = hidden = 16, nfeat = %d", g.dim == 2 ? 7 : 13);
        return ADLBR_E_UNSUPPORTED;
    }
    *d = net_dims(g.dim, net->width, net->hidden);
    return ADLBR_OK;
}

struct Pt {
    int x, y, z;
};

__device__ __forceinline__ Pt coord_of(long long i, const GridInfo &g) {
    Pt p;
    p.x = (int)(i % g.nx);
    const long long r = i / g.nx;
    p.y = (int)(r % g.ny);
    p.z = (int)(r / g.ny);
    return p;
}

// neighbour of p at tap t (returns -1 outside the grid)
template <int DIM>
__device__ __forceinline__ long long tap_nb(const Pt &p, long long i, int t, const GridInfo &g) {
    const int dx = t % 3 - 1, dy = (t / 3) % 3 - 1, dz = DIM == 3 ? t / 9 - 1 : 0;
    const int x = p.x + dx, y = p.y + dy, z = p.z + dz;
    if (x < 0 || x >= g.nx || y < 0 || y >= g.ny || z < 0 || z >= g.nz) return -1;
    return i + dx + (long long)g.nx * (dy + (long long)g.ny * dz);
}

// ------------------------------------------------------------- features --
template <int DIM, typename TD>
__global__ void k_features(GridInfo g, const TD *diag, const float *w, const void *sbv, int wide,
                           double dt, float *F) {
    const long long i = (long long)blockIdx.x * kBS + threadIdx.x;
    const long long N = g.N;
    if (i >= N) return;
    constexpr int S = DIM == 2 ? 3 : 6;
    const double kd = 1.0 + dt * (double)diag[i];
    F[i] = (float)(1.0 / kd);
    double wq[S];
    for (int q = 0; q < S; ++q) {
        wq[q] = (double)w[widx<S>(q, i, N)];
        F[(1 + q) * N + i] = (float)(dt * wq[q] / kd);
    }
    // slots from the compact superbase form
    int o[6][3];
    if (DIM == 2) {
        int e0, e1, f0, f1;
        if (wide) {
            const short4 v = ((const short4 *)sbv)[i];
            e0 = v.x; e1 = v.y; f0 = v.z; f1 = v.w;
        } else {
            const char4 v = ((const char4 *)sbv)[i];
            e0 = v.x; e1 = v.y; f0 = v.z; f1 = v.w;
        }
        o[0][0] = e0; o[0][1] = e1; o[1][0] = f0; o[1][1] = f1;
        o[2][0] = -e0 - f0; o[2][1] = -e1 - f1;
    } else {
        for (int q = 0; q < 3; ++q)
            for (int c = 0; c < 3; ++c)
                o[q][c] = wide ? ((const int16_t *)sbv)[12 * i + 3 * q + c]
                               : ((const int8_t *)sbv)[12 * i + 3 * q + c];
        for (int c = 0; c < 3; ++c) {
            o[3][c] = -(o[0][c] + o[1][c]);
            o[4][c] = o[0][c] - o[2][c];
            o[5][c] = o[1][c] + o[2][c];
        }
    }
    if (DIM == 2) {
        double xx = 0, xy = 0, yy = 0;
        for (int q = 0; q < 3; ++q) {
            xx += 2 * wq[q] * o[q][0] * o[q][0];
            xy += 2 * wq[q] * o[q][0] * o[q][1];
            yy += 2 * wq[q] * o[q][1] * o[q][1];
        }
        double tr = xx + yy;
        tr = tr > 0 ? tr : 1.0;
        F[(1 + S) * N + i] = (float)(xx / tr);
        F[(2 + S) * N + i] = (float)(xy / tr);
        F[(3 + S) * N + i] = (float)(yy / tr);
    } else {
        const int pr[6][2] = {{0, 0}, {0, 1}, {0, 2}, {1, 1}, {1, 2}, {2, 2}};
        double Dc[6];
        for (int k = 0; k < 6; ++k) {
            Dc[k] = 0.0;
            for (int q = 0; q < 6; ++q) Dc[k] += 2 * wq[q] * o[q][pr[k][0]] * o[q][pr[k][1]];
        }
        double tr = Dc[0] + Dc[3] + Dc[5];
        tr = tr > 0 ? tr : 1.0;
        for (int k = 0; k < 6; ++k) F[(1 + S + k) * N + i] = (float)(Dc[k] / tr);
    }
}

// ------------------------------------------------------- convolutions --
typedef float f32x4v __attribute__((ext_vector_type(4)));

// Tiles of points of the convolution kernels, and the staged region (tile and
// a one-point halo): long in x, so that the planes are read and written in
// whole lines (16 -> 16 channels at 1024^2 with 16 x 16 tiles: 155 us).  CS,
// the LDS stride of a channel's plane, puts the four k-groups of an operand
// read on different banks.
template <int DIM> struct ConvTile;
template <> struct ConvTile<2> {
    static constexpr int TX = 64, TY = 4, TZ = 1, HX = 66, HY = 6, HZ = 1;
    static constexpr int CS = 400;
};
template <> struct ConvTile<3> {
    static constexpr int TX = 32, TY = 4, TZ = 4, HX = 34, HY = 6, HZ = 6;
    static constexpr int CS = 1232;
};

template <int DIM> struct TileAt {
    using C = ConvTile<DIM>;
    int x0, y0, z0;
    __device__ __forceinline__ TileAt(const GridInfo &g, int tile) {
        const int ntx = (g.nx + C::TX - 1) / C::TX, nty = (g.ny + C::TY - 1) / C::TY;
        x0 = (tile % ntx) * C::TX;
        y0 = (tile / ntx) % nty * C::TY;
        z0 = DIM == 3 ? tile / (ntx * nty) * C::TZ : 0;
    }
};

template <int DIM> long long conv_tiles(const GridInfo &g) {
    using C = ConvTile<DIM>;
    return (long long)((g.nx + C::TX - 1) / C::TX) * ((g.ny + C::TY - 1) / C::TY) *
           (DIM == 3 ? (g.nz + C::TZ - 1) / C::TZ : 1);
}

// Stage CH channel planes over a tile's halo region (origin x0 - 1, ... of
// HX x HY x HZ points, 0 outside the grid) in LDS, channel stride `stride`, each
// value times its gate (if given).  Wave w takes channels w * CW .. + CW, its
// lanes 64 points at a time; R x CW loads are issued before their stores.
template <typename C, int CH, int R>
__device__ __forceinline__ void stage_halo(const GridInfo &g, int x0, int y0, int z0,
                                           const float *__restrict__ in,
                                           const float *__restrict__ in_gate, float *sx, int stride) {
    constexpr int HP = C::HX * C::HY * C::HZ, CW = (CH + 3) / 4, NB = (HP + 63) / 64;
    const int lane = (int)(threadIdx.x & 63u), c0 = (int)(threadIdx.x >> 6) * CW;
#pragma unroll 1
    for (int b0 = 0; b0 < NB; b0 += R) {
        float v[R][CW], gt[R][CW];
#pragma unroll
        for (int b = 0; b < R; ++b) {
            const int q = (b0 + b) * 64 + lane;
            const int x = x0 - 1 + q % C::HX, y = y0 - 1 + (q / C::HX) % C::HY;
            const int z = C::HZ > 1 ? z0 - 1 + q / (C::HX * C::HY) : 0;
            const bool ok = q < HP && (unsigned)x < (unsigned)g.nx && (unsigned)y < (unsigned)g.ny &&
                            (unsigned)z < (unsigned)g.nz;
            const int idx = ok ? x + g.nx * (y + g.ny * z) : 0;
#pragma unroll
            for (int c = 0; c < CW; ++c) {
                const long long k = (c0 + c < CH ? c0 + c : 0) * g.N + idx;
                v[b][c] = in[k];
                gt[b][c] = in_gate ? in_gate[k] : 1.f;
                if (!ok) gt[b][c] = v[b][c] = 0.f;
            }
        }
#pragma unroll
        for (int b = 0; b < R; ++b)
#pragma unroll
            for (int c = 0; c < CW; ++c) {
                const int q = (b0 + b) * 64 + lane;
                if (q < HP && c0 + c < CH) sx[(c0 + c) * stride + q] = v[b][c] * gt[b][c];
            }
    }
}

// 3^d convolution on the matrix cores in FP32 (v_mfma_f32_16x16x4f32), as an
// implicit GEMM of 16 output channels by 16 points, K = input channels, tap by
// tap.  Blocks walk tiles: the input on the tile and halo is staged in LDS (all
// of a thread's loads first), the weights stay in registers as MFMA operands.
//   forward (ADJ = false): y[co] = sum_{t, ci} W[co][ci][t] in[ci](p + off_t)
//     (+ bias); pre = y (if given), out = y * gate (if given).
//   adjoint (ADJ): y[ci] = sum_{t, co} W[co][ci][t] in[co](p - off_t), the
//     gradient of the layer's input; the previous layer's gates follow at
//     once: out = y * gate, gsum += y * pre.
// KIN: channels of `in` (K), MOUT: output channels.  Bound by the matrix cores
// and the planes: 16 -> 16 at 1024^2 takes 31 us of MFMA and 200 MB.
template <int DIM, int KIN, int MOUT, bool ADJ>
__global__ __launch_bounds__(256, DIM == 2 ? (KIN > 8 ? 3 : 4) : 2) void k_conv_mfma(GridInfo g, int ntiles, const float *__restrict__ in,
                                                   const float *__restrict__ W,
                                                   const float *__restrict__ bias,
                                                   float *__restrict__ out,
                                                   float *__restrict__ pre_out,
                                                   const float *__restrict__ pre_in,
                                                   const float *__restrict__ gate,
                                                   float *__restrict__ gsum) {
    using C = ConvTile<DIM>;
    constexpr int T = DIM == 2 ? 9 : 27, KJ = (KIN + 3) / 4;
    constexpr int HP = C::HX * C::HY * C::HZ, TP = C::TX * C::TY * C::TZ, NG = TP / 64;
    __shared__ float sx[KJ * 4 * C::CS];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int i = lane & 15, kk = lane >> 4;
    const long long N = g.N;
    float a[T][KJ];
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
        for (int j = 0; j < KJ; ++j) {
            const int k = 4 * j + kk;
            a[t][j] = i < MOUT && k < KIN
                          ? W[ADJ ? (k * MOUT + i) * T + (T - 1 - t) : (i * KIN + k) * T + t]
                          : 0.f;
        }
    float bv[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) bv[c] = bias && 4 * kk + c < MOUT ? bias[4 * kk + c] : 0.f;
    // channels past KIN meet zero weights; they must be finite
    if (KIN % 4) {
        for (int e = tid; e < (KJ * 4 - KIN) * HP; e += 256) sx[(KIN + e / HP) * C::CS + e % HP] = 0.f;
    }
    for (int tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        const TileAt<DIM> t0(g, tile);
        __syncthreads();
        stage_halo<C, KIN, DIM == 2 ? 7 : 5>(g, t0.x0, t0.y0, t0.z0, in, nullptr, sx, C::CS);
        __syncthreads();
        // 16-point groups of a row; a wave takes a row of the tile in 2D, a
        // plane in 3D (two rows at a time)
        for (int r = 0; r < NG; r += 4) {
            f32x4v acc[4];
            int hb[4];
            long long pt[4];  // this lane's first output value, -1 past the grid
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                constexpr int RG = C::TX / 16;  // groups of a row
                const int x = (r + q) % RG * 16 + i;
                const int y = DIM == 2 ? wave : (r + q) / RG, z = DIM == 2 ? 0 : wave;
                hb[q] = (z * C::HY + y) * C::HX + x + kk * C::CS;  // tap (-1, -1, -1)
                const int gx = t0.x0 + x, gy = t0.y0 + y, gz = t0.z0 + z;
                pt[q] = gx < g.nx && gy < g.ny && gz < g.nz
                            ? 4 * kk * N + gx + g.nx * (gy + g.ny * gz) : -1;
                acc[q] = f32x4v{bv[0], bv[1], bv[2], bv[3]};
            }
            // what the results meet (from value 0 where there is no result):
            // requested before the products where the registers allow
            constexpr bool kEarly = DIM == 3 || !ADJ || KIN <= 8;
            float ge[4][4], pe[4][4], se[4][4];
            const auto meet = [&] {
#pragma unroll
                for (int q = 0; q < 4; ++q)
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        const long long o = pt[q] >= 0 && 4 * kk + c < MOUT ? pt[q] + c * N : 0;
                        ge[q][c] = gate ? gate[o] : 1.f;
                        pe[q][c] = ADJ ? pre_in[o] : 0.f;
                        se[q][c] = ADJ ? gsum[o] : 0.f;
                    }
            };
            if (kEarly) meet();
            // a tap's operands are read while the one before is multiplied; the
            // scheduling barriers keep the reads of later taps from moving up
            // (they filled the registers: 304 instead of 128)
            float x[2][KJ][4];
            const auto read = [&](int t) {
                const int off = ((t / 9) * C::HY + (t / 3) % 3) * C::HX + t % 3;
#pragma unroll
                for (int j = 0; j < KJ; ++j)
#pragma unroll
                    for (int q = 0; q < 4; ++q) x[t & 1][j][q] = sx[hb[q] + off + 4 * j * C::CS];
            };
            read(0);
#pragma unroll
            for (int t = 0; t < T; ++t) {
                if (t + 1 < T) read(t + 1);
#pragma unroll
                for (int j = 0; j < KJ; ++j)
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        acc[q] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[t][j], x[t & 1][j][q],
                                                                      acc[q], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
            if (!kEarly) meet();
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    if (pt[q] < 0 || 4 * kk + c >= MOUT) continue;
                    const long long o = pt[q] + c * N;
                    const float v = acc[q][c];
                    out[o] = v * ge[q][c];
                    if (ADJ) gsum[o] = se[q][c] + v * pe[q][c];
                    else if (pre_out) pre_out[o] = v;
                }
        }
    }
}

// Gate layer B (1x1) + sigmoid: g[k] = 1 / (1 + exp(-(WB[k] . relu(h) + bB[k]))),
// k < 2W, written expanded for the four-layer stack: Gout = [g1, g2, g1, 1]
// ([3W+1][N]); G8 holds g1, g2 per point as 8-bit fixed point round(255 g)
// ([N][2W]) for the inference kernel.
template <int H, int W>
__global__ __launch_bounds__(kBS) void k_gate_b(long long N, const float *__restrict__ h,
                                                const float *__restrict__ WB,
                                                const float *__restrict__ bB, float *__restrict__ Gout,
                                                uint8_t *__restrict__ G8) {
    constexpr int GX = 3 * W + 1;
    const long long i = (long long)blockIdx.x * kBS + threadIdx.x;
    if (i >= N) return;
    float hr[H];
#pragma unroll
    for (int c = 0; c < H; ++c) hr[c] = fmaxf(h[c * N + i], 0.f);
    static_assert(W % 8 == 0, "whole 16-byte groups of gates");
#pragma unroll 1
    for (int k0 = 0; k0 < 2 * W; k0 += 16) {
        uint32_t q[4] = {0u, 0u, 0u, 0u};  // sixteen gates, one store
#pragma unroll
        for (int k1 = 0; k1 < 16; ++k1) {
            const int k = k0 + k1;
            float a = bB[k];
#pragma unroll
            for (int c = 0; c < H; ++c) a += WB[k * H + c] * hr[c];
            const float gv = 1.f / (1.f + expf(-a));
            Gout[k * N + i] = gv;
            q[k1 >> 2] |= (uint32_t)(uint8_t)__float2int_rn(gv * 255.f) << (8 * (k1 & 3));
            if (k < W) Gout[(2 * W + k) * N + i] = gv;
        }
        if (!G8) continue;
        uint8_t *o = G8 + i * 2 * W + k0;
        if (((uintptr_t)G8 & 15) == 0) {  // the caller's buffer may start anywhere
            *(uint4 *)o = make_uint4(q[0], q[1], q[2], q[3]);
        } else {
#pragma unroll
            for (int b = 0; b < 16; ++b) o[b] = (uint8_t)(q[b >> 2] >> (8 * (b & 3)));
        }
    }
    Gout[(GX - 1) * N + i] = 1.f;
}

// Expanded layer weights: L1 = W1, L2 = W2, L3[o][i][t] = W2[i][o][T-1-t],
// L4[0][i][t] = W1[i][0][T-1-t].
__global__ void k_expand_weights(const float *__restrict__ W1, const float *__restrict__ W2,
                                 float *__restrict__ L, int W, int T, size_t l2, size_t l3,
                                 size_t l4) {
    const int n1 = W * T, n2 = W * W * T;
    for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < n2; e += gridDim.x * blockDim.x) {
        const int t = e % T, io = e / T, i = io % W, o = io / W;  // e = (o * W + i) * T + t
        L[l2 + e] = W2[e];
        L[l3 + e] = W2[(i * W + o) * T + (T - 1 - t)];
        if (e < n1) {
            const int tt = e % T, c = e / T;  // e = c * T + t
            L[e] = W1[e];
            L[l4 + e] = W1[c * T + (T - 1 - tt)];
        }
    }
}

// Fold the expanded-stack gradients onto the tied parameters:
// gW1 += gL1 + flip(gL4), gW2 += gL2 + flip(gL3)^T.
__global__ void k_fold_weight_grads(const float *__restrict__ gL, float *__restrict__ gW1,
                                    float *__restrict__ gW2, int W, int T, size_t l2, size_t l3,
                                    size_t l4) {
    const int n1 = W * T, n2 = W * W * T;
    for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < n2; e += gridDim.x * blockDim.x) {
        const int t = e % T, io = e / T, i = io % W, o = io / W;  // W2 index (o, i, t)
        gW2[e] += gL[l2 + e] + gL[l3 + (i * W + o) * T + (T - 1 - t)];
        if (e < n1) {
            const int tt = e % T, c = e / T;
            gW1[e] += gL[e] + gL[l4 + c * T + (T - 1 - tt)];
        }
    }
}

__global__ void k_fill_f32(float *p, long long n, float v) {
    const long long i = (long long)blockIdx.x * kBS + threadIdx.x;
    if (i < n) p[i] = v;
}

// z = r * F0 + out   (F0 = 1 / diag K)
__global__ void k_precond_out(long long N, const float *r, const float *F0, const float *o,
                              float *z) {
    const long long i = (long long)blockIdx.x * kBS + threadIdx.x;
    if (i < N) z[i] = r[i] * F0[i] + o[i];
}

// ------------------------------------------------------------ backward --
// ga = g * gate; ggate += g * pre   (per channel plane)
__global__ void k_gate_grad(long long n, const float *g, const float *gate, const float *pre,
                            float *ga, float *ggate) {
    const long long i = (long long)blockIdx.x * kBS + threadIdx.x;
    if (i >= n) return;
    const float gv = g[i];
    ga[i] = gv * gate[i];
    ggate[i] += gv * pre[i];
}

// Weight gradient of a 3^d layer on the matrix cores, dW[co][ci][t] = sum_p
// ga[co](p) x_ci(p + off_t) with x_ci = in[ci] (* in_gate[ci]), and the bias
// gradient db[co] = sum_p ga[co](p): GEMMs D_t[co][ci] += A[co][4 points]
// B_t[4 points][ci] with v_mfma_f32_16x16x4f32 (FP32 operands and
// accumulation).  Blocks walk tiles of points (2D 64 x 4, 3D 32 x 4 x 2): ga
// on the tile and x on the tile plus a one-point halo (0 outside the grid) are
// staged in LDS (every load of a thread is issued before its stores), then
// every wave takes a quarter of the tile's four-point steps for all taps.  The
// four waves' sums are added in LDS in wave order (the x buffer is reused for
// that once the tiles are done) and written as this block's partials
// [COUT * CIN * T weights, COUT biases].
// Bound by latency between the stagings: three blocks a CU, whole lines and
// unconflicted LDS strides took 16 x 16 at 1024^2 from 385 us (one block a CU,
// 16 x 16 tiles).
template <int DIM> struct GradTile;
template <> struct GradTile<2> {
    static constexpr int TX = 64, TY = 4, TZ = 1, HX = 66, HY = 6, HZ = 1;
};
template <> struct GradTile<3> {
    static constexpr int TX = 32, TY = 4, TZ = 2, HX = 34, HY = 6, HZ = 4;
};
template <int DIM> long long grad_tiles(const GridInfo &g) {
    using C = GradTile<DIM>;
    return (long long)((g.nx + C::TX - 1) / C::TX) * ((g.ny + C::TY - 1) / C::TY) *
           (DIM == 3 ? (g.nz + C::TZ - 1) / C::TZ : 1);
}

template <int DIM, int CIN, int COUT>
__global__ __launch_bounds__(256, DIM == 2 ? 3 : 2) void k_conv_bwd_w(GridInfo g, int ntiles, const float *__restrict__ in,
                                                    const float *__restrict__ in_gate,
                                                    const float *__restrict__ ga,
                                                    float *__restrict__ partials) {
    using C = GradTile<DIM>;
    constexpr int T = DIM == 2 ? 9 : 27;
    constexpr int TP = C::TX * C::TY * C::TZ, HP = C::HX * C::HY * C::HZ;
    static_assert(TP == 256 && CIN <= 16 && COUT <= 16, "one 16 x 16 MFMA tile");
    // channel strides of 4 modulo the 64 banks: the sixteen channels of an
    // operand read, four points each, fall on different banks
    constexpr int XS = (HP - 4 + 63) / 64 * 64 + 4, GS = TP + 4;
    static_assert(XS >= HP && XS % 64 == 4 && GS % 64 == 4, "strides");
    constexpr int stride = COUT * CIN * T + COUT;
    constexpr int SX = CIN * XS > stride ? CIN * XS : stride;
    __shared__ float sx[SX];  // x on the halo region; at the end the wave sums
    __shared__ float sg[COUT * GS];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int nx = g.nx, ny = g.ny, nz = g.nz;
    const int ntx = (nx + C::TX - 1) / C::TX, nty = (ny + C::TY - 1) / C::TY;
    const int i = lane & 15, kk = lane >> 4;  // A row (co) / B column (ci), k
    f32x4v acc[T];
#pragma unroll
    for (int t = 0; t < T; ++t) acc[t] = f32x4v{0.f, 0.f, 0.f, 0.f};
    float accb = 0.f;  // bias: sum of ga[co = i] over this lane's points
    for (int tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        const int x0 = tile % ntx * C::TX, y0 = tile / ntx % nty * C::TY,
                  z0 = DIM == 3 ? tile / (ntx * nty) * C::TZ : 0;
        __syncthreads();
        {
            stage_halo<C, CIN, 4>(g, x0, y0, z0, in, in_gate, sx, XS);
            // ga: one point of the tile per thread, all channels
            const int gx = x0 + tid % C::TX, gy = y0 + (tid / C::TX) % C::TY,
                      gz = DIM == 3 ? z0 + tid / (C::TX * C::TY) : 0;
            const bool ok = gx < nx && gy < ny && gz < nz;
            const long long k = ok ? ((long long)gz * ny + gy) * nx + gx : 0;
            float w[COUT];
#pragma unroll
            for (int co = 0; co < COUT; ++co) w[co] = ga[co * g.N + k];
#pragma unroll
            for (int co = 0; co < COUT; ++co) sg[co * GS + tid] = ok ? w[co] : 0.f;
        }
        __syncthreads();
        for (int ks = wave; ks < TP / 4; ks += 4) {
            const int p = ks * 4 + kk;
            const int px = p % C::TX, py = (p / C::TX) % C::TY, pz = p / (C::TX * C::TY);
            const float a = i < COUT ? sg[(i < COUT ? i : 0) * GS + p] : 0.f;
            accb += a;
            const int hb = (i < CIN ? i : 0) * XS + (pz * C::HY + py) * C::HX + px;
#pragma unroll
            for (int t = 0; t < T; ++t) {
                const int off = ((t / 9) * C::HY + (t / 3) % 3) * C::HX + t % 3;
                const float b = i < CIN ? sx[hb + off] : 0.f;
                acc[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, acc[t], 0, 0, 0);
            }
        }
    }
    // D: lane holds D[co = 4 (lane >> 4) + c][ci = lane & 15].  Bias: lanes
    // with the same co (i) hold disjoint point sets.
    for (int d = 16; d < 64; d <<= 1) accb += __shfl_xor(accb, d, 64);
    __syncthreads();  // the tiles are done with sx
    for (int w = 0; w < 4; ++w) {
        if (wave == w) {
#pragma unroll
            for (int t = 0; t < T; ++t)
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const int co = 4 * kk + c, ci = i;
                    if (co < COUT && ci < CIN) {
                        float &r = sx[(co * CIN + ci) * T + t];
                        r = w == 0 ? acc[t][c] : r + acc[t][c];
                    }
                }
            if (kk == 0 && i < COUT) {
                float &r = sx[COUT * CIN * T + i];
                r = w == 0 ? accb : r + accb;
            }
        }
        __syncthreads();
    }
    for (int e = tid; e < stride; e += 256) partials[(long long)blockIdx.x * stride + e] = sx[e];
}

// grad[k] += sum over blocks of partials[b][k]; weights go to gW[0 .. nw),
// biases (the last nb entries) to gb (if given).  64 columns a block, its
// sixteen wavefronts a sixteenth of the rows each (a chain of rounds of loads:
// 58 us with all rows in one thread), in FP64 in a fixed order.
constexpr int kRedWaves = 16;
__global__ __launch_bounds__(64 * kRedWaves) void k_reduce_partials(
    const float *__restrict__ partials, int nblocks, int stride, int nw, float *gW, float *gb) {
    __shared__ double red[kRedWaves][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int k = blockIdx.x * 64 + lane, kc = k < stride ? k : 0;
    double s = 0.0;
    int b = wave;
    for (; b + 7 * kRedWaves < nblocks; b += 8 * kRedWaves) {  // eight rows in flight
        float v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = partials[(long long)(b + kRedWaves * j) * stride + kc];
#pragma unroll
        for (int j = 0; j < 8; ++j) s += (double)v[j];
    }
    for (; b < nblocks; b += kRedWaves) s += (double)partials[(long long)b * stride + kc];
    red[wave][lane] = s;
    __syncthreads();
    if (wave != 0 || k >= stride) return;
    s = 0.0;
#pragma unroll
    for (int j = 0; j < kRedWaves; ++j) s += red[j][lane];
    if (k < nw) gW[k] += (float)s;
    else if (gb) gb[k - nw] += (float)s;
}

// Gate net backward from the gradients gx of the expanded gates ([3W+1][N]), in
// one pass over the points: the gates' gradients folded (dg1 = dG[0:W] +
// dG[2W:3W], dg2 = dG[W:2W]; the constant last gate has none), gg = dg g
// (1 - g), gh = (WB^T gg) * [h > 0] (written), and the 1x1 layer's weight
// gradient dWB[k][c] = sum_p gg[k] relu(h[c]), dbB[k] = sum_p gg[k]; the
// products on the matrix cores (FP32), the wave's 64 points staged in LDS
// (with WB in scalar registers, 512 of them, the loop spilled: 265 us).  Partials per block:
// [2W * H weights, 2W biases].  Bound by its planes: 48 + 32 + 16 read, 16
// written (1024^2: 470 MB).
template <int H, int W>
__global__ __launch_bounds__(256, 4) void k_gate_bwd(long long N, const float *__restrict__ gx,
                                                  const float *__restrict__ Gv,
                                                  const float *__restrict__ h,
                                                  const float *__restrict__ WB,
                                                  float *__restrict__ gh,
                                                  float *__restrict__ partials) {
    static_assert(H == 16 && W == 16, "two 16 x 16 MFMA tiles");
    constexpr int G = 2 * W, S = 68;  // LDS stride of a channel: 4 modulo the 64 banks
    __shared__ float sg[4][W * S];
    __shared__ float sh[4][H * S];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int i = lane & 15, kk = lane >> 4;
    float *mg = sg[wave], *mh = sh[wave];
    f32x4v acc[2] = {f32x4v{0.f, 0.f, 0.f, 0.f}, f32x4v{0.f, 0.f, 0.f, 0.f}};
    float accb[2] = {0.f, 0.f};
    float wb[2][4];  // WB^T as MFMA operands: row c = i, k = 16 m + 4 j + kk
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
        for (int j = 0; j < 4; ++j) wb[m][j] = WB[(16 * m + 4 * j + kk) * H + i];
    const long long nchunk = (N + 255) / 256;
    for (long long ch = blockIdx.x; ch < nchunk; ch += gridDim.x) {
        const long long p = ch * 256 + threadIdx.x;
        const bool ok = p < N;
        const long long q = ok ? p : 0;
        float hv[H];
#pragma unroll
        for (int c = 0; c < H; ++c) hv[c] = h[c * N + q];
        f32x4v a[4];  // gh of the wave's four 16-point groups
#pragma unroll
        for (int r = 0; r < 4; ++r) a[r] = f32x4v{0.f, 0.f, 0.f, 0.f};
        // g1's sixteen gates, then g2's: every load of the half first
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            float d[W], e[W], gv[W];
#pragma unroll
            for (int j = 0; j < W; ++j) {
                d[j] = gx[(m * W + j) * N + q];
                e[j] = m == 0 ? gx[(2 * W + j) * N + q] : 0.f;
                gv[j] = Gv[(m * W + j) * N + q];
            }
            if (m == 0) {
#pragma unroll
                for (int c = 0; c < H; ++c) mh[c * S + lane] = ok ? fmaxf(hv[c], 0.f) : 0.f;
            }
#pragma unroll
            for (int j = 0; j < W; ++j)
                mg[j * S + lane] = ok ? (d[j] + e[j]) * gv[j] * (1.f - gv[j]) : 0.f;
            // LDS serves a wave's reads after its writes; the barriers keep the
            // compiler from moving them
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int s = 0; s < 16; ++s) {
                const float av = mg[i * S + 4 * s + kk], b = mh[i * S + 4 * s + kk];
                accb[m] += av;
                acc[m] = __builtin_amdgcn_mfma_f32_16x16x4f32(av, b, acc[m], 0, 0, 0);
            }
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    a[r] = __builtin_amdgcn_mfma_f32_16x16x4f32(
                        wb[m][j], mg[(4 * j + kk) * S + 16 * r + i], a[r], 0, 0, 0);
            __builtin_amdgcn_wave_barrier();
        }
        // a: lane holds channels 4 kk + c of point 16 r + i of the wave
        const long long pw = ch * 256 + wave * 64;
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const long long pr = pw + 16 * r + i;
                const bool on = mh[(4 * kk + c) * S + 16 * r + i] > 0.f;
                if (pr < N) gh[(4 * kk + c) * N + pr] = on ? a[r][c] : 0.f;
            }
        __builtin_amdgcn_wave_barrier();
    }
#pragma unroll
    for (int m = 0; m < 2; ++m)
        for (int d = 16; d < 64; d <<= 1) accb[m] += __shfl_xor(accb[m], d, 64);
    // the waves' sums, in wave order
    constexpr int stride = G * H + G;
    static_assert(stride <= 4 * W * S, "the sums fit where the gates were");
    float *tot = sg[0];
    __syncthreads();
    for (int w = 0; w < 4; ++w) {
        if (wave == w) {
#pragma unroll
            for (int m = 0; m < 2; ++m) {
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    float &r = tot[(16 * m + 4 * kk + c) * H + i];
                    r = w == 0 ? acc[m][c] : r + acc[m][c];
                }
                if (kk == 0) {
                    float &r = tot[G * H + 16 * m + i];
                    r = w == 0 ? accb[m] : r + accb[m];
                }
            }
        }
        __syncthreads();
    }
    for (int e = threadIdx.x; e < stride; e += 256)
        partials[(long long)blockIdx.x * stride + e] = tot[e];
}

// ------------------------------------------------------------ loss, Adam --
struct LossState {
    double rr;
};

__global__ __launch_bounds__(kBS) void k_dot_self(long long N, const float *r, double *part) {
    const long long i = (long long)blockIdx.x * kBS + threadIdx.x;
    const double v = i < N ? (double)r[i] * (double)r[i] : 0.0;
    block_partial_sum(v, part);
}

__global__ __launch_bounds__(kFinish) void k_dot_self_fin(LossState *ls, const double *part,
                                                      long long nb) {
    const double t = reduce_partials(part, nb);
    if (threadIdx.x == 0) ls->rr = t;
}

// gz = (Kz - r) / rr  (Kz already in gz); partials of (z.Kz/2 - z.r) / rr
__global__ __launch_bounds__(kBS) void k_loss_grad(long long N, const float *z, const float *r,
                                                   float *gz, const LossState *ls, double *part) {
    const long long i = (long long)blockIdx.x * kBS + threadIdx.x;
    const double rr = ls->rr;
    double v = 0.0;
    if (i < N) {
        const double kz = (double)gz[i], zi = (double)z[i], ri = (double)r[i];
        v = (0.5 * zi * kz - zi * ri) / rr;
        gz[i] = (float)((kz - ri) / rr);
    }
    block_partial_sum(v, part);
}

// loss += sum of the partials
__global__ __launch_bounds__(kFinish) void k_loss_fin(const double *part, long long nb, double *loss) {
    const double t = reduce_partials(part, nb);
    if (threadIdx.x == 0) *loss += t;
}

__global__ void k_adam(float *p, const float *g, float *m, float *v, long long n, float gscale,
                       float lr, float b1, float b2, float eps, float c1, float c2) {
    const long long i = (long long)blockIdx.x * kBS + threadIdx.x;
    if (i >= n) return;
    const float gi = gscale * g[i];
    const float mi = b1 * m[i] + (1.f - b1) * gi;
    const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    p[i] -= lr * (mi / c1) / (sqrtf(vi / c2) + eps);
}

template <typename T>
__global__ void k_residual_vec(long long N, const T *b, const T *kx, T *r) {
    const long long i = (long long)blockIdx.x * kBS + threadIdx.x;
    if (i < N) r[i] = b[i] - kx[i];
}

// ------------------------------------------------------------- drivers --
unsigned nblk(long long N) { return (unsigned)((N + kBS - 1) / kBS); }

// Blocks of the tile-walking kernels: enough to fill 256 CUs a few times over
// (LDS and registers leave room for 3 to 6 a CU), fewer where there are fewer
// tiles.
constexpr int kWgBlocks = 768;

template <int DIM> unsigned conv_blocks(long long tiles) {
    constexpr long long most = DIM == 2 ? 768 : 512;
    return (unsigned)(tiles < most ? tiles : most);
}

template <int DIM>
int conv_launch(const GridInfo &g, int cin, int cout, const float *in, const float *W,
                const float *bias, float *out, float *pre, const float *gate, hipStream_t s) {
    const int nt = (int)conv_tiles<DIM>(g);  // N < 2^28
    const unsigned nb = conv_blocks<DIM>(nt);
#define ADLBR_CONV(CI, CO)                                                                     \
    if (cin == CI && cout == CO) {                                                             \
        hipLaunchKernelGGL((k_conv_mfma<DIM, CI, CO, false>), dim3(nb), dim3(256), 0, s, g, nt, \
                           in, W, bias, out, pre, nullptr, gate, nullptr);                     \
        return ADLBR_OK;                                                                       \
    }
    ADLBR_CONV(1, 16)
    ADLBR_CONV(16, 16)
    ADLBR_CONV(16, 1)
    ADLBR_CONV(7, 16)
    ADLBR_CONV(13, 16)
#undef ADLBR_CONV
    set_error("conv: unsupported channel counts %d -> %d", cin, cout);
    return ADLBR_E_UNSUPPORTED;
}

// Gradient of a layer's input from ga, then the previous layer's gates: out =
// gin * gate, ggate += gin * pre.
template <int DIM>
int bwd_data_launch(const GridInfo &g, int cin, int cout, const float *ga, const float *W,
                    const float *pre, const float *gate, float *out, float *ggate, hipStream_t s) {
    const int nt = (int)conv_tiles<DIM>(g);
    const unsigned nb = conv_blocks<DIM>(nt);
    if (cin == 16 && cout == 16) {
        hipLaunchKernelGGL((k_conv_mfma<DIM, 16, 16, true>), dim3(nb), dim3(256), 0, s, g, nt, ga, W,
                           nullptr, out, nullptr, pre, gate, ggate);
        return ADLBR_OK;
    }
    if (cin == 16 && cout == 1) {
        hipLaunchKernelGGL((k_conv_mfma<DIM, 1, 16, true>), dim3(nb), dim3(256), 0, s, g, nt, ga, W,
                           nullptr, out, nullptr, pre, gate, ggate);
        return ADLBR_OK;
    }
    set_error("conv backward: unsupported channel counts");
    return ADLBR_E_UNSUPPORTED;
}

void reduce_launch(const float *partials, int nblocks, int stride, int nw, float *gW, float *gb,
                   hipStream_t s) {
    hipLaunchKernelGGL(k_reduce_partials, dim3((stride + 63) / 64), dim3(64 * kRedWaves), 0, s, partials,
                       nblocks, stride, nw, gW, gb);
}

template <int DIM>
int bwd_w_launch(const GridInfo &g, int cin, int cout, const float *in, const float *in_gate,
                 const float *ga, float *partials, float *gW, float *gb, hipStream_t s) {
    const int nt = (int)grad_tiles<DIM>(g), nb = nt < kWgBlocks ? nt : kWgBlocks;
    constexpr int T = DIM == 2 ? 9 : 27;
#define ADLBR_BW(CI, CO)                                                                      \
    if (cin == CI && cout == CO) {                                                            \
        hipLaunchKernelGGL((k_conv_bwd_w<DIM, CI, CO>), dim3(nb), dim3(256), 0, s, g, nt, in,  \
                           in_gate, ga, partials);                                            \
        reduce_launch(partials, nb, CO * CI * T + CO, CO * CI * T, gW, gb, s);                \
        return ADLBR_OK;                                                                      \
    }
    ADLBR_BW(1, 16)
    ADLBR_BW(16, 16)
    ADLBR_BW(16, 1)
    ADLBR_BW(7, 16)
    ADLBR_BW(13, 16)
#undef ADLBR_BW
    set_error("conv weight gradient: unsupported channel counts");
    return ADLBR_E_UNSUPPORTED;
}

struct NetWs {
    float *g0, *g1, *ga, *gl, *partials;
    size_t total;
};

NetWs net_ws(long long N, const NetDims &d, char *base) {
    NetWs w;
    size_t o = 0;
    const size_t plane = align_up(4 * (size_t)N);
    w.g0 = (float *)(base + o);  o += 16 * plane;
    w.g1 = (float *)(base + o);  o += 16 * plane;
    w.ga = (float *)(base + o);  o += plane;
    w.gl = (float *)(base + o);  o += align_up(4 * d.lcount);
    w.partials = (float *)(base + o);
    o += align_up(4 * (size_t)kWgBlocks * (16 * 16 * d.T + 64));
    w.total = o;
    return w;
}

template <int DIM>
int forward_impl(const adlbr_operator *op, const adlbr_net *net, const NetDims &d, const float *r,
                 float *z, float *saved, float *bufA, float *bufB, hipStream_t s) {
    const GridInfo &g = operator_grid(op);
    const long long N = g.N;
    const float *L = net->layers;
    const float *G = net->gates;
    float *pre = saved;
    int rc;
    rc = conv_launch<DIM>(g, 1, 16, r, L + d.l1, nullptr, bufA, pre, G, s);
    if (rc) return rc;
    rc = conv_launch<DIM>(g, 16, 16, bufA, L + d.l2, nullptr, bufB, pre ? pre + 16 * N : nullptr,
                          G + 16 * N, s);
    if (rc) return rc;
    rc = conv_launch<DIM>(g, 16, 16, bufB, L + d.l3, nullptr, bufA, pre ? pre + 32 * N : nullptr,
                          G + 32 * N, s);
    if (rc) return rc;
    rc = conv_launch<DIM>(g, 16, 1, bufA, L + d.l4, nullptr, bufB, pre ? pre + 48 * N : nullptr,
                          G + 48 * N, s);
    if (rc) return rc;
    hipLaunchKernelGGL(k_precond_out, dim3(nblk(N)), dim3(kBS), 0, s, N, r, net->features, bufB, z);
    return ADLBR_OK;
}

}  // namespace

int net_apply(const adlbr_net *net, const adlbr_operator *op, double dt, const void *r, void *z,
              hipStream_t s) {
    (void)dt;
    NetDims d;
    int rc = check_net(op, net, &d);
    if (rc) return rc;
    if (operator_storage(op) != ADLBR_F32) {
        set_error("net: the operator's storage must be ADLBR_F32");
        return ADLBR_E_UNSUPPORTED;
    }
    if (d.dim == 2 && net->gates8)
        return net_apply_mfma(net, op, (const float *)r, (float *)z, nullptr, nullptr, nullptr, s);
    if (d.dim == 3 && net->gates8 && net->scratch)
        return net_apply_mfma3d(net, op, (const float *)r, (float *)z, nullptr, nullptr, nullptr,
                                s);
    if (!net->scratch) {
        set_error("net: the FP32 inference path needs net->scratch ([2W][N] FP32)");
        return ADLBR_E_INVALID;
    }
    const long long N = operator_grid(op).N;
    float *A = net->scratch, *B = net->scratch + 16 * N;
    return d.dim == 2 ? forward_impl<2>(op, net, d, (const float *)r, (float *)z, nullptr, A, B, s)
                      : forward_impl<3>(op, net, d, (const float *)r, (float *)z, nullptr, A, B, s);
}

namespace {
// Partials of <z, r> and <z, rp> (rp may be null) over 256-point blocks.
__global__ __launch_bounds__(kBS) void k_dots2(long long N, const float *__restrict__ z,
                                               const float *__restrict__ r,
                                               const float *__restrict__ rp, double *part) {
    const long long i = (long long)blockIdx.x * kBS + threadIdx.x;
    double a = 0.0, b = 0.0;
    if (i < N) {
        const double zi = (double)z[i];
        a = zi * (double)r[i];
        if (rp) b = zi * (double)rp[i];
    }
    block_partial_sum2(a, b, part, part + gridDim.x);
}
}  // namespace

int net_apply_dots(const adlbr_net *net, const adlbr_operator *op, const float *r,
                   const float *rp, float *z, double *part, long long *nparts,
                   const CgState *st, hipStream_t s) {
    NetDims d;
    int rc = check_net(op, net, &d);
    if (rc) return rc;
    const GridInfo &g = operator_grid(op);
    if (d.dim == 2 && net->gates8 && operator_storage(op) == ADLBR_F32) {
        *nparts = net_mfma_blocks(g.nx, g.ny);
        return net_apply_mfma(net, op, r, z, rp, part, st, s);
    }
    if (d.dim == 3 && net->gates8 && net->scratch && operator_storage(op) == ADLBR_F32) {
        *nparts = net3d_tiles(g);
        return net_apply_mfma3d(net, op, r, z, rp, part, st, s);
    }
    rc = net_apply(net, op, 0.0, r, z, s);
    if (rc) return rc;
    *nparts = nblk(g.N);
    hipLaunchKernelGGL(k_dots2, dim3((unsigned)*nparts), dim3(kBS), 0, s, g.N, (const float *)z, r,
                       rp, part);
    return ADLBR_OK;
}

long long net_dot_parts(const GridInfo &g) {
    const long long fused = g.dim == 2 ? (long long)net_mfma_blocks(g.nx, g.ny) : net3d_tiles(g);
    const long long nb = nblk(g.N);
    return fused > nb ? fused : nb;
}

}  // namespace adlbr

using namespace adlbr;

extern "C" int adlbr_net_param_count(int dim, int width, int hidden, size_t *count) {
    clear_error();
    if ((dim != 2 && dim != 3) || width != 16 || hidden != 16 || !count) {
        set_error("adlbr_net_param_count: dim 2/3, width = hidden = 16");
        return ADLBR_E_INVALID;
    }
    *count = net_dims(dim, width, hidden).count;
    return ADLBR_OK;
}

extern "C" int adlbr_net_workspace(adlbr_operator *op, const adlbr_net *net, size_t *bytes) {
    clear_error();
    NetDims d;
    int rc = check_net(op, net, &d);
    if (rc) return rc;
    if (!bytes) return ADLBR_E_INVALID;
    *bytes = net_ws(operator_grid(op).N, d, nullptr).total;
    return ADLBR_OK;
}

extern "C" int adlbr_net_features(adlbr_operator *op, double dt, adlbr_net *net, void *stream) {
    clear_error();
    NetDims d;
    int rc = check_net(op, net, &d);
    if (rc) return rc;
    if (!net->features || !(dt >= 0.0)) {
        set_error("adlbr_net_features: need net->features and dt >= 0");
        return ADLBR_E_INVALID;
    }
    if (operator_storage(op) != ADLBR_F32) {
        set_error("adlbr_net_features: the operator's storage must be ADLBR_F32");
        return ADLBR_E_UNSUPPORTED;
    }
    const GridInfo &g = operator_grid(op);
    hipStream_t s = as_stream(stream);
    const float *w = (const float *)operator_weights(op);
    if (g.dim == 2)
        hipLaunchKernelGGL((k_features<2, float>), dim3(nblk(g.N)), dim3(kBS), 0, s, g,
                           (const float *)operator_diag(op), w, operator_slots(op),
                           operator_wide(op), dt, net->features);
    else
        hipLaunchKernelGGL((k_features<3, float>), dim3(nblk(g.N)), dim3(kBS), 0, s, g,
                           (const float *)operator_diag(op), w, operator_slots(op),
                           operator_wide(op), dt, net->features);
    ADLBR_LAUNCH_CHECK();
    return ADLBR_OK;
}

extern "C" int adlbr_net_gates(adlbr_operator *op, adlbr_net *net, void *stream) {
    clear_error();
    NetDims d;
    int rc = check_net(op, net, &d);
    if (rc) return rc;
    if (!net->features || !net->hidden_act || !net->gates) {
        set_error("adlbr_net_gates: need features, hidden_act and gates buffers");
        return ADLBR_E_INVALID;
    }
    const GridInfo &g = operator_grid(op);
    hipStream_t s = as_stream(stream);
    const float *P = net->params;
    rc = g.dim == 2 ? conv_launch<2>(g, d.nf, 16, net->features, P + d.oWA, P + d.obA,
                                     net->hidden_act, nullptr, nullptr, s)
                    : conv_launch<3>(g, d.nf, 16, net->features, P + d.oWA, P + d.obA,
                                     net->hidden_act, nullptr, nullptr, s);
    if (rc) return rc;
    hipLaunchKernelGGL((k_gate_b<16, 16>), dim3(nblk(g.N)), dim3(kBS), 0, s, g.N,
                       (const float *)net->hidden_act, P + d.oWB, P + d.obB, net->gates,
                       net->gates8);
    hipLaunchKernelGGL(k_expand_weights, dim3(16), dim3(kBS), 0, s, P + d.oW1, P + d.oW2,
                       net->layers, d.W, d.T, d.l2, d.l3, d.l4);
    rc = g.dim == 2 ? net_pack_mfma(net, s) : net_pack_mfma3d(net, s);
    if (rc) return rc;
    ADLBR_LAUNCH_CHECK();
    return ADLBR_OK;
}

extern "C" int adlbr_net_forward(adlbr_operator *op, const adlbr_net *net, const float *r, float *z,
                                 float *saved, void *stream) {
    clear_error();
    NetDims d;
    int rc = check_net(op, net, &d);
    if (rc) return rc;
    if (!r || !z || !net->gates || !net->features) {
        set_error("adlbr_net_forward: null argument");
        return ADLBR_E_INVALID;
    }
    const GridInfo &g = operator_grid(op);
    hipStream_t s = as_stream(stream);
    if (!net->scratch) {
        set_error("adlbr_net_forward: net->scratch ([2W][N] FP32) is required");
        return ADLBR_E_INVALID;
    }
    float *A = net->scratch, *B = net->scratch + 16 * g.N;
    rc = g.dim == 2 ? forward_impl<2>(op, net, d, r, z, saved, A, B, s)
                    : forward_impl<3>(op, net, d, r, z, saved, A, B, s);
    if (rc) return rc;
    ADLBR_LAUNCH_CHECK();
    return ADLBR_OK;
}

extern "C" int adlbr_net_precondition(adlbr_operator *op, const adlbr_net *net, const float *r,
                                      float *z, void *stream) {
    clear_error();
    if (!r || !z || r == z) {
        set_error("adlbr_net_precondition: null or aliased argument");
        return ADLBR_E_INVALID;
    }
    return net_apply(net, op, 0.0, r, z, as_stream(stream));
}

extern "C" int adlbr_net_backward(adlbr_operator *op, const adlbr_net *net, const float *r,
                                  const float *gz, const float *saved, float *gparams,
                                  float *ggates, void *workspace, size_t ws_bytes, void *stream) {
    clear_error();
    NetDims d;
    int rc = check_net(op, net, &d);
    if (rc) return rc;
    if (!r || !gz || !saved || !gparams || !ggates || !workspace) {
        set_error("adlbr_net_backward: null argument");
        return ADLBR_E_INVALID;
    }
    const GridInfo &g = operator_grid(op);
    const long long N = g.N;
    NetWs w = net_ws(N, d, (char *)workspace);
    if (ws_bytes < w.total) {
        set_error("adlbr_net_backward: workspace has %zu bytes, %zu needed", ws_bytes, w.total);
        return ADLBR_E_NOMEM;
    }
    hipStream_t s = as_stream(stream);
    const float *L = net->layers;
    const float *G = net->gates;
    // gradients of the expanded layers go to w.gl, then fold onto W1, W2
    hipLaunchKernelGGL(k_fill_f32, dim3(nblk((long long)d.lcount)), dim3(kBS), 0, s, w.gl,
                       (long long)d.lcount, 0.f);
    // layer 4: out = pre4 * G[48]; dL/dout = gz
    const size_t offs[4] = {0, 16, 32, 48};
    const int cins[4] = {1, 16, 16, 16}, couts[4] = {16, 16, 16, 1};
    const size_t oW[4] = {d.l1, d.l2, d.l3, d.l4};
    // ga: the gradient of a layer's pre-gate output; the last layer's here, the
    // others' with their gates' gradients as the layer above is passed back
    float *gbuf[2] = {w.g0, w.g1};
    const float *ga = w.ga;
    hipLaunchKernelGGL(k_gate_grad, dim3(nblk(N)), dim3(kBS), 0, s, N, gz, G + 48 * N,
                       saved + 48 * N, w.ga, ggates + 48 * N);
    for (int l = 3; l >= 0; --l) {
        // input of layer l: r, or the previous layer's pre-gate output times its gates
        const float *in = l == 0 ? r : saved + offs[l - 1] * N;
        const float *in_gate = l == 0 ? nullptr : G + offs[l - 1] * N;
        rc = g.dim == 2 ? bwd_w_launch<2>(g, cins[l], couts[l], in, in_gate, ga, w.partials,
                                          w.gl + oW[l], nullptr, s)
                        : bwd_w_launch<3>(g, cins[l], couts[l], in, in_gate, ga, w.partials,
                                          w.gl + oW[l], nullptr, s);
        if (rc) return rc;
        if (l > 0) {
            float *gin = gbuf[l & 1];
            rc = g.dim == 2 ? bwd_data_launch<2>(g, cins[l], couts[l], ga, L + oW[l], in, in_gate,
                                                 gin, ggates + offs[l - 1] * N, s)
                            : bwd_data_launch<3>(g, cins[l], couts[l], ga, L + oW[l], in, in_gate,
                                                 gin, ggates + offs[l - 1] * N, s);
            if (rc) return rc;
            ga = gin;
        }
    }
    hipLaunchKernelGGL(k_fold_weight_grads, dim3(16), dim3(kBS), 0, s, (const float *)w.gl,
                       gparams + d.oW1, gparams + d.oW2, d.W, d.T, d.l2, d.l3, d.l4);
    ADLBR_LAUNCH_CHECK();
    return ADLBR_OK;
}

extern "C" int adlbr_net_gates_backward(adlbr_operator *op, const adlbr_net *net,
                                        const float *ggates, float *gparams, void *workspace,
                                        size_t ws_bytes, void *stream) {
    clear_error();
    NetDims d;
    int rc = check_net(op, net, &d);
    if (rc) return rc;
    if (!ggates || !gparams || !workspace || !net->hidden_act) {
        set_error("adlbr_net_gates_backward: null argument");
        return ADLBR_E_INVALID;
    }
    const GridInfo &g = operator_grid(op);
    const long long N = g.N;
    NetWs w = net_ws(N, d, (char *)workspace);
    if (ws_bytes < w.total) {
        set_error("adlbr_net_gates_backward: workspace too small");
        return ADLBR_E_NOMEM;
    }
    hipStream_t s = as_stream(stream);
    const float *P = net->params;
    // gh (in w.g0) and the gradients of WB, bB, then those of WA, bA from gh
    const long long nchunk = (N + 255) / 256;
    const int nb = (int)(nchunk < kWgBlocks ? nchunk : kWgBlocks);
    hipLaunchKernelGGL((k_gate_bwd<16, 16>), dim3(nb), dim3(256), 0, s, N, ggates,
                       (const float *)net->gates, (const float *)net->hidden_act, P + d.oWB, w.g0,
                       w.partials);
    reduce_launch(w.partials, nb, 32 * 16 + 32, 32 * 16, gparams + d.oWB, gparams + d.obB, s);
    rc = g.dim == 2 ? bwd_w_launch<2>(g, d.nf, 16, net->features, nullptr, w.g0, w.partials,
                                      gparams + d.oWA, gparams + d.obA, s)
                    : bwd_w_launch<3>(g, d.nf, 16, net->features, nullptr, w.g0, w.partials,
                                      gparams + d.oWA, gparams + d.obA, s);
    if (rc) return rc;
    ADLBR_LAUNCH_CHECK();
    return ADLBR_OK;
}

extern "C" int adlbr_net_loss_grad(adlbr_operator *op, double dt, const float *r, const float *z,
                                   float *gz, double *loss, void *workspace, size_t ws_bytes,
                                   void *stream) {
    clear_error();
    if (!op || !r || !z || !gz || !loss || !workspace || operator_storage(op) != ADLBR_F32) {
        set_error("adlbr_net_loss_grad: bad argument (FP32 operator required)");
        return ADLBR_E_INVALID;
    }
    const long long N = operator_grid(op).N;
    const size_t need = align_up(sizeof(LossState)) + align_up(8 * (size_t)nblk(N) + 64);
    if (ws_bytes < need) {
        set_error("adlbr_net_loss_grad: workspace too small");
        return ADLBR_E_NOMEM;
    }
    hipStream_t s = as_stream(stream);
    LossState *ls = (LossState *)workspace;
    double *part = (double *)((char *)workspace + align_up(sizeof(LossState)));
    const long long nb = nblk(N);
    hipLaunchKernelGGL(k_dot_self, dim3(nb), dim3(kBS), 0, s, N, r, part);
    hipLaunchKernelGGL(k_dot_self_fin, dim3(1), dim3(kFinish), 0, s, ls, (const double *)part, nb);
    int rc = apply_K_loss(op, z, gz, dt, s);  // gz = K z
    if (rc) return rc;
    hipLaunchKernelGGL(k_loss_grad, dim3(nb), dim3(kBS), 0, s, N, z, r, gz, (const LossState *)ls,
                       part);
    hipLaunchKernelGGL(k_loss_fin, dim3(1), dim3(kFinish), 0, s, (const double *)part, nb, loss);
    ADLBR_LAUNCH_CHECK();
    return ADLBR_OK;
}

extern "C" int adlbr_net_adam(float *params, const float *grads, float *m, float *v, int64_t n,
                              int32_t step, double grad_scale, double lr, double beta1,
                              double beta2, double eps, void *stream) {
    clear_error();
    if (!params || !grads || !m || !v || n < 1 || step < 1 || !(grad_scale > 0.0)) {
        set_error("adlbr_net_adam: bad argument");
        return ADLBR_E_INVALID;
    }
    const float c1 = (float)(1.0 - pow(beta1, step)), c2 = (float)(1.0 - pow(beta2, step));
    hipLaunchKernelGGL(k_adam, dim3(nblk(n)), dim3(kBS), 0, as_stream(stream), params, grads, m, v,
                       (long long)n, (float)grad_scale, (float)lr, (float)beta1, (float)beta2, (float)eps, c1, c2);
    ADLBR_LAUNCH_CHECK();
    return ADLBR_OK;
}

extern "C" int adlbr_residual(adlbr_operator *op, double dt, const void *b, const void *x, void *r,
                              void *stream) {
    clear_error();
    if (!op || !b || !x || !r || r == x) {
        set_error("adlbr_residual: null or aliased argument");
        return ADLBR_E_INVALID;
    }
    hipStream_t s = as_stream(stream);
    const long long N = operator_grid(op).N;
    int rc = apply_K(op, x, r, dt, s);  // r = K x
    if (rc) return rc;
    const int sto = operator_storage(op);
    if (sto == ADLBR_F32)
        hipLaunchKernelGGL(k_residual_vec<float>, dim3(nblk(N)), dim3(kBS), 0, s, N,
                           (const float *)b, (const float *)r, (float *)r);
    else if (sto == ADLBR_F64)
        hipLaunchKernelGGL(k_residual_vec<double>, dim3(nblk(N)), dim3(kBS), 0, s, N,
                           (const double *)b, (const double *)r, (double *)r);
    else {
        set_error("adlbr_residual: storage must be F32 or F64");
        return ADLBR_E_UNSUPPORTED;
    }
    ADLBR_LAUNCH_CHECK();
    return ADLBR_OK;
}
