// Learned initial guess for the forward PCG solves: a four-layer 3x3x3
// convolutional network on the node lattice (channels 3 -> 16 -> 16 -> 16 -> 1,
// ReLU between layers, zero padding), BF16 weights and activations, FP32
// accumulation on MFMA, trained on the device.
//
// Inputs per illumination k (nodal): log(mu/mu0), log(kappa/kappa0) and
// log(phi_hom,k), the fluence of the homogeneous (kappa0, mu0) medium for that
// source. Output: the log correction, phi0 = phi_hom,k exp(net). The solve that
// starts from phi0 stops on the same ||b - K x|| <= rtol ||b|| as a zero start.
//
// Convolutions are implicit GEMMs on the 16x16x16 BF16 MFMA over 16 output
// channels x 16 lattice points; the K dimension is one tap x 16 input channels
// (or four taps x 4 channels for the 3-channel input layer, padded to 4). Weight gradients are the same product with the voxel
// index as the K dimension, split over wavefronts and reduced in fixed order.
#include <cmath>

#include "qpat_internal.h"

namespace qpat {
namespace {

typedef short s4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));

constexpr int kLayers = 4;
constexpr int kCin[kLayers] = {3, 16, 16, 16};
constexpr int kCout[kLayers] = {16, 16, 16, 1};
constexpr int kParams = 15601;

__host__ __device__ inline int param_offset(int layer) {
    int off = 0;
    for (int l = 0; l < layer; ++l) off += kCout[l] * kCin[l] * 27 + kCout[l];
    return off;
}

__device__ __forceinline__ uint16_t f2bf(float f) {
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7f800000u) == 0x7f800000u) return static_cast<uint16_t>(u >> 16);  // inf / nan
    u += 0x7fffu + ((u >> 16) & 1u);                                              // round to nearest even
    return static_cast<uint16_t>(u >> 16);
}

__device__ __forceinline__ float bf2f(uint16_t b) { return __uint_as_float(static_cast<uint32_t>(b) << 16); }

// The node lattice and its padded image. Activations live on a padded lattice
// (stride sx >= nx + 1 along x, sy = ny + 1 rows a plane, guard cells before
// and after) whose cells outside the lattice hold zeros that nothing
// overwrites, so a tap is a constant offset from a cell with no test of the
// lattice's edge: the cell past the end of a row is the zero neighbour of both
// that row's last node and the next row's first. sx is a multiple of 4, so a
// group of 4 consecutive cells never straddles two rows.
struct Lat {
    int nx, ny, nz;
    int64_t V;
    int sx, sy;
    int64_t g0;   // cell of node (0, 0, 0)
    int64_t P;    // cells, guards included

    static Lat of(int nx, int ny, int nz) {
        Lat L{nx, ny, nz, (int64_t)nx * ny * nz, (nx + 4) / 4 * 4, ny + 1, 0, 0};
        // the lowest tap is one plane, one row and one cell back; a tile of row
        // pairs that runs past the last row reads up to two planes, three rows
        // and 28 cells past the last node
        const int64_t plane = (int64_t)L.sx * L.sy;
        L.g0 = (plane + L.sx + 1 + 15) / 16 * 16;
        L.P = L.g0 + plane * nz + 2 * plane + 4 * L.sx + 128;
        return L;
    }
    __device__ __forceinline__ int64_t cell(int x, int y, int z) const {
        return g0 + x + (int64_t)sx * (y + (int64_t)sy * z);
    }
    __device__ __forceinline__ int64_t cell(int64_t v) const {
        const int64_t q = v / nx;
        return cell(static_cast<int>(v % nx), static_cast<int>(q % ny), static_cast<int>(q / ny));
    }
    // offset of tap t ((dz, dy, dx) in {-1,0,1}^3, dx fastest)
    __device__ __forceinline__ int64_t tap(int t) const {
        return (t % 3 - 1) + (int64_t)sx * ((t / 3) % 3 - 1 + (int64_t)sy * (t / 9 - 1));
    }
};

// ---------------------------------------------------------------- forward / backward-data
// MODE 0: out bf16 [P][16] = relu(z + bias)
// MODE 1: out f32 [V]      = z[:, 0] + bias[0]
// MODE 2: out bf16 [P][16] = z * (mask[P][16] > 0)          (backward data; no bias)
//
// A wavefront owns 16 cells x 2 rows x 2 planes: the weights are the MFMA's A
// operand (rows = output channels) and stay in registers, the cells its B
// operand (columns), so a lane ends with 4 channels of one cell, one 8-byte
// store. An input row serves up to four outputs: 48 loads for 108 MFMAs, where
// a tile of 16 cells alone takes 27 for 27. Taps reach each output in ascending
// order (planes, rows, cells), one 16x16x16 MFMA each. At 97^3 a 16-channel
// layer takes 36 us and the input layer 22 us; with the edge tests, the weights
// in LDS and 2-byte stores they took 85 and 37 us. Load latency bounds it.
template <int CIN, int MODE>
__global__ __launch_bounds__(kThreads, 4) void k_conv(Lat L, const uint16_t* __restrict__ X,
                                                      const uint16_t* __restrict__ Wp, const float* __restrict__ bias,
                                                      const uint16_t* __restrict__ mask, void* __restrict__ out) {
    constexpr int NCH = CIN == 16 ? 27 : 7;
    const int lane = threadIdx.x % 64, g = lane / 16, n = lane % 16;
    s4 w[NCH];
#pragma unroll
    for (int m = 0; m < NCH; ++m) w[m] = *reinterpret_cast<const s4*>(Wp + (m * 16 + n) * 16 + 4 * g);
    f4 bs = {0.f, 0.f, 0.f, 0.f};
    if (MODE == 0)
#pragma unroll
        for (int j = 0; j < 4; ++j) bs[j] = bias[4 * g + j];
    if (MODE == 1) bs[0] = bias[0];
    const int64_t plane = (int64_t)L.sx * L.sy;
    int64_t toff[7];   // the 3-channel layer: group g takes tap 4m + g of product m (the last one has none)
    if (CIN == 4)
#pragma unroll
        for (int m = 0; m < 7; ++m) toff[m] = 4 * m + g < 27 ? L.tap(4 * m + g) * 4 : 0;
    const int ypairs = (L.ny + 1) / 2, chunks = (ypairs * L.sx + 15) / 16;
    const int64_t items = (int64_t)chunks * ((L.nz + 1) / 2);
    for (int64_t it = (int64_t)blockIdx.x * (kThreads / 64) + threadIdx.x / 64; it < items;
         it += (int64_t)gridDim.x * (kThreads / 64)) {
        const int z = 2 * static_cast<int>(it / chunks);
        const int e = static_cast<int>(it % chunks) * 16 + n;
        const int y = 2 * (e / L.sx), x = e % L.sx;
        const int64_t p = L.cell(x, y, z);
        f4 acc[2][2];
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[q / 2][q % 2] = f4{0.f, 0.f, 0.f, 0.f};
        if constexpr (CIN == 16) {
            const uint16_t* lp = X + p * 16 + 4 * g;
#pragma unroll
            for (int zz = 0; zz < 4; ++zz) {
                s4 v[4][3];
#pragma unroll
                for (int yy = 0; yy < 4; ++yy) {
                    const uint16_t* row = lp + ((zz - 1) * plane + (int64_t)(yy - 1) * L.sx) * 16;
#pragma unroll
                    for (int d = 0; d < 3; ++d) v[yy][d] = *reinterpret_cast<const s4*>(row + (d - 1) * 16);
                }
#pragma unroll
                for (int yy = 0; yy < 4; ++yy)
#pragma unroll
                    for (int d = 0; d < 3; ++d)
#pragma unroll
                        for (int oz = 0; oz < 2; ++oz)
#pragma unroll
                            for (int oy = 0; oy < 2; ++oy) {
                                const int tz = zz - oz, ty = yy - oy;   // dz + 1, dy + 1
                                if (tz < 0 || tz > 2 || ty < 0 || ty > 2) continue;
                                acc[oz][oy] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(w[tz * 9 + ty * 3 + d], v[yy][d],
                                                                                        acc[oz][oy], 0, 0, 0);
                            }
            }
        } else {
            s4 v[2][2][NCH];
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int m = 0; m < NCH; ++m)
                    v[q / 2][q % 2][m] =
                        *reinterpret_cast<const s4*>(X + (p + (q / 2) * plane + (q % 2) * L.sx) * 4 + toff[m]);
            if (4 * (NCH - 1) + g >= 27)   // no 28th tap: 0, not the cell itself (its weight is 0, but 0 inf is no 0)
#pragma unroll
                for (int q = 0; q < 4; ++q) v[q / 2][q % 2][NCH - 1] = s4{0, 0, 0, 0};
#pragma unroll
            for (int m = 0; m < NCH; ++m)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    acc[q / 2][q % 2] =
                        __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(w[m], v[q / 2][q % 2][m], acc[q / 2][q % 2], 0, 0, 0);
        }
        if (x >= L.nx) continue;   // a cell outside the lattice stays zero
#pragma unroll
        for (int oz = 0; oz < 2; ++oz)
#pragma unroll
            for (int oy = 0; oy < 2; ++oy) {
                if (y + oy >= L.ny || z + oz >= L.nz) continue;
                const int64_t po = p + oz * plane + oy * L.sx;
                const f4 val = acc[oz][oy];
                if (MODE == 1) {
                    if (g == 0)
                        static_cast<float*>(out)[x + (int64_t)L.nx * (y + oy + (int64_t)L.ny * (z + oz))] = val[0] + bs[0];
                    continue;
                }
                s4 r;
                if (MODE == 0) {
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const float t = val[j] + bs[j];
                        r[j] = static_cast<short>(f2bf(t > 0.f ? t : 0.f));
                    }
                } else {
                    const s4 on = *reinterpret_cast<const s4*>(mask + po * 16 + 4 * g);
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        r[j] = static_cast<short>(f2bf(bf2f(static_cast<uint16_t>(on[j])) > 0.f ? val[j] : 0.f));
                }
                *reinterpret_cast<s4*>(static_cast<uint16_t*>(out) + po * 16 + 4 * g) = r;
            }
    }
}

// ---------------------------------------------------------------- weight gradients
// partial[b][m*256 + co*16 + n] = sum over this block's lattice points of
// dZ[v][co] X[v + tap][ci], with (tap, ci) = (m, n) for CIN = 16 and
// (4m + n/4, n%4) for CIN = 4; partial[b][NCH*256 + co] = sum dZ[v][co].
// One resident set of blocks (two waves a SIMD: 108 accumulators), the four
// wavefronts' sums added in LDS, so that 512 partials leave the kernel and not
// one a wavefront.
template <int CIN>
__global__ __launch_bounds__(kThreads) void k_wgrad(Lat L, const uint16_t* __restrict__ dZ,
                                                    const uint16_t* __restrict__ X, float* __restrict__ partial) {
    constexpr int NCH = CIN == 16 ? 27 : 7;
    constexpr int STRIDE = NCH * 256 + 16;
    const int wave = threadIdx.x / 64, lane = threadIdx.x % 64;
    const int g = lane / 16, n = lane % 16;
    const int64_t wg = (int64_t)blockIdx.x * 4 + wave;
    const int64_t nw = (int64_t)gridDim.x * 4;
    const int64_t ntiles = ((int64_t)L.sx * L.sy * L.nz + 15) / 16;   // every cell: dZ is zero outside the lattice
    const int ci = CIN == 16 ? n : n % 4;
    f4 acc[NCH];
#pragma unroll
    for (int m = 0; m < NCH; ++m) acc[m] = f4{0.f, 0.f, 0.f, 0.f};
    float db = 0.f;
    for (int64_t tile = wg; tile < ntiles; tile += nw) {
        const int64_t p = L.g0 + tile * 16 + 4 * g;
        // a cell outside the lattice has dZ = 0, but its taps may reach an infinite
        // activation, and 0 inf is no 0: their values are masked (sx is a multiple
        // of 4, so the four cells share a row)
        const uint32_t q0 = static_cast<uint32_t>(tile * 16 + 4 * g), row = q0 / L.sx;
        const int in = row % L.sy < static_cast<uint32_t>(L.ny) && row < static_cast<uint32_t>(L.sy) * L.nz
                           ? L.nx - static_cast<int>(q0 % L.sx) : 0;   // of them inside, from the first
        s4 on;
#pragma unroll
        for (int j = 0; j < 4; ++j) on[j] = j < in ? -1 : 0;
        s4 a;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint16_t d = dZ[(p + j) * 16 + n];
            a[j] = static_cast<short>(d);
            db += bf2f(d);
        }
#pragma unroll
        for (int m = 0; m < NCH; ++m) {
            const int t = CIN == 16 ? m : 4 * m + n / 4;
            s4 b;
#pragma unroll
            for (int j = 0; j < 4; ++j) b[j] = static_cast<short>(X[(p + j + (t < 27 ? L.tap(t) : 0)) * CIN + ci]);
            b &= on;
            acc[m] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, acc[m], 0, 0, 0);
        }
    }
    db += __shfl_xor(db, 16);
    db += __shfl_xor(db, 32);
    __shared__ float sm[STRIDE];
    for (int q = 0; q < kThreads / 64; ++q) {   // wavefront by wavefront: a fixed order
        if (wave == q) {
#pragma unroll
            for (int m = 0; m < NCH; ++m)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    float* d = sm + m * 256 + (4 * g + j) * 16 + n;
                    *d = q == 0 ? acc[m][j] : *d + acc[m][j];
                }
            if (lane < 16) sm[NCH * 256 + lane] = q == 0 ? db : sm[NCH * 256 + lane] + db;
        }
        __syncthreads();
    }
    float* P = partial + (int64_t)blockIdx.x * STRIDE;
    for (int i = threadIdx.x; i < STRIDE; i += kThreads) P[i] = sm[i];
}

// The gradient of one layer = the sum over blocks of their partials, in two
// passes of fixed order. One thread per parameter walking 8192 partials in one
// 28-block launch had one load in flight per thread: 2539 us a layer at 97^3.
constexpr int kSegs = 16;

// part2[s][p] = sum of partial[w][p] over segment s of the blocks
__global__ __launch_bounds__(kThreads) void k_wgrad_sum(const float* __restrict__ partial, int64_t nw, int stride,
                                                        float* __restrict__ part2) {
    __shared__ float sm[kThreads / 64][64];
    const int lane = threadIdx.x % 64, row = threadIdx.x / 64;
    const int p = blockIdx.x * 64 + lane;
    const int64_t per = (nw + kSegs - 1) / kSegs;
    const int64_t w1 = min(nw, (blockIdx.y + 1) * per);
    float s = 0.f;
    if (p < stride) {
#pragma unroll 8
        for (int64_t w = blockIdx.y * per + row; w < w1; w += kThreads / 64) s += partial[w * stride + p];
    }
    sm[row][lane] = s;
    __syncthreads();
    if (row == 0 && p < stride) part2[(int64_t)blockIdx.y * stride + p] = (sm[0][lane] + sm[1][lane]) + (sm[2][lane] + sm[3][lane]);
}

// grad (canonical [co][ci][27] + [co]) = sum over the segments
template <int CIN>
__global__ void k_wgrad_reduce(const float* __restrict__ part2, int cin, int cout, float* __restrict__ grad) {
    constexpr int NCH = CIN == 16 ? 27 : 7;
    constexpr int STRIDE = NCH * 256 + 16;
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p >= STRIDE) return;
    float s = 0.f;
#pragma unroll
    for (int w = 0; w < kSegs; ++w) s += part2[w * STRIDE + p];
    if (p >= NCH * 256) {
        const int co = p - NCH * 256;
        if (co < cout) grad[cout * cin * 27 + co] = s;
        return;
    }
    const int m = p / 256, co = (p / 16) % 16, nn = p % 16;
    const int tap = CIN == 16 ? m : 4 * m + nn / 4;
    const int ci = CIN == 16 ? nn : nn % 4;
    if (co < cout && ci < cin && tap < 27) grad[(co * cin + ci) * 27 + tap] = s;
}

// BF16 weights for the MFMA A operand, [m][n = output channel][k]:
// forward (trans = 0): n = co, k = ci (CIN 16) or k = 4 tl + ci, tap = 4m + tl (CIN 4)
// backward data (trans = 1): the adjoint convolution, n = ci, k = co, tap mirrored
__global__ void k_pack(const float* __restrict__ w, int cin, int cout, int nch, int trans, uint16_t* __restrict__ Wp) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= nch * 256) return;
    const int m = i / 256, n = (i / 16) % 16, k = i % 16;
    float val = 0.f;
    if (!trans) {
        int tap, ci;
        if (nch == 27) {
            tap = m;
            ci = k;
        } else {
            tap = 4 * m + k / 4;
            ci = k % 4;
        }
        if (n < cout && ci < cin && tap < 27) val = w[(n * cin + ci) * 27 + tap];
    } else {
        // dX[v][ci] = sum_tap' sum_co dZ[v + tap'][co] w[co][ci][26 - tap']
        const int tap = m, co = k, ci = n;
        if (co < cout && ci < cin) val = w[(co * cin + ci) * 27 + (26 - tap)];
    }
    Wp[i] = f2bf(val);
}

// The discrete fluence can dip slightly below zero far from the sources (the P1
// mass matrix has positive off-diagonal entries), so logs of fluences are
// taken of max(phi, kPhiFloor); corrections are clamped to e^{+-kMaxCorr}.
constexpr double kPhiFloor = 1e-16;
constexpr float kMaxCorr = 8.f;

__device__ __forceinline__ void put_input(const Lat& L, int64_t v, float a, float b, float c, uint16_t* __restrict__ X) {
    const s4 r = {static_cast<short>(f2bf(a)), static_cast<short>(f2bf(b)), static_cast<short>(f2bf(c)), 0};
    *reinterpret_cast<s4*>(X + L.cell(v) * 4) = r;
}

// network input for illumination k: [P][4] bf16 = (log mu/mu0, log kappa/kappa0, log phi_hom, 0)
__global__ void k_inputs(Lat L, const double* __restrict__ kappa, const double* __restrict__ mu, double k0,
                         double m0, const double* __restrict__ phih, uint16_t* __restrict__ X) {
    int64_t v = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (v >= L.V) return;
    put_input(L, v, static_cast<float>(log(mu[v] / m0)), static_cast<float>(log(kappa[v] / k0)),
              static_cast<float>(log(fmax(phih[v], kPhiFloor))), X);
}

// raw input [3][V] f32 -> [P][4] bf16
__global__ void k_inputs_raw(Lat L, const float* __restrict__ in, uint16_t* __restrict__ X) {
    int64_t v = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (v >= L.V) return;
    put_input(L, v, in[v], in[L.V + v], in[2 * L.V + v], X);
}

// target = log phi - log phi_hom (f32)
__global__ void k_target(int64_t V, const double* __restrict__ phi, const double* __restrict__ phih,
                         float* __restrict__ t) {
    int64_t v = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (v >= V) return;
    const double d = log(fmax(phi[v], kPhiFloor)) - log(fmax(phih[v], kPhiFloor));
    t[v] = static_cast<float>(fmin(fmax(d, -(double)kMaxCorr), (double)kMaxCorr));
}

// phi0 = phi_hom exp(pred)
__global__ void k_fluence(int64_t V, const float* __restrict__ pred, const double* __restrict__ phih,
                          double* __restrict__ phi0) {
    int64_t v = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (v >= V) return;
    float p = pred[v];
    if (!(p == p)) p = 0.f;   // a non-finite prediction falls back to phi_hom
    p = fminf(fmaxf(p, -kMaxCorr), kMaxCorr);
    phi0[v] = phih[v] * exp(static_cast<double>(p));
}

// mean squared error: per-block partial sums; dZ4[v][0] = 2 (pred - t) / V
__global__ __launch_bounds__(kThreads) void k_loss(Lat L, const float* __restrict__ pred,
                                                   const float* __restrict__ t, uint16_t* __restrict__ dZ,
                                                   double* __restrict__ part) {
    __shared__ double sm[kThreads / 64];
    double acc = 0.0;
    const int64_t V = L.V;
    for (int64_t v = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; v < V; v += (int64_t)gridDim.x * blockDim.x) {
        const float d = pred[v] - t[v];
        acc += static_cast<double>(d) * d;
        uint4* row = reinterpret_cast<uint4*>(dZ + L.cell(v) * 16);
        row[0] = uint4{f2bf(2.f * d / static_cast<float>(V)), 0, 0, 0};
        row[1] = uint4{0, 0, 0, 0};
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) acc += __shfl_xor(acc, off);
    if ((threadIdx.x & 63) == 0) sm[threadIdx.x >> 6] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        double s = 0.0;
        for (int w = 0; w < kThreads / 64; ++w) s += sm[w];
        part[blockIdx.x] = s;
    }
}

__global__ void k_loss_final(const double* __restrict__ part, int nb, int64_t V, double* __restrict__ out) {
    // one wavefront: 65 us for 892 blocks at 97^3 while one thread added them, 5 us now
    double s = 0.0;
    for (int b = threadIdx.x; b < nb; b += 64) s += part[b];
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) s += __shfl_xor(s, off);
    if (threadIdx.x == 0) *out = s / static_cast<double>(V);
}

// Adam on the FP32 master parameters (Kingma and Ba's update with bias correction)
__global__ void k_adam(int n, float* __restrict__ w, const float* __restrict__ g, float* __restrict__ m1,
                       float* __restrict__ m2, float lr, float b1, float b2, float eps, float c1, float c2) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float gi = g[i];
    const float a = b1 * m1[i] + (1.f - b1) * gi;
    const float b = b2 * m2[i] + (1.f - b2) * gi * gi;
    m1[i] = a;
    m2[i] = b;
    w[i] -= lr * (a / c1) / (sqrtf(b / c2) + eps);
}

__global__ void k_zero_16(int64_t n, uint4* p) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = uint4{0, 0, 0, 0};
}

__global__ void k_zero_f(int n, float* p) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0.f;
}

// One resident set of blocks on 256 CUs, for both. A gradient's weight kernels
// hold 108 accumulators (two blocks a CU); with 256, 512, 768 and 1024 blocks the
// gradient takes 268, 248, 278, 278 us on 65^3 nodes and 1162, 960, 1039, 997 on
// 129^3 (a net of 17^3 nodes: 137, 150, 174, 182, its partials' sums being most of it).
constexpr int kWgradBlocks = 512;
// The convolutions keep their weights in registers (128: four blocks a CU) and
// walk the items. Inference with 512, 768, 1024, 1536 and 2048 blocks: 76, 70,
// 70, 76, 76 us on 65^3 nodes, 318, 270, 268, 277, 270 on 129^3.
constexpr int kConvBlocks = 1024;

int nch_of(int layer) { return layer == 0 ? 7 : 27; }

}  // namespace

// ---------------------------------------------------------------- host side
struct GuessNet {
    Lat L{};
    float* params = nullptr;   // [kParams] FP32 master
    float* grads = nullptr;
    float* m1 = nullptr;
    float* m2 = nullptr;
    uint16_t* Wf[kLayers] = {};  // forward A operands
    uint16_t* Wb[kLayers] = {};  // backward-data A operands
    // on the padded lattice, zero outside the node lattice
    uint16_t* X0 = nullptr;      // [P][4]
    uint16_t* Y[3] = {};         // hidden activations [P][16]
    uint16_t* dA = nullptr;      // [P][16]
    uint16_t* dB = nullptr;      // [P][16]
    float* pred = nullptr;       // [V]
    float* target = nullptr;     // [V]
    float* partial = nullptr;    // [kWgradBlocks][27*256+16]
    float* part2 = nullptr;      // [kSegs][27*256+16]
    double* lossp = nullptr;     // [blocks]
    double* lossv = nullptr;     // [1]
    int step = 0;
    bool have_params = false;    // zeroed at the first set-up, or the caller's
    bool ready = false;          // every array is there, for the sides of L
};

static qpat_status guess_pack(qpat_ctx* c) {
    GuessNet* G = c->guess;
    for (int l = 0; l < kLayers; ++l) {
        const float* w = G->params + param_offset(l);
        const int nch = nch_of(l);
        hipLaunchKernelGGL(k_pack, dim3((nch * 256 + 255) / 256), dim3(256), 0, c->stream, w, kCin[l], kCout[l], nch, 0,
                           G->Wf[l]);
        if (l > 0)
            hipLaunchKernelGGL(k_pack, dim3(27), dim3(256), 0, c->stream, w, kCin[l], kCout[l], 27, 1, G->Wb[l]);
    }
    QPAT_HIP(c, hipGetLastError());
    return QPAT_OK;
}

// forward pass; the last layer writes its single output channel, FP32 [V]
static qpat_status guess_forward(qpat_ctx* c, float* out) {
    GuessNet* G = c->guess;
    const dim3 g(kConvBlocks), b(kThreads);
    const float* bias[kLayers];
    for (int l = 0; l < kLayers; ++l) bias[l] = G->params + param_offset(l) + kCout[l] * kCin[l] * 27;
    hipLaunchKernelGGL((k_conv<4, 0>), g, b, 0, c->stream, G->L, G->X0, G->Wf[0], bias[0], nullptr, (void*)G->Y[0]);
    hipLaunchKernelGGL((k_conv<16, 0>), g, b, 0, c->stream, G->L, G->Y[0], G->Wf[1], bias[1], nullptr, (void*)G->Y[1]);
    hipLaunchKernelGGL((k_conv<16, 0>), g, b, 0, c->stream, G->L, G->Y[1], G->Wf[2], bias[2], nullptr, (void*)G->Y[2]);
    hipLaunchKernelGGL((k_conv<16, 1>), g, b, 0, c->stream, G->L, G->Y[2], G->Wf[3], bias[3], nullptr, (void*)out);
    QPAT_HIP(c, hipGetLastError());
    return QPAT_OK;
}

// loss and gradients of the current sample (input in X0, target in G->target)
static qpat_status guess_backward(qpat_ctx* c) {
    GuessNet* G = c->guess;
    const int64_t V = G->L.V;
    const dim3 g(kConvBlocks), gw(kWgradBlocks), b(kThreads);
    const int lb = grid_for(V, kThreads, 1024);
    QPAT_TRY(guess_forward(c, G->pred));
    hipLaunchKernelGGL(k_loss, dim3(lb), b, 0, c->stream, G->L, G->pred, G->target, G->dA, G->lossp);
    hipLaunchKernelGGL(k_loss_final, dim3(1), dim3(64), 0, c->stream, G->lossp, lb, V, G->lossv);
    const int64_t nw = kWgradBlocks;
    // dZ of layer l in cur; its input activation is Y[l-1] (X0 for l = 0)
    uint16_t* cur = G->dA;
    uint16_t* nxt = G->dB;
    for (int l = kLayers - 1; l >= 0; --l) {
        const uint16_t* Xin = l == 0 ? G->X0 : G->Y[l - 1];
        float* grad = G->grads + param_offset(l);
        if (l == 0) {
            hipLaunchKernelGGL(k_wgrad<4>, gw, b, 0, c->stream, G->L, cur, Xin, G->partial);
            hipLaunchKernelGGL(k_wgrad_sum, dim3((7 * 256 + 16 + 63) / 64, kSegs), b, 0, c->stream, G->partial, nw,
                               7 * 256 + 16, G->part2);
            hipLaunchKernelGGL(k_wgrad_reduce<4>, dim3((7 * 256 + 16 + 255) / 256), dim3(256), 0, c->stream, G->part2,
                               kCin[l], kCout[l], grad);
        } else {
            hipLaunchKernelGGL(k_wgrad<16>, gw, b, 0, c->stream, G->L, cur, Xin, G->partial);
            hipLaunchKernelGGL(k_wgrad_sum, dim3((27 * 256 + 16 + 63) / 64, kSegs), b, 0, c->stream, G->partial, nw,
                               27 * 256 + 16, G->part2);
            hipLaunchKernelGGL(k_wgrad_reduce<16>, dim3((27 * 256 + 16 + 255) / 256), dim3(256), 0, c->stream, G->part2,
                               kCin[l], kCout[l], grad);
            // dZ of layer l-1 = (adjoint convolution of dZ_l) masked by ReLU(Y[l-1]) > 0
            hipLaunchKernelGGL((k_conv<16, 2>), g, b, 0, c->stream, G->L, cur, G->Wb[l], nullptr, G->Y[l - 1],
                               (void*)nxt);
            uint16_t* t = cur;
            cur = nxt;
            nxt = t;
        }
    }
    QPAT_HIP(c, hipGetLastError());
    return QPAT_OK;
}

qpat_status guess_setup(qpat_ctx* c, int nx, int ny, int nz) {
    if ((int64_t)nx * ny * nz != c->N) return fail(c, QPAT_ERR_ARG, "guess_setup: nx*ny*nz must equal N");
    if (c->N * 16 * 2 >= (int64_t(1) << 31))   // 2 GB an activation
        return fail(c, QPAT_ERR_ARG, "guess_setup: lattice too large for the network (N = %lld)", (long long)c->N);
    if (!c->guess) c->guess = new GuessNet();
    GuessNet* G = c->guess;
    if (G->ready && G->L.nx == nx && G->L.ny == ny && G->L.nz == nz) return QPAT_OK;
    G->ready = false;   // until the last allocation has succeeded
    G->L = Lat::of(nx, ny, nz);
    const int64_t V = c->N, P = G->L.P;
    QPAT_TRY(dalloc_once(c, &G->params, kParams));
    QPAT_TRY(dalloc_once(c, &G->grads, kParams));
    QPAT_TRY(dalloc_once(c, &G->m1, kParams));
    QPAT_TRY(dalloc_once(c, &G->m2, kParams));
    for (int l = 0; l < kLayers; ++l) {
        QPAT_TRY(dalloc_once(c, &G->Wf[l], (size_t)nch_of(l) * 256));
        QPAT_TRY(dalloc_once(c, &G->Wb[l], (size_t)27 * 256));
    }
    QPAT_TRY(dalloc_once(c, &G->pred, V));
    QPAT_TRY(dalloc_once(c, &G->target, V));
    QPAT_TRY(dalloc_once(c, &G->partial, (size_t)kWgradBlocks * (27 * 256 + 16)));
    QPAT_TRY(dalloc_once(c, &G->part2, (size_t)kSegs * (27 * 256 + 16)));
    QPAT_TRY(dalloc_once(c, &G->lossp, 1024));
    QPAT_TRY(dalloc_once(c, &G->lossv, 1));
    // the padded lattice follows the sides; on other sides than before its arrays
    // are made anew (their padding must be zero), the parameters stay
    auto zeroed = [&](uint16_t** q, int64_t n) -> qpat_status {   // n: a multiple of 8
        QPAT_TRY(dfree(c, *q));
        QPAT_TRY(dalloc(c, q, n));
        hipLaunchKernelGGL(k_zero_16, dim3(grid_for(n / 8, kThreads, 4096)), dim3(kThreads), 0, c->stream, n / 8,
                           reinterpret_cast<uint4*>(*q));
        return QPAT_OK;
    };
    QPAT_TRY(zeroed(&G->X0, (P + 1) / 2 * 2 * 4));
    for (int l = 0; l < 3; ++l) QPAT_TRY(zeroed(&G->Y[l], P * 16));
    QPAT_TRY(zeroed(&G->dA, P * 16));
    QPAT_TRY(zeroed(&G->dB, P * 16));
    if (!G->have_params) {
        hipLaunchKernelGGL(k_zero_f, dim3((kParams + 255) / 256), dim3(256), 0, c->stream, kParams, G->params);
        QPAT_TRY(guess_pack(c));
        G->have_params = true;
    }
    QPAT_HIP(c, hipGetLastError());
    G->ready = true;
    return QPAT_OK;
}

bool guess_ready(const qpat_ctx* c) { return c->guess && c->guess->ready; }

qpat_status guess_set_params(qpat_ctx* c, const float* p) {
    GuessNet* G = c->guess;
    QPAT_HIP(c, hipMemcpyAsync(G->params, p, sizeof(float) * kParams, hipMemcpyDeviceToDevice, c->stream));
    hipLaunchKernelGGL(k_zero_f, dim3((kParams + 255) / 256), dim3(256), 0, c->stream, kParams, G->m1);
    hipLaunchKernelGGL(k_zero_f, dim3((kParams + 255) / 256), dim3(256), 0, c->stream, kParams, G->m2);
    G->step = 0;
    return guess_pack(c);
}

qpat_status guess_get_params(qpat_ctx* c, float* p) {
    QPAT_HIP(c, hipMemcpyAsync(p, c->guess->params, sizeof(float) * kParams, hipMemcpyDeviceToDevice, c->stream));
    return QPAT_OK;
}

qpat_status guess_eval_raw(qpat_ctx* c, const float* in, float* out) {
    GuessNet* G = c->guess;
    hipLaunchKernelGGL(k_inputs_raw, dim3(grid_for(G->L.V, kThreads, 1 << 30)), dim3(kThreads), 0, c->stream,
                       G->L, in, G->X0);
    return guess_forward(c, out);
}

qpat_status guess_grad_raw(qpat_ctx* c, const float* in, const float* target, float* grad, double* loss) {
    GuessNet* G = c->guess;
    hipLaunchKernelGGL(k_inputs_raw, dim3(grid_for(G->L.V, kThreads, 1 << 30)), dim3(kThreads), 0, c->stream,
                       G->L, in, G->X0);
    QPAT_HIP(c, hipMemcpyAsync(G->target, target, sizeof(float) * G->L.V, hipMemcpyDeviceToDevice, c->stream));
    QPAT_TRY(guess_backward(c));
    if (grad) QPAT_HIP(c, hipMemcpyAsync(grad, G->grads, sizeof(float) * kParams, hipMemcpyDeviceToDevice, c->stream));
    QPAT_HIP(c, hipMemcpyAsync(c->red_host, G->lossv, sizeof(double), hipMemcpyDeviceToHost, c->stream));
    QPAT_HIP(c, hipStreamSynchronize(c->stream));
    if (loss) *loss = c->red_host[0];
    return QPAT_OK;
}

static qpat_status adam_step(qpat_ctx* c, float lr) {
    GuessNet* G = c->guess;
    G->step += 1;
    const float b1 = 0.9f, b2 = 0.999f;
    const float c1 = 1.f - std::pow(b1, (float)G->step), c2 = 1.f - std::pow(b2, (float)G->step);
    hipLaunchKernelGGL(k_adam, dim3((kParams + 255) / 256), dim3(256), 0, c->stream, kParams, G->params, G->grads,
                       G->m1, G->m2, lr, b1, b2, 1e-8f, c1, c2);
    return guess_pack(c);
}

// one Adam step on the sample of illumination k: input from (kappa, mu, phi_hom_k), target log(phi_k / phi_hom_k)
qpat_status guess_train(qpat_ctx* c, const double* kappa, const double* mu, double k0, double m0,
                        const double* phih, const double* phi, float lr, double* loss) {
    GuessNet* G = c->guess;
    const dim3 gg(grid_for(G->L.V, kThreads, 1 << 30)), b(kThreads);
    hipLaunchKernelGGL(k_inputs, gg, b, 0, c->stream, G->L, kappa, mu, k0, m0, phih, G->X0);
    hipLaunchKernelGGL(k_target, gg, b, 0, c->stream, G->L.V, phi, phih, G->target);
    QPAT_TRY(guess_backward(c));
    QPAT_TRY(adam_step(c, lr));
    if (loss) {
        QPAT_HIP(c, hipMemcpyAsync(c->red_host, G->lossv, sizeof(double), hipMemcpyDeviceToHost, c->stream));
        QPAT_HIP(c, hipStreamSynchronize(c->stream));
        *loss = c->red_host[0];
    }
    return QPAT_OK;
}

qpat_status guess_train_raw(qpat_ctx* c, const float* in, const float* target, float lr, double* loss) {
    QPAT_TRY(guess_grad_raw(c, in, target, nullptr, loss));
    return adam_step(c, lr);
}

// phi0_k = phi_hom_k exp(net(log mu/mu0, log kappa/kappa0, log phi_hom_k)) for every illumination
qpat_status guess_fluence(qpat_ctx* c, const double* kappa, const double* mu, double k0, double m0,
                          const double* phih, double* phi0) {
    GuessNet* G = c->guess;
    const int64_t V = G->L.V;
    const dim3 gg(grid_for(V, kThreads, 1 << 30)), b(kThreads);
    for (int k = 0; k < c->n_ill; ++k) {
        hipLaunchKernelGGL(k_inputs, gg, b, 0, c->stream, G->L, kappa, mu, k0, m0, phih + k * V, G->X0);
        QPAT_TRY(guess_forward(c, G->pred));
        hipLaunchKernelGGL(k_fluence, gg, b, 0, c->stream, V, G->pred, phih + k * V, phi0 + k * V);
    }
    QPAT_HIP(c, hipGetLastError());
    return QPAT_OK;
}

void guess_destroy(qpat_ctx* c) {
    delete c->guess;
    c->guess = nullptr;
}

}  // namespace qpat
