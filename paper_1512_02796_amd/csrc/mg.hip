// Geometric multigrid preconditioner for the K and M_delta solves on lattice
// meshes.
//
// K (the forward and adjoint diffusion operator, Sec. 2 and the Appendix) and
// each block of M_delta (Sec. 4 eqs. (4.5), (4.8)) are SPD FEM matrices on the
// node lattice. Their solves are PCG preconditioned by one symmetric V-cycle:
//   * levels: the lattice and its vertex-centred coarsenings, n -> n/2 + 1 per
//     axis, down to the first coarse level of at most kMgDenseK nodes (or at
//     most kMgCoarse nodes per axis);
//   * prolongation P: trilinear interpolation (weights 1, 1/2 per axis),
//     restriction P^T;
//   * coarse operators by Galerkin products A_c = P^T A P, stored like the fine
//     stencil form (diagonal + upper offsets, node-major), 27-point;
//   * smoother: kMgNu weighted Jacobi sweeps before and after the coarse
//     correction, weight 8/(5 g) with g >= lambda_max(D^{-1} A) the Gershgorin
//     bound: the first-degree Chebyshev weight for the interval [g/4, g] that
//     the sweep has to damp; 19/(10 g) on the coarse levels (w lambda < 2
//     keeps the cycle SPD);
//   * coarsest level: the explicit inverse (dense).
// Vectors hold B right-hand sides interleaved ([sys][N][B]); every lane
// (system, right-hand side) has its own PCG scalars and stops on its own.
// With deflation (M_delta: the exact eigenpair (delta, 1) of each block) the
// solve runs on the complement of the constants as the Jacobi-PCG path does:
// b <- b - mean(b), z <- V(r) - mean(V(r)), and the mean of the solution is
// mean(b)/delta. The stopping rule is the same as Jacobi-PCG's:
// ||b - A x||_2 <= rtol ||b||_2 on the FP64 residual, confirmed on the true
// residual at the end. The PCG's iterate, residual, product and dot products and
// the set-up are FP64, and its direction but for mixed precision. The V-cycle
// keeps parts of its own work in FP32: M_delta's finest vectors, rows and
// transfer weights, and with 16 right-hand sides on the tiled levels of K the
// finest residual it restricts, its output z, level 1's vectors and the 27-point
// rows.
#include <cmath>
#include <cstring>
#include <functional>
#include <map>
#include <mutex>
#include <tuple>


#include "qpat_internal.h"

namespace qpat {

struct MgLevel {
    int32_t nx = 0, ny = 0, nz = 0;
    int64_t N = 0;
    int32_t m = 0;                 // stored upper offsets
    int32_t kind = 0;              // row kernel: 0 generic table, 1 Kuhn offsets, 2 27-point, 3 Kuhn upper rows
                                   // entry-major (Uf), 4 whole 27-point rows (Uf)
    const int4* tab = nullptr;     // [m]: dx, dy, dz, dx + nx (dy + ny dz)
    int4* tab_own = nullptr;
    double* U = nullptr;           // [nsys][N][m+1] (level 0: the context's stencil arrays)
    double* dinv = nullptr;        // [nsys][N] 1 / a_ii
    double* b = nullptr;           // [nsys][N][B] (level 0: the PCG residual)
    double* x = nullptr;           // [nsys][N][B]
    double* t = nullptr;           // ping-pong partner of x
    double* r = nullptr;           // residual before restriction
    double* W = nullptr;           // [nsys][8][N] operator-dependent prolongation weights to the next level (corner-major)
    float* Wc = nullptr;           // [nsys][WPack size] the nonzero ones of W in FP32, packed by corner: the V-cycle's
                                   // transfers read these (W holds the same rounded values for the Galerkin set-up:
                                   // one P throughout)
    double* Uf = nullptr;          // kind 3: [nsys][kUpRow][N] Kuhn diagonal + upper entries, entry-major;
                                   // kind 4: [nsys][27][N]
    float* Uf32 = nullptr;         // kind 5 / 6: the kind-3 / kind-4 rows in FP32 (M_delta's V-cycle)
    float* Uf27p = nullptr;        // K tiled levels >= 1: the 27-point rows in FP32 as [N][16] pairs (entry k, entry k + 16)
    int32_t vkind = -1;            // row kind of the V-cycle's kernels on this level (-1: kind)
};

struct MgScal {
    double rz, pq, alpha, beta, c, rr, bnorm2, mean, rr0;   // rr0: rr at the start of the solve
    int32_t active, done, iters, pad;
};

// Tiling of the finest level for one block size (LDS-tiled kernels)
constexpr int kMgMaxLevels = 12;   // levels with a tiled-kernel geometry (more levels run untiled)
struct TileGeo {
    bool ready = false, on = false;
    int32_t tiles_x = 0, tiles_y = 0, zc = 0, items = 0, blocks = 0;
    // the tiled restrictions, level l to l + 1 (coarse tiles, coarse z-chunk, blocks)
    struct Rst {
        bool on = false;
        int32_t tx = 0, ty = 0, zc = 0, items = 0, blocks = 0;
    };
    Rst rst[kMgMaxLevels];
    // the fused prolongation + last sweep (even z-chunks)
    int32_t ps_zc = 0, ps_items = 0, ps_blocks = 0;
    // the cost model's z-chunk lengths (tiles, prolongation + sweep) and whether the ones in
    // use were picked by timing them (autotune)
    int32_t zc_model = 0, ps_zc_model = 0;
    bool tuned = false;
    // the tiled 27-point kernels of the coarse levels (16 right-hand sides)
    struct Lv27 {
        bool on = false;
        int32_t tx = 0, ty = 0, zc = 0, items = 0, blocks = 0;
    };
    Lv27 t27[kMgMaxLevels];
};

struct MgState {
    int32_t nsys = 1;              // 1 (K) or 2 (the blocks of M_delta)
    bool opdep = false;            // operator-dependent prolongation (else trilinear)
    int32_t bmax = 1;              // right-hand sides the vectors are sized for
    bool current = false;          // built from the operator now assembled
    std::vector<MgLevel> lv;
    double* w = nullptr;           // [nsys][levels] Jacobi weights
    double* ainv = nullptr;        // [nsys][Nc][Nc]
    double* ainv_t = nullptr;      // the other buffer of its steps
    double* apiv = nullptr;        // [2][nsys][kGj][kGj] their inverted pivot blocks
    int* bad = nullptr;            // [nsys + 1] set-up checks: a pivot of system s, a diagonal, not positive
    double *pr = nullptr, *pa = nullptr, *pb = nullptr, *pq = nullptr;  // PCG r, p (two), q: [nsys][N][bmax]
    double* pr2 = nullptr;         // the other residual buffer of the fused update (odd iterations write r here)
    double* pring = nullptr;       // [kRing][N][bmax] directions of the tiled iterations (FP32 or FP64 elements)
    double* ahist = nullptr;       // [kRing][lanes] their alphas (0: the lane did not iterate)
    int32_t* pslot = nullptr;      // iterations of the current run so far (the ring slot of the next one)
    double* parts = nullptr;       // [lanes][4][kMgBlocks]
    uint64_t* gmax = nullptr;      // [nsys][levels] Gershgorin bounds (bit patterns)
    MgScal* sc = nullptr;          // [lanes], lane = sys B + k
    MgScal* sc_host = nullptr;
    // region coarse space (M_delta): z += Z E^{-1} Z^T r, E = Z^T A Z
    int32_t kreg = 0;              // regions of the system with most (0: off)
    int32_t nreg[2] = {0, 0};
    int32_t* reg = nullptr;        // [nsys][N] region of each node, -1: none
    double* einv = nullptr;        // [nsys][kRegMax][kRegMax]
    double* rsize = nullptr;       // [nsys][kRegMax] nodes per region
    double* rparts = nullptr;      // [nsys][kRegMax][kMgBlocks] partial sums of Z^T r
    double* ry = nullptr;          // [nsys][kRegMax] y = E^{-1} Z^T r
    double* rcorr = nullptr;       // [nsys][2] r.(Z y), mean(Z y) (0 without deflation)
    std::map<int, TileGeo> tiles;  // by block size
    std::vector<hipEvent_t> ev;    // per-launch timing (profiling)
    std::map<std::string, hipGraphExec_t> graphs;
    hipStream_t cap = nullptr;
};

namespace {

constexpr int kMgCoarse = 5;      // coarsest lattice: at most this many nodes per axis, or
constexpr int64_t kMgDenseK = 1000;   // the first coarse level of at most this many nodes
constexpr int kMgNu = 1;          // Jacobi sweeps before and after the coarse correction
constexpr int kMgBlocks = 2048;   // most blocks of a kernel that writes partial sums (8 per CU)
constexpr int kMgGrid = 512;      // blocks of the vector kernels of several right-hand sides
constexpr int kMgT = 256;
constexpr int kMgLanes = 32;      // systems x right-hand sides
constexpr int kMgChunk0 = 4;      // PCG iterations before the first host check of a run
// The tiled K iterations keep their last kRing directions and alphas instead of
// updating x each iteration; x is formed from them before it is read (the
// true residual) or when the ring is full.
constexpr int kRing = 16;
// Region coarse space of M_delta: regions are the connected components of the
// graph of strong couplings |a_ij| > kRegTheta sqrt(a_ii a_jj); the kRegMax
// largest with at least kRegMin nodes get an indicator vector.
constexpr int kRegMax = 16;
constexpr int kRegMin = 64;
constexpr double kRegTheta = 1e-2;
constexpr int kRegList = 4096;    // candidate regions collected per system

__device__ __forceinline__ void coords(int32_t i, int nx, int ny, int& ix, int& iy, int& iz) {
    ix = i % nx;
    const int32_t q = i / nx;
    iy = q % ny;
    iz = q / ny;
}

// The rows with compile-time offsets: KIND 1 the Kuhn split (7 upper offsets,
// the fine level of a Kuhn mesh), KIND 2 the full 27-point stencil (13 upper
// offsets in code order, the Galerkin levels); KIND 0 the generic table.
constexpr int kKx[7] = {1, 0, 1, 0, 1, 0, 1};
constexpr int kKy[7] = {0, 1, 1, 0, 0, 1, 1};
constexpr int kKz[7] = {0, 0, 0, 1, 1, 1, 1};

// The stencil and V-cycle kernels give each thread V = 2 adjacent right-hand
// sides of one node (16-byte loads and stores; the row of the operator is read
// once for both); BV = B / V threads share a node.
typedef double d2v __attribute__((ext_vector_type(2)));
template <int B>
struct Pk {
    static constexpr int V = B >= 2 ? 2 : 1;
    static constexpr int BV = B / V;
};
template <int V>
struct VecT {
    using T = double;
};
template <>
struct VecT<2> {
    using T = d2v;
};
template <int B>
using TB = typename VecT<Pk<B>::V>::T;

template <typename T>
__device__ __forceinline__ T vld(const double* p) {
    return *reinterpret_cast<const T*>(p);
}
template <typename T>
__device__ __forceinline__ void vst(double* p, T v) {
    *reinterpret_cast<T*>(p) = v;
}
// the same from / to FP32 storage (a coarse level's vectors kept in FP32)
template <typename T>
__device__ __forceinline__ T vldf(const float* p) {
    if constexpr (sizeof(T) == 8) {
        return static_cast<double>(*p);
    } else {
        typedef float f2v __attribute__((ext_vector_type(2)));
        const f2v t = *reinterpret_cast<const f2v*>(p);
        return T{static_cast<double>(t.x), static_cast<double>(t.y)};
    }
}
template <typename T>
__device__ __forceinline__ void vstf(float* p, T v) {
    if constexpr (sizeof(T) == 8) {
        *p = static_cast<float>(v);
    } else {
        typedef float f2v __attribute__((ext_vector_type(2)));
        *reinterpret_cast<f2v*>(p) = f2v{static_cast<float>(v.x), static_cast<float>(v.y)};
    }
}
// vectors kept in FP64 or in FP32, by the pointer's type
template <typename T>
__device__ __forceinline__ T vldx(const double* p) {
    return vld<T>(p);
}
template <typename T>
__device__ __forceinline__ T vldx(const float* p) {
    return vldf<T>(p);
}
template <typename T>
__device__ __forceinline__ void vstx(double* p, T v) {
    vst<T>(p, v);
}
template <typename T>
__device__ __forceinline__ void vstx(float* p, T v) {
    vstf<T>(p, v);
}
// v as a vector of element type VT holds it (FP32: rounded)
template <typename VT>
__device__ __forceinline__ double held_as(double v) {
    return static_cast<double>(static_cast<VT>(v));
}
__device__ __forceinline__ double comp(double v, int) { return v; }
__device__ __forceinline__ double comp(d2v v, int c) { return c ? v.y : v.x; }

// Node order of the stencil kernels. The blocks of XCD x (block b runs on XCD
// b mod 8) take the y-strip [x ny / 8, (x + 1) ny / 8) of every plane (z-slabs
// when ny < 8) and sweep it plane by plane, x fastest. The strip's planes
// around the sweep (about 0.3 MB per plane of a 129^2 lattice with 16
// right-hand sides) then stay in that XCD's 4 MB L2 while the up to 27
// neighbours of every node are read, so each vector comes from HBM about
// once. Calls f(ix, iy, iz, node, thread-in-node). The thread-in-node is
// threadIdx.x mod BV for every element of a thread.
template <int BV, typename F>
__device__ __forceinline__ void walk(int32_t nx, int32_t ny, int32_t nz, F&& f) {
    const int32_t xcd = blockIdx.x & 7;
    int32_t y0 = 0, ys = ny, z0 = 0, zs = nz;
    if (ny >= 8) {
        y0 = xcd * ny / 8;
        ys = (xcd + 1) * ny / 8 - y0;
    } else {
        z0 = xcd * nz / 8;
        zs = (xcd + 1) * nz / 8 - z0;
    }
    const int32_t total = nx * ys * zs * BV;
    const int32_t step = (gridDim.x >> 3) * kMgT;
    for (int32_t e = (blockIdx.x >> 3) * kMgT + threadIdx.x; e < total; e += step) {
        const int32_t v = e % BV, n = e / BV;
        const int32_t ix = n % nx, q = n / nx;
        const int32_t iy = y0 + q % ys, iz = z0 + q / ys;
        f(ix, iy, iz, ix + nx * (iy + ny * iz), v);
    }
}

struct LvArgs {
    const double* U;
    const int4* tab;
    int32_t m, nx, ny, nz;
    int64_t N;
    int32_t kind;         // row kernel: 0 generic table, 1 Kuhn offsets, 2 full 27-point, 3 Kuhn upper rows
                          // entry-major, 4 27-point whole rows entry-major (5, 6: 3, 4 in FP32)
    const double* Uf;     // kind 3: [nsys][kUpRow][N]; kind 4: [nsys][27][N]
    const float* Uf32;    // kind 5 / 6: the same in FP32
};

// Kuhn rows for the one-right-hand-side kernels: the diagonal and the 7 upper
// entries, entry-major ([kUpRow][N] per system), so that a wavefront's loads of
// one entry for consecutive nodes are contiguous, the lower entries included
// (each is a partner row's upper entry at a shifted index)
constexpr int kUpRow = 8;

// first stored row of system sys in the form the row kernel KIND reads
template <int KIND>
__device__ __forceinline__ const double* rows_of(const LvArgs& L, int sys) {
    if constexpr (KIND == 3) return L.Uf + (int64_t)sys * L.N * kUpRow;
    if constexpr (KIND == 4) return L.Uf + (int64_t)sys * L.N * 27;
    if constexpr (KIND == 6) return reinterpret_cast<const double*>(L.Uf32 + (int64_t)sys * L.N * 27);
    if constexpr (KIND == 5) return reinterpret_cast<const double*>(L.Uf32 + (int64_t)sys * L.N * kUpRow);
    return L.U + (int64_t)sys * L.N * (L.m + 1);
}

// the thread's V right-hand sides of a node, from memory: x points at its
// first right-hand side of node 0 ([N][B] interleaved)
template <int B, typename XT>
struct VecAt {
    const XT* x;
    __device__ __forceinline__ TB<B> operator()(int32_t i) const { return vldx<TB<B>>(x + i * B); }
};

// which neighbours of a node are on the lattice: six tests a node, whose lane
// masks the (compile-time) offsets combine on the scalar unit
struct Edges {
    bool xp, xm, yp, ym, zp, zm;
    __device__ __forceinline__ Edges(int32_t nx, int32_t ny, int32_t nz, int32_t ix, int32_t iy, int32_t iz)
        : xp(ix + 1 < nx), xm(ix > 0), yp(iy + 1 < ny), ym(iy > 0), zp(iz + 1 < nz), zm(iz > 0) {}
    __device__ __forceinline__ bool has(int dx, int dy, int dz) const {
        return (dx == 0 || (dx > 0 ? xp : xm)) & (dy == 0 || (dy > 0 ? yp : ym)) & (dz == 0 || (dz > 0 ? zp : zm));
    }
};

// (A x)_i for the thread's V right-hand sides; x(j): its values at node j
// (VecAt, or formed on the fly: DirAt). A row's loads, from clamped indices,
// are all issued before its sums: a scheduling barrier keeps them together
// (left to itself the compiler takes them in five or six round trips: the
// last sweep on 33^3 nodes 19 us instead of 7 with 4 right-hand sides, 18
// instead of 5 in FP32 with one).
template <int KIND, int B, typename X>
__device__ __forceinline__ TB<B> apply(const LvArgs& L, const double* __restrict__ U, const X& x, int32_t ix,
                                       int32_t iy, int32_t iz, int32_t i) {
    using T = TB<B>;
    if constexpr (KIND == 0) {
        const int32_t M1 = L.m + 1;
        T s = U[i * M1] * x(i);
        for (int j = 0; j < L.m; ++j) {
            const int4 t = L.tab[j];
            if (ix + t.x >= 0 && ix + t.x < L.nx && iy + t.y >= 0 && iy + t.y < L.ny && iz + t.z < L.nz)
                s += U[i * M1 + j + 1] * x(i + t.w);
            if (ix - t.x >= 0 && ix - t.x < L.nx && iy - t.y >= 0 && iy - t.y < L.ny && iz - t.z >= 0)
                s += U[(i - t.w) * M1 + j + 1] * x(i - t.w);
        }
        return s;
    } else if constexpr (KIND == 4 || KIND == 6) {
        // 27-point whole rows, entry-major ([27][N]; 4: FP64, 6: FP32)
        using W = std::conditional_t<KIND == 6, float, double>;
        const W* Uw = reinterpret_cast<const W*>(U);
        const Edges in(L.nx, L.ny, L.nz, ix, iy, iz);
        T s = static_cast<double>(Uw[i]) * x(i), xu[13], xl[13];
        W cu[13], cl[13];
#pragma unroll
        for (int j = 0; j < 13; ++j) {
            const int code = 14 + j;
            const int dx = code % 3 - 1, dy = (code / 3) % 3 - 1, dz = code / 9 - 1;
            const int32_t lin = dx + L.nx * (dy + L.ny * dz);
            xu[j] = x(in.has(dx, dy, dz) ? i + lin : i);
            xl[j] = x(in.has(-dx, -dy, -dz) ? i - lin : i);
            cu[j] = Uw[(1 + j) * L.N + i];
            cl[j] = Uw[(14 + j) * L.N + i];
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < 13; ++j) {
            const int code = 14 + j;
            const int dx = code % 3 - 1, dy = (code / 3) % 3 - 1, dz = code / 9 - 1;
            s = in.has(dx, dy, dz) ? s + static_cast<double>(cu[j]) * xu[j] : s;
            s = in.has(-dx, -dy, -dz) ? s + static_cast<double>(cl[j]) * xl[j] : s;
        }
        return s;
    } else if constexpr (KIND == 3 || KIND == 5) {
        // Kuhn rows' diagonal and upper entries, entry-major (3: FP64, 5: FP32).
        // The lower entry of offset j of row i is the upper entry j of row
        // i - u_j, read at the shifted index of the same entry array: the
        // partner row's entries were read moments before in the sweep order,
        // so the shifted reads come from L2 and each row crosses HBM once.
        using W = std::conditional_t<KIND == 5, float, double>;
        const W* Uw = reinterpret_cast<const W*>(U);
        double u[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) u[k] = static_cast<double>(Uw[k * L.N + i]);
        const Edges in(L.nx, L.ny, L.nz, ix, iy, iz);
        T s = u[0] * x(i), xu[7], xl[7];
        double cl[7];
#pragma unroll
        for (int j = 0; j < 7; ++j) {
            const int dx = kKx[j], dy = kKy[j], dz = kKz[j];
            const int32_t lin = dx + L.nx * (dy + L.ny * dz);
            const bool up = in.has(dx, dy, dz);
            const bool lo = in.has(-dx, -dy, -dz);
            const int32_t il = lo ? i - lin : i;
            xu[j] = x(up ? i + lin : i);
            xl[j] = x(il);
            cl[j] = static_cast<double>(Uw[(1 + j) * L.N + il]);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < 7; ++j) {
            s = in.has(kKx[j], kKy[j], kKz[j]) ? s + u[1 + j] * xu[j] : s;
            s = in.has(-kKx[j], -kKy[j], -kKz[j]) ? s + cl[j] * xl[j] : s;
        }
        return s;
    } else {
        constexpr int MM = KIND == 1 ? 7 : 13;
        constexpr int M1 = MM + 1;   // even: the row is M1 / 2 16-byte loads
        double u[M1];
        const d2v* Ur = reinterpret_cast<const d2v*>(U + i * M1);
#pragma unroll
        for (int k = 0; k < M1 / 2; ++k) {
            const d2v t = Ur[k];
            u[2 * k] = t.x;
            u[2 * k + 1] = t.y;
        }
        const Edges in(L.nx, L.ny, L.nz, ix, iy, iz);
        T s = u[0] * x(i), xu[MM], xl[MM];
        double cl[MM];
#pragma unroll
        for (int j = 0; j < MM; ++j) {
            const int code = 14 + j;
            const int dx = KIND == 1 ? kKx[j] : code % 3 - 1;
            const int dy = KIND == 1 ? kKy[j] : (code / 3) % 3 - 1;
            const int dz = KIND == 1 ? kKz[j] : code / 9 - 1;
            const int32_t lin = dx + L.nx * (dy + L.ny * dz);
            const bool up = in.has(dx, dy, dz);
            const bool lo = in.has(-dx, -dy, -dz);
            const int32_t il = lo ? i - lin : i;
            xu[j] = x(up ? i + lin : i);
            xl[j] = x(il);
            cl[j] = U[il * M1 + j + 1];
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < MM; ++j) {
            const int code = 14 + j;
            const int dx = KIND == 1 ? kKx[j] : code % 3 - 1;
            const int dy = KIND == 1 ? kKy[j] : (code / 3) % 3 - 1;
            const int dz = KIND == 1 ? kKz[j] : code / 9 - 1;
            s = in.has(dx, dy, dz) ? s + u[j + 1] * xu[j] : s;
            s = in.has(-dx, -dy, -dz) ? s + cl[j] * xl[j] : s;
        }
        return s;
    }
}

// Compensated accumulation of s - a x: the product's rounding error comes
// from a fused multiply-add and the sum's from a two-sum, so that s + c holds
// b - sum a_j x_j to a few ulps of the result instead of ulps of
// sum |a_j x_j| (the true residual near the attainable accuracy of PCG).
struct CompSum {
    double s, c;
    __device__ __forceinline__ explicit CompSum(double b) : s(b), c(0.0) {}
    __device__ __forceinline__ void sub(double a, double x) {
        const double p = a * x;
        const double e = fma(a, x, -p);   // a x = p + e exactly
        const double t = s - p;
        const double bp = t - s;
        const double err = (s - (t - bp)) + (-p - bp);   // s - p = t + err exactly
        s = t;
        c += err - e;
    }
    __device__ __forceinline__ void add(double b) {
        const double t = s + b;
        const double bp = t - s;
        c += (s - (t - bp)) + (b - bp);   // s + b = t + that exactly
        s = t;
    }
    __device__ __forceinline__ double value() const { return s + c; }
};

// b_i - (A x)_i of one right-hand side (x: its entry of node 0, stride B),
// compensated; any stencil form (the offset table)
template <int B>
__device__ double resid_comp(const LvArgs& L, const double* __restrict__ U, const double* __restrict__ x, double bi,
                             int32_t ix, int32_t iy, int32_t iz, int32_t i) {
    const int32_t M1 = L.m + 1;
    CompSum r(bi);
    r.sub(U[i * M1], x[i * B]);
    for (int j = 0; j < L.m; ++j) {
        const int4 t = L.tab[j];
        if (ix + t.x >= 0 && ix + t.x < L.nx && iy + t.y >= 0 && iy + t.y < L.ny && iz + t.z < L.nz)
            r.sub(U[i * M1 + j + 1], x[(i + t.w) * B]);
        if (ix - t.x >= 0 && ix - t.x < L.nx && iy - t.y >= 0 && iy - t.y < L.ny && iz - t.z >= 0)
            r.sub(U[(i - t.w) * M1 + j + 1], x[(i - t.w) * B]);
    }
    return r.value();
}

// The same for a stencil form of 7 offsets (the Kuhn lattice), all loads in
// flight before the sums: indices clamped to the node itself and the terms of
// neighbours off the lattice replaced by 0 * 0, which the compensated sum
// takes exactly (so the value is bitwise that of resid_comp).
template <int B>
__device__ double resid_comp7(const LvArgs& L, const double* __restrict__ U, const double* __restrict__ x, double bi,
                              int32_t ix, int32_t iy, int32_t iz, int32_t i) {
    constexpr int32_t M1 = 8;
    double cu[7], xu[7], cl[7], xl[7];
    const double c0 = U[i * M1], x0 = x[i * B];
#pragma unroll
    for (int j = 0; j < 7; ++j) {
        const int4 t = L.tab[j];
        const bool up = ix + t.x >= 0 && ix + t.x < L.nx && iy + t.y >= 0 && iy + t.y < L.ny && iz + t.z < L.nz;
        const bool lo = ix - t.x >= 0 && ix - t.x < L.nx && iy - t.y >= 0 && iy - t.y < L.ny && iz - t.z >= 0;
        const int32_t iu = up ? i + t.w : i, il = lo ? i - t.w : i;
        const double a = U[i * M1 + j + 1], xa = x[iu * B], c = U[il * M1 + j + 1], xc = x[il * B];
        cu[j] = up ? a : 0.0;
        xu[j] = up ? xa : 0.0;
        cl[j] = lo ? c : 0.0;
        xl[j] = lo ? xc : 0.0;
    }
    CompSum r(bi);
    r.sub(c0, x0);
#pragma unroll
    for (int j = 0; j < 7; ++j) {
        r.sub(cu[j], xu[j]);
        r.sub(cl[j], xl[j]);
    }
    return r.value();
}

// plain grid-stride loop over n elements (one right-hand side each; the lane
// of a thread is threadIdx.x mod B)
#define QPAT_MG_ELEMS(e, n) \
    for (int64_t e = blockIdx.x * (int64_t)kMgT + threadIdx.x; e < (n); e += (int64_t)gridDim.x * kMgT)

// Sum over the threads with equal threadIdx.x mod G; the result is valid in
// threads threadIdx.x < G (group threadIdx.x).
template <int G>
__device__ __forceinline__ double group_sum(double v, double* sm) {
#pragma unroll
    for (int off = 32; off >= G; off >>= 1) v += __shfl_xor(v, off);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane < G) sm[wave * G + lane] = v;
    __syncthreads();
    double t = 0.0;
    if (threadIdx.x < G)
        for (int w = 0; w < kMgT / 64; ++w) t += sm[w * G + threadIdx.x];
    __syncthreads();
    return t;
}

// any of the V right-hand sides of thread-in-node v of system sys still iterating
template <int B>
__device__ __forceinline__ bool pair_active(const MgScal* sc, int sys, int v) {
    bool on = false;
#pragma unroll
    for (int c = 0; c < Pk<B>::V; ++c) on = on || sc[sys * B + v * Pk<B>::V + c].active;
    return on;
}

// partial sums of the block: parts[lane][slot][block]
// a block's partial sum; the reduction that follows is told how many blocks wrote
__device__ __forceinline__ void put(double* parts, int lane, int slot, double val) {
    parts[(lane * 4 + slot) * kMgBlocks + blockIdx.x] = val;
}

// per-right-hand-side block sums of NS V-wide accumulators, written as the
// partials of their slots: the shuffles of all of them interleave and they
// share one barrier (one after the other they were 3 us of a small lattice's
// last sweep). sm: kSumLds doubles.
constexpr int kSumLds = (kMgT / 64) * 16 * 3;
template <int B, int... SLOT>
__device__ __forceinline__ void put_sums(double* parts, int sys, const TB<B> (&acc)[sizeof...(SLOT)], double* sm) {
    constexpr int V = Pk<B>::V, BV = Pk<B>::BV, NS = sizeof...(SLOT);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    double t[NS][V];
#pragma unroll
    for (int n = 0; n < NS; ++n)
#pragma unroll
        for (int c = 0; c < V; ++c) t[n][c] = comp(acc[n], c);
#pragma unroll
    for (int off = 32; off >= BV; off >>= 1)
#pragma unroll
        for (int n = 0; n < NS; ++n)
#pragma unroll
            for (int c = 0; c < V; ++c) t[n][c] += __shfl_xor(t[n][c], off);
    __syncthreads();   // sm's last use
    if (lane < BV)
#pragma unroll
        for (int n = 0; n < NS; ++n)
#pragma unroll
            for (int c = 0; c < V; ++c) sm[(wave * NS + n) * B + lane * V + c] = t[n][c];
    __syncthreads();
    if (threadIdx.x < NS * B) {
        double v = 0.0;
#pragma unroll
        for (int w = 0; w < kMgT / 64; ++w) v += sm[w * NS * B + threadIdx.x];
        int n = threadIdx.x / B, at = 0;
        ((at = n-- == 0 ? SLOT : at), ...);
        put(parts, sys * B + threadIdx.x % B, at, v);
    }
}

// Kuhn rows from the stencil form (zero where the partner is off the lattice),
// the row kind 3: the diagonal and upper entries entry-major [kUpRow][N]
__global__ __launch_bounds__(kMgT) void k_mg_fullrows(LvArgs L, double* __restrict__ Uf) {
    const int sys = blockIdx.y;
    constexpr int M1 = 8;
    const double* U = L.U + (int64_t)sys * L.N * M1;
    double* F = Uf + (int64_t)sys * L.N * kUpRow;
    for (int64_t i = blockIdx.x * (int64_t)kMgT + threadIdx.x; i < L.N; i += (int64_t)gridDim.x * kMgT) {
        int ix, iy, iz;
        coords(static_cast<int32_t>(i), L.nx, L.ny, ix, iy, iz);
        F[i] = U[i * M1];
#pragma unroll
        for (int j = 0; j < 7; ++j) {
            const bool up = ix + kKx[j] < L.nx && iy + kKy[j] < L.ny && iz + kKz[j] < L.nz;
            F[(1 + j) * L.N + i] = up ? U[i * M1 + 1 + j] : 0.0;
        }
    }
}

__global__ __launch_bounds__(kMgT) void k_to_f32(const double* __restrict__ a, float* __restrict__ b, int64_t n) {
    for (int64_t i = blockIdx.x * (int64_t)kMgT + threadIdx.x; i < n; i += (int64_t)gridDim.x * kMgT)
        b[i] = static_cast<float>(a[i]);
}

// 1 / a_ii and the Gershgorin bound max_i sum_j |a_ij| / a_ii
// (M: room for the stored upper offsets, at least L.m; a row's loads go out
// together: the five levels of 97^3 136 -> 75 us)
template <int M>
__global__ __launch_bounds__(kMgT) void k_mg_diag(LvArgs L, double* __restrict__ dinv, uint64_t* __restrict__ gmax,
                                                  int nlev, int lev) {
    __shared__ double sm[kMgT / 64];
    const int sys = blockIdx.y;
    const int M1 = L.m + 1;
    const double* U = L.U + (int64_t)sys * L.N * M1;
    double g = 0.0;
    for (int64_t i = blockIdx.x * (int64_t)kMgT + threadIdx.x; i < L.N; i += (int64_t)gridDim.x * kMgT) {
        const double d = U[i * M1];
        dinv[sys * L.N + i] = 1.0 / d;
        int ix, iy, iz;
        coords(static_cast<int32_t>(i), L.nx, L.ny, ix, iy, iz);
        double up[M], lo[M];
#pragma unroll
        for (int j = 0; j < M; ++j) {
            const int4 t = L.tab[j < L.m ? j : 0];
            const bool u = j < L.m && ix + t.x >= 0 && ix + t.x < L.nx && iy + t.y >= 0 && iy + t.y < L.ny && iz + t.z < L.nz;
            const bool l = j < L.m && ix - t.x >= 0 && ix - t.x < L.nx && iy - t.y >= 0 && iy - t.y < L.ny && iz - t.z >= 0;
            const double a = U[i * M1 + (u ? j + 1 : 0)], b = U[(l ? i - t.w : i) * M1 + (l ? j + 1 : 0)];
            up[j] = u ? a : 0.0;
            lo[j] = l ? b : 0.0;
        }
        __builtin_amdgcn_sched_barrier(0);
        double row = fabs(d);
#pragma unroll
        for (int j = 0; j < M; ++j) {
            row += fabs(up[j]);
            row += fabs(lo[j]);
        }
        g = fmax(g, row / d);
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) g = fmax(g, __shfl_xor(g, off));
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0) sm[wave] = g;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int w = 0; w < kMgT / 64; ++w) t = fmax(t, sm[w]);
        // positive doubles order like their bit patterns
        atomicMax(reinterpret_cast<unsigned long long*>(gmax + sys * nlev + lev),
                  static_cast<unsigned long long>(__double_as_longlong(t)));
    }
}

// Prolongation weight of fine node i (coords fx, fy, fz) towards coarse node
// J0(i) + corner c, J0(i) = (fx/2, fy/2, fz/2), c = cz 4 + cy 2 + cx. W: the
// operator-dependent weights of the system, corner-major ([8][N]: the loads of
// one corner for consecutive nodes are contiguous), or null for trilinear
// interpolation (1 on an even axis, 1/2 to both sides on an odd one).
__device__ __forceinline__ double pweight(const double* __restrict__ W, int64_t N, int64_t i, int fx, int fy, int fz,
                                          int c) {
    if (W) return W[c * N + i];
    const int bx = c & 1, by = (c >> 1) & 1, bz = c >> 2;
    const double wx = (fx & 1) ? 0.5 : (bx ? 0.0 : 1.0);
    const double wy = (fy & 1) ? 0.5 : (by ? 0.0 : 1.0);
    const double wz = (fz & 1) ? 0.5 : (bz ? 0.0 : 1.0);
    return wx * wy * wz;
}

// Packed prolongation weights. Fine node (ix, iy, iz) takes its value from the
// corners J0 + (a, b, c) of the coarse cell J0 = (ix/2, iy/2, iz/2). Along an
// axis where the node's coordinate is even it lies on a coarse plane, so a
// corner one step up that axis has weight 0 (trilinear and operator-dependent
// alike: the collapsed stencil has no extent along an even axis). Corner
// cn = a + 2 b + 4 c is therefore kept only on the sub-lattice of nodes that are
// odd along every axis of its set bits, indexed (a ? ix/2 : ix, b ? iy/2 : iy,
// c ? iz/2 : iz); the eight sub-lattices follow one another in corner order,
// 27/8 values per node instead of 8.
struct WPack {
    int32_t nx, ny, nz;
    __host__ __device__ __forceinline__ int64_t size() const {
        return (int64_t)(nx + (nx >> 1)) * (ny + (ny >> 1)) * (nz + (nz >> 1));
    }
    // (32-bit: the set-up keeps size() below 2^31)
    __device__ __forceinline__ int32_t at(int cn, int32_t ix, int32_t iy, int32_t iz) const {
        const int a = cn & 1, b = (cn >> 1) & 1, c = cn >> 2;
        const int32_t sx = a ? nx >> 1 : nx, sy = b ? ny >> 1 : ny, sz = c ? nz >> 1 : nz;
        const int32_t off = (c ? (nx + (nx >> 1)) * (ny + (ny >> 1)) * nz : 0) + (b ? (nx + (nx >> 1)) * ny * sz : 0) +
                            (a ? nx * sy * sz : 0);
        return off + (a ? ix >> 1 : ix) + sx * ((b ? iy >> 1 : iy) + sy * (c ? iz >> 1 : iz));
    }
    // at() for any node inside the lattice, clamped into the array: a load that
    // is always in bounds, whose value is used only where held() is true
    __device__ __forceinline__ int32_t atc(int cn, int32_t ix, int32_t iy, int32_t iz) const {
        return min(at(cn, ix, iy, iz), static_cast<int32_t>(size() - 1));
    }
    // whether corner cn can carry a nonzero weight for node (ix, iy, iz)
    __device__ __forceinline__ static bool held(int cn, int32_t ix, int32_t iy, int32_t iz) {
        return !((cn & 1) && !(ix & 1)) && !((cn & 2) && !(iy & 1)) && !((cn & 4) && !(iz & 1));
    }
};

// W rounded to FP32 in place (the Galerkin product then uses exactly the values
// the transfers apply) and its nonzero entries packed into Wc
__global__ __launch_bounds__(kMgT) void k_mg_wpack(LvArgs L, double* __restrict__ Wall, float* __restrict__ Wc) {
    const int sys = blockIdx.y;
    const WPack pk{L.nx, L.ny, L.nz};
    double* W = Wall + (int64_t)sys * L.N * 8;
    float* P = Wc + sys * pk.size();
    for (int64_t i = blockIdx.x * (int64_t)kMgT + threadIdx.x; i < L.N; i += (int64_t)gridDim.x * kMgT) {
        int ix, iy, iz;
        coords(static_cast<int32_t>(i), L.nx, L.ny, ix, iy, iz);
        for (int cn = 0; cn < 8; ++cn) {
            const float v = static_cast<float>(W[cn * L.N + i]);
            W[cn * L.N + i] = static_cast<double>(v);
            if (WPack::held(cn, ix, iy, iz)) P[pk.at(cn, ix, iy, iz)] = v;
        }
    }
}

// Galerkin coarse operator A_c = P^T A P, diagonal and the 13 upper offsets
// (code order (dx+1) + 3 (dy+1) + 9 (dz+1) = 13 ... 26) of every coarse node:
// sum over the fine nodes i in the support of I, the fine stencil entries
// a_ij, and the coarse nodes J whose support holds j, of P(i,I) a_ij P(j,J).
// W: [nsys][8][N] weights of P, or null (trilinear).
// 32 lanes share a coarse node, one for each of the 27 fine nodes of its support,
// and their sums are added in LDS in that order. With one thread a coarse node
// the few thousand serial loads of a thread bounded every level alike (560 us
// a level at 65^3, 370 us at 17^3). A fine row's loads go out together (M: room
// for its stored upper offsets), and the sums go to LDS as adds nobody waits
// for, each thread its own column (the four levels of 97^3: 382 -> 319 us).
constexpr int kRapLanes = 32;
constexpr int kRapNodes = kMgT / kRapLanes;   // coarse nodes a block
template <int M>
__global__ __launch_bounds__(kMgT) void k_mg_rap(LvArgs F, const double* __restrict__ Wall, double* __restrict__ Uc,
                                                 int cx, int cy, int cz) {
    __shared__ double acc[14][kMgT];
    const int sys = blockIdx.y;
    const int64_t Nc = (int64_t)cx * cy * cz;
    const int64_t I0 = blockIdx.x * (int64_t)kRapNodes, I = I0 + threadIdx.x / kRapLanes;
    const int di = threadIdx.x % kRapLanes;
    const int Mf = F.m + 1;
    const double* U = F.U + (int64_t)sys * F.N * Mf;
    const double* W = Wall ? Wall + (int64_t)sys * F.N * 8 : nullptr;
    for (int k = 0; k < 14; ++k) acc[k][threadIdx.x] = 0.0;
    int Ix, Iy, Iz;
    coords(static_cast<int32_t>(min(I, Nc - 1)), cx, cy, Ix, Iy, Iz);
    const int ax = di % 3 - 1, ay = (di / 3) % 3 - 1, az = di / 9 - 1;
    const int fx = 2 * Ix + ax, fy = 2 * Iy + ay, fz = 2 * Iz + az;
    const bool in = I < Nc && di < 27 && fx >= 0 && fx < F.nx && fy >= 0 && fy < F.ny && fz >= 0 && fz < F.nz;
    if (in) {
        const int32_t i = fx + F.nx * (fy + F.ny * fz);
        // I = J0(i) + corner, corner 1 exactly along the axes where i sits below 2 I
        const double wi = pweight(W, F.N, i, fx, fy, fz, (ax < 0 ? 1 : 0) + (ay < 0 ? 2 : 0) + (az < 0 ? 4 : 0));
        // the fine row: lower entries, diagonal, upper entries
        double a[2 * M + 1];
        const auto off = [&](int s) {   // dx, dy, dz, linear
            const int4 t = F.tab[abs(s) <= F.m ? abs(s) - 1 : 0];
            return s > 0 ? t : make_int4(-t.x, -t.y, -t.z, -t.w);
        };
        const auto at = [&](int s, const int4& t) {   // on the lattice
            const int jx = fx + t.x, jy = fy + t.y, jz = fz + t.z;
            return abs(s) <= F.m && jx >= 0 && jx < F.nx && jy >= 0 && jy < F.ny && jz >= 0 && jz < F.nz;
        };
#pragma unroll
        for (int s = -M; s <= M; ++s) {
            const int4 t = s ? off(s) : make_int4(0, 0, 0, 0);
            const bool on = s == 0 || at(s, t);
            a[s + M] = U[(int64_t)(on && s < 0 ? i + t.w : i) * Mf + (on ? abs(s) : 0)];
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int s = -M; s <= M; ++s) {
            const int4 t = s ? off(s) : make_int4(0, 0, 0, 0);
            if ((s != 0 && !at(s, t)) || wi == 0.0) continue;
            const int jx = fx + t.x, jy = fy + t.y, jz = fz + t.z;
            const int32_t j = i + t.w;
            const double wa = wi * a[s + M];
            // corners that can carry a weight: one step up only along odd axes
            const int px = jx & 1, py = jy & 1, pz = jz & 1;
            const int code0 = ((jx >> 1) - Ix) + 3 * ((jy >> 1) - Iy) + 9 * ((jz >> 1) - Iz);
#pragma unroll
            for (int cj = 0; cj < 8; ++cj) {
                const int bx = cj & 1, by = (cj >> 1) & 1, bz = cj >> 2;
                if (bx > px || by > py || bz > pz) continue;
                const int code = code0 + bx + 3 * by + 9 * bz;   // the lower half is stored at the partner row
                if (code < 0) continue;
                const double wj = W ? W[cj * F.N + j] : (px ? 0.5 : 1.0) * (py ? 0.5 : 1.0) * (pz ? 0.5 : 1.0);
                (void)__hip_atomic_fetch_add(&acc[code][threadIdx.x], wa * wj, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            }
        }
    }
    __syncthreads();
    const int node = threadIdx.x / 14, k = threadIdx.x % 14;
    if (node < kRapNodes && I0 + node < Nc) {
        double t = 0.0;
#pragma unroll
        for (int d = 0; d < 27; ++d) t += acc[k][node * kRapLanes + d];
        Uc[((int64_t)sys * Nc + I0 + node) * 14 + k] = t;
    }
}

// ------------------------------------------------ operator-dependent transfer
// Prolongation weights from the operator (M_delta, whose diffusivity drops by
// orders of magnitude across the edges of the image). A fine node with one odd
// coordinate takes its two coarse neighbours along that axis with weights
// -C(-1)/C(0), -C(+1)/C(0) of its stencil collapsed onto the axis (summed
// over the two even axes); one with two odd coordinates combines its eight
// in-plane neighbours (interpolated already) with the stencil collapsed over
// the even axis; one with three odd coordinates its 26 neighbours with the
// stencil itself. Across an interface the weights towards the weakly coupled
// side vanish, so the coarse levels keep the regions apart where trilinear
// interpolation would mix them. A node whose collapsed centre is not positive,
// or that has no +1 neighbour along an odd axis, keeps the trilinear weights.
// Parity class = number of odd coordinates; classes run in order 0 ... 3.
template <int CLASS>
__global__ __launch_bounds__(kMgT) void k_mg_pweights(LvArgs L, double* __restrict__ Wall) {
    const int sys = blockIdx.y;
    const int M1 = L.m + 1;
    const double* U = L.U + (int64_t)sys * L.N * M1;
    double* W = Wall + (int64_t)sys * L.N * 8;
    for (int64_t i = blockIdx.x * (int64_t)kMgT + threadIdx.x; i < L.N; i += (int64_t)gridDim.x * kMgT) {
        int ix, iy, iz;
        coords(static_cast<int32_t>(i), L.nx, L.ny, ix, iy, iz);
        const int px = ix & 1, py = iy & 1, pz = iz & 1;
        if (px + py + pz != CLASS) continue;
        double w[8];
        for (int c = 0; c < 8; ++c) w[c] = pweight(nullptr, L.N, i, ix, iy, iz, c);
        bool ok = CLASS > 0 && !(px && ix + 1 >= L.nx) && !(py && iy + 1 >= L.ny) && !(pz && iz + 1 >= L.nz);
        if (ok) {
            // the row, collapsed over the even axes: C[(dx+1) + 3 (dy+1) + 9 (dz+1)]
            double C[27];
            for (int k = 0; k < 27; ++k) C[k] = 0.0;
            auto put_c = [&](int dx, int dy, int dz, double v) {
                C[(px ? dx + 1 : 1) + 3 * (py ? dy + 1 : 1) + 9 * (pz ? dz + 1 : 1)] += v;
            };
            put_c(0, 0, 0, U[i * M1]);
            for (int j = 0; j < L.m; ++j) {
                const int4 t = L.tab[j];
                if (ix + t.x >= 0 && ix + t.x < L.nx && iy + t.y >= 0 && iy + t.y < L.ny && iz + t.z < L.nz)
                    put_c(t.x, t.y, t.z, U[i * M1 + j + 1]);
                if (ix - t.x >= 0 && ix - t.x < L.nx && iy - t.y >= 0 && iy - t.y < L.ny && iz - t.z >= 0)
                    put_c(-t.x, -t.y, -t.z, U[(i - t.w) * M1 + j + 1]);
            }
            const double c0 = C[13];
            double acc[8];
            for (int c = 0; c < 8; ++c) acc[c] = 0.0;
            for (int k = 0; k < 27 && ok; ++k) {
                if (k == 13 || C[k] == 0.0) continue;
                const int dx = k % 3 - 1, dy = (k / 3) % 3 - 1, dz = k / 9 - 1;
                const int nxp = ix + dx, nyp = iy + dy, nzp = iz + dz;
                if (nxp < 0 || nxp >= L.nx || nyp < 0 || nyp >= L.ny || nzp < 0 || nzp >= L.nz) continue;
                const int64_t n = nxp + (int64_t)L.nx * (nyp + (int64_t)L.ny * nzp);
                const double f = -C[k] / c0;
                // the neighbour's weights, re-indexed to this node's corners
                for (int cn = 0; cn < 8; ++cn) {
                    const double wn = W[cn * L.N + n];
                    if (wn == 0.0) continue;
                    const int rx = (nxp >> 1) + (cn & 1) - (ix >> 1);
                    const int ry = (nyp >> 1) + ((cn >> 1) & 1) - (iy >> 1);
                    const int rz = (nzp >> 1) + (cn >> 2) - (iz >> 1);
                    if (rx < 0 || rx > 1 || ry < 0 || ry > 1 || rz < 0 || rz > 1) {
                        ok = false;
                        break;
                    }
                    acc[rx + 2 * ry + 4 * rz] += f * wn;
                }
            }
            ok = ok && c0 > 0.0;
            for (int c = 0; c < 8 && ok; ++c) ok = isfinite(acc[c]);
            if (ok)
                for (int c = 0; c < 8; ++c) w[c] = acc[c];
        }
        for (int c = 0; c < 8; ++c) W[c * L.N + i] = w[c];
    }
}

struct SmArgs {
    LvArgs L;
    const double* dinv;  // [nsys][N]
    const double* w;     // [nsys][levels]
    int32_t nlev, lev, nsys;
    const MgScal* sc;    // [nsys][B]
};

// x = w D^{-1} b (the first sweep from zero; on the finest level only at the
// start of a run, elsewhere the kernel that writes b also writes x)
template <int B, typename VT = double>
__global__ __launch_bounds__(kMgT) void k_mg_first(SmArgs a, const double* __restrict__ b, VT* __restrict__ x) {
    const int k = threadIdx.x % B;
    for (int sys = blockIdx.y; sys < a.nsys; sys += gridDim.y) {
        if (!a.sc[sys * B + k].active) continue;
        const double w = a.w[sys * a.nlev + a.lev];
        const int64_t o = sys * a.L.N * B;
        const double* dinv = a.dinv + sys * a.L.N;
        QPAT_MG_ELEMS(e, a.L.N * B) x[o + e] = static_cast<VT>(w * dinv[e / B] * b[o + e]);
    }
}

// y = x + w D^{-1} (b - A x). The systems are swept one after the other by
// the same blocks. DOTS (the last sweep on the finest level, where b = r and
// y = z): also the partial sums r.z of every right-hand side and, for one (M_delta's
// deflation), sum z and sum r, of y as stored. x and y in FP64 or FP32 (VT).
template <int KIND, int B, bool DOTS, typename VT = double>
__global__ __launch_bounds__(kMgT) void k_mg_smooth(SmArgs a, const double* __restrict__ b,
                                                    const VT* __restrict__ x, VT* __restrict__ y,
                                                    double* __restrict__ parts) {
    using T = TB<B>;
    constexpr int V = Pk<B>::V;
    __shared__ double sm[kSumLds];
    const int v = threadIdx.x % Pk<B>::BV;
    for (int sys = blockIdx.y; sys < a.nsys; sys += gridDim.y) {
        const double w = a.w[sys * a.nlev + a.lev];
        const double* U = rows_of<KIND>(a.L, sys);
        const double* dinv = a.dinv + sys * a.L.N;
        const int64_t o = sys * a.L.N * B + v * V;
        const double* bs = b + o;
        const VT* xs = x + o;
        VT* ys = y + o;
        T rz = 0.0, z1 = 0.0, r1 = 0.0;
        if (pair_active<B>(a.sc, sys, v)) {
            walk<Pk<B>::BV>(a.L.nx, a.L.ny, a.L.nz, [&](int32_t ix, int32_t iy, int32_t iz, int32_t i, int32_t) {
                const T bi = vld<T>(bs + i * B);
                const T ax = apply<KIND, B>(a.L, U, VecAt<B, VT>{xs}, ix, iy, iz, i);
                T yi = vldx<T>(xs + i * B) + (w * dinv[i]) * (bi - ax);
                if constexpr (sizeof(VT) == 4) {
                    static_assert(B == 1, "FP32 sweep output: one right-hand side per thread");
                    yi = held_as<float>(yi);
                }
                vstx<T>(ys + i * B, yi);
                if constexpr (DOTS) {
                    rz += bi * yi;
                    z1 += yi;
                    r1 += bi;
                }
            });
        }
        if constexpr (DOTS) {
            if constexpr (B == 1)   // M_delta's deflation
                put_sums<B, 0, 2, 3>(parts, sys, {rz, z1, r1}, sm);
            else
                put_sums<B, 0>(parts, sys, {rz}, sm);
        }
    }
}

// r = b - A x (x and r in FP64 or FP32: VT)
template <int KIND, int B, typename VT = double>
__global__ __launch_bounds__(kMgT) void k_mg_resid(SmArgs a, const double* __restrict__ b,
                                                   const VT* __restrict__ x, VT* __restrict__ r) {
    using T = TB<B>;
    constexpr int V = Pk<B>::V;
    const int v = threadIdx.x % Pk<B>::BV;
    for (int sys = blockIdx.y; sys < a.nsys; sys += gridDim.y) {
        if (!pair_active<B>(a.sc, sys, v)) continue;
        const double* U = rows_of<KIND>(a.L, sys);
        const int64_t o = sys * a.L.N * B + v * V;
        const double* bs = b + o;
        const VT* xs = x + o;
        VT* rs = r + o;
        walk<Pk<B>::BV>(a.L.nx, a.L.ny, a.L.nz, [&](int32_t ix, int32_t iy, int32_t iz, int32_t i, int32_t) {
            vstx<T>(rs + i * B, vld<T>(bs + i * B) - apply<KIND, B>(a.L, U, VecAt<B, VT>{xs}, ix, iy, iz, i));
        });
    }
}

// the two coarse nodes (or one) whose support holds fine node i along an
// axis: J0 = i / 2 (weight 1 if i is even, 1/2 if odd) and J0 + 1 (1/2 if odd)
struct Span {
    int32_t j0, j1;
    double w0, w1;
    __device__ __forceinline__ Span(int32_t i, int32_t c) {
        j0 = i >> 1;
        const bool odd = i & 1;
        j1 = min(j0 + (odd ? 1 : 0), c - 1);
        w0 = odd ? 0.5 : 1.0;
        w1 = odd ? 0.5 : 0.0;
    }
};

// bc = P^T r on the coarse level c, and the first sweep there, xc = w D^{-1} bc
// (r in FP64 or FP32: RT).
// Fine nodes 2 I + {-1, 0, 1} per axis, weights 1/2, 1, 1/2 (trilinear) or
// from Wc ([nsys][WPack size], operator-dependent, packed); the ones past the
// lattice get weight 0 (their loads are clamped inside it).
template <int B, bool OPW, typename RT = double>
__global__ __launch_bounds__(kMgT) void k_mg_restrict(SmArgs c, int32_t nx, int32_t ny, int32_t nz,
                                                      const RT* __restrict__ r, double* __restrict__ bc,
                                                      double* __restrict__ xc, const float* __restrict__ Wc) {
    using T = TB<B>;
    constexpr int V = Pk<B>::V;
    const int v = threadIdx.x % Pk<B>::BV;
    const int64_t Nf = (int64_t)nx * ny * nz, Nc = c.L.N;
    const WPack pk{nx, ny, nz};
    for (int sys = blockIdx.y; sys < c.nsys; sys += gridDim.y) {
        if (!pair_active<B>(c.sc, sys, v)) continue;
        const double w = c.w[sys * c.nlev + c.lev];
        const double* dinv = c.dinv + sys * Nc;
        const RT* rs = r + sys * Nf * B + v * V;
        const float* Ws = OPW ? Wc + sys * pk.size() : nullptr;
        const int64_t oc = sys * Nc * B + v * V;
        walk<Pk<B>::BV>(c.L.nx, c.L.ny, c.L.nz, [&](int32_t Ix, int32_t Iy, int32_t Iz, int32_t I, int32_t) {
            int32_t fx[3], fy[3], fz[3];
            double wx[3], wy[3], wz[3];
#pragma unroll
            for (int d = 0; d < 3; ++d) {
                const int32_t gx = 2 * Ix + d - 1, gy = 2 * Iy + d - 1, gz = 2 * Iz + d - 1;
                const double wd = d == 1 ? 1.0 : 0.5;
                wx[d] = gx >= 0 && gx < nx ? wd : 0.0;
                wy[d] = gy >= 0 && gy < ny ? wd : 0.0;
                wz[d] = gz >= 0 && gz < nz ? wd : 0.0;
                fx[d] = min(max(gx, 0), nx - 1);
                fy[d] = min(max(gy, 0), ny - 1);
                fz[d] = min(max(gz, 0), nz - 1);
            }
            // the 27 fine values (and weights) first (clamped indices, all loads
            // in flight together: the tiny levels are latency-bound), then the
            // sum in the order dz, dy, dx
            T fv[27];
            float wv[OPW ? 27 : 1];
#pragma unroll
            for (int dz = 0; dz < 3; ++dz)
#pragma unroll
                for (int dy = 0; dy < 3; ++dy) {
                    const int32_t row = nx * (fy[dy] + ny * fz[dz]);
#pragma unroll
                    for (int dx = 0; dx < 3; ++dx) {
                        const int k = (dz * 3 + dy) * 3 + dx;
                        fv[k] = vldx<T>(rs + (row + fx[dx]) * B);
                        // I is corner (d == 0 per axis) of fine node 2 I + d - 1, which is
                        // odd along each such axis: the packed entry exists where the
                        // node is inside the lattice (elsewhere the weight is 0 and the
                        // load, clamped, is not used)
                        if constexpr (OPW)
                            wv[k] = Ws[pk.atc((dx == 0) + 2 * (dy == 0) + 4 * (dz == 0), fx[dx], fy[dy], fz[dz])];
                    }
                }
            __builtin_amdgcn_sched_barrier(0);
            T s = 0.0;
#pragma unroll
            for (int dz = 0; dz < 3; ++dz)
#pragma unroll
                for (int dy = 0; dy < 3; ++dy) {
                    const double wyz = wy[dy] * wz[dz];
#pragma unroll
                    for (int dx = 0; dx < 3; ++dx) {
                        double wgt = wyz * wx[dx];
                        if constexpr (OPW)
                            if (wgt != 0.0) wgt = static_cast<double>(wv[(dz * 3 + dy) * 3 + dx]);
                        s += wgt * fv[(dz * 3 + dy) * 3 + dx];
                    }
                }
            vst<T>(bc + oc + I * B, s);
            vst<T>(xc + oc + I * B, (w * dinv[I]) * s);
        });
    }
}

// k_mg_resid on level f and k_mg_restrict into level c in one pass: 32 lanes a
// coarse node, each of the first 27 forming the residual at one fine node of
// its support (every fine residual is formed up to 8 times, and never stored)
// and the weighted sum taken across the lanes. One launch less on the levels
// where launches are the time (fuse_small): 4.8 us against 4.3 + 3.8 on 17^3
// nodes with 4 right-hand sides.
template <int KIND, int B, bool OPW, typename VT = double>
__global__ __launch_bounds__(kMgT) void k_mg_resid_restrict(SmArgs f, SmArgs c, const double* __restrict__ b,
                                                            const VT* __restrict__ x, double* __restrict__ bc,
                                                            double* __restrict__ xc, const float* __restrict__ Wc) {
    using T = TB<B>;
    constexpr int V = Pk<B>::V, BV = Pk<B>::BV;
    const int32_t nx = f.L.nx, ny = f.L.ny, nz = f.L.nz;
    const int64_t Nf = f.L.N, Nc = c.L.N;
    const int sub = threadIdx.x & 31;
    const int64_t item = (blockIdx.x * (int64_t)kMgT + threadIdx.x) >> 5;
    if (item >= Nc * BV) return;   // whole groups of 32 lanes
    const int v = static_cast<int>(item % BV);
    const int32_t I = static_cast<int32_t>(item / BV);
    const WPack pk{nx, ny, nz};
    int32_t Ix, Iy, Iz;
    coords(I, c.L.nx, c.L.ny, Ix, Iy, Iz);
    const int dx = sub % 3, dy = (sub / 3) % 3, dz = sub / 9;
    const int32_t gx = 2 * Ix + dx - 1, gy = 2 * Iy + dy - 1, gz = 2 * Iz + dz - 1;
    const bool in = sub < 27 && gx >= 0 && gx < nx && gy >= 0 && gy < ny && gz >= 0 && gz < nz;
    for (int sys = blockIdx.y; sys < f.nsys; sys += gridDim.y) {
        if (!pair_active<B>(c.sc, sys, v)) continue;
        T s = 0.0;
        if (in) {
            const int32_t i = gx + nx * (gy + ny * gz);
            double wgt;
            if constexpr (OPW)
                wgt = static_cast<double>(
                    (Wc + sys * pk.size())[pk.atc((dx == 0) + 2 * (dy == 0) + 4 * (dz == 0), gx, gy, gz)]);
            else
                wgt = (dx == 1 ? 1.0 : 0.5) * (dy == 1 ? 1.0 : 0.5) * (dz == 1 ? 1.0 : 0.5);
            const int64_t o = sys * Nf * B + v * V;
            T ri = vld<T>(b + o + i * B) -
                   apply<KIND, B>(f.L, rows_of<KIND>(f.L, sys), VecAt<B, VT>{x + o}, gx, gy, gz, i);
            if constexpr (sizeof(VT) == 4) ri = held_as<VT>(ri);   // as the two kernels store it between them
            s = wgt * ri;
        }
        double t[V];
#pragma unroll
        for (int k = 0; k < V; ++k) {
            t[k] = comp(s, k);
#pragma unroll
            for (int off = 16; off >= 1; off >>= 1) t[k] += __shfl_xor(t[k], off);
        }
        if (sub == 0) {
            const double wd = c.w[sys * c.nlev + c.lev] * c.dinv[sys * Nc + I];
            const int64_t oc = sys * Nc * B + I * (int64_t)B + v * V;
#pragma unroll
            for (int k = 0; k < V; ++k) {
                bc[oc + k] = t[k];
                xc[oc + k] = wd * t[k];
            }
        }
    }
}

// x = x + P xc on fine level f (coarse lattice cx, cy, cz). P: trilinear, or
// the packed weights Wc ([nsys][WPack size]).
template <int B, bool OPW, bool XF = false>
__global__ __launch_bounds__(kMgT) void k_mg_prolong(SmArgs f, int32_t cx, int32_t cy, int32_t cz,
                                                     const double* __restrict__ xc, double* __restrict__ x,
                                                     const float* __restrict__ Wc) {
    using T = TB<B>;
    constexpr int V = Pk<B>::V;
    const int v = threadIdx.x % Pk<B>::BV;
    const int64_t Nf = f.L.N, Nc = (int64_t)cx * cy * cz;
    for (int sys = blockIdx.y; sys < f.nsys; sys += gridDim.y) {
        if (!pair_active<B>(f.sc, sys, v)) continue;
        const double* xs = xc + sys * Nc * B + v * V;
        double* xf = x + sys * Nf * B + v * V;
        float* xf32 = reinterpret_cast<float*>(x) + sys * Nf * B + v * V;   // XF: the fine x in FP32
        const WPack pk{f.L.nx, f.L.ny, f.L.nz};
        const float* Ws = OPW ? Wc + sys * pk.size() : nullptr;
        walk<Pk<B>::BV>(f.L.nx, f.L.ny, f.L.nz, [&](int32_t ix, int32_t iy, int32_t iz, int32_t i, int32_t) {
            const Span sx(ix, cx), sy(iy, cy), sz(iz, cz);
            const int32_t jx[2] = {sx.j0, sx.j1}, jy[2] = {sy.j0, sy.j1}, jz[2] = {sz.j0, sz.j1};
            const double wx[2] = {sx.w0, sx.w1}, wy[2] = {sy.w0, sy.w1}, wz[2] = {sz.w0, sz.w1};
            T s;
            if constexpr (XF)
                s = vldf<T>(xf32 + i * B);
            else
                s = vld<T>(xf + i * B);
            // the 8 coarse values (and weights) first, all loads in flight together
            T cv[8];
            double wgt[8];
#pragma unroll
            for (int c2 = 0; c2 < 2; ++c2)
#pragma unroll
                for (int b2 = 0; b2 < 2; ++b2) {
                    const int32_t row = cx * (jy[b2] + cy * jz[c2]);
                    const double wyz = wy[b2] * wz[c2];
#pragma unroll
                    for (int a2 = 0; a2 < 2; ++a2) {
                        // corner (a2, b2, c2) from J0 = (ix/2, iy/2, iz/2); Span
                        // clamps the index of a zero-weight corner
                        const int cn = a2 + 2 * b2 + 4 * c2;
                        if constexpr (OPW)
                            wgt[cn] = static_cast<double>(Ws[pk.atc(cn, ix, iy, iz)]);
                        else
                            wgt[cn] = wyz * wx[a2];
                        cv[cn] = vld<T>(xs + (row + jx[a2]) * B);
                    }
                }
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (OPW)
#pragma unroll
                for (int cn = 0; cn < 8; ++cn)
                    if (!WPack::held(cn, ix, iy, iz)) wgt[cn] = 0.0;
#pragma unroll
            for (int cn = 0; cn < 8; ++cn) s += wgt[cn] * cv[cn];
            if constexpr (XF)
                vstf<T>(xf32 + i * B, s);
            else
                vst<T>(xf + i * B, s);
        });
    }
}

// x = Ainv b on the coarsest level: one wavefront per output (system, row,
// thread-in-node), its lanes splitting the row and summing by shuffles
template <int B>
__global__ __launch_bounds__(kMgT) void k_mg_dense(int64_t Nc, int nsys, const double* __restrict__ ainv,
                                                   const double* __restrict__ b, double* __restrict__ x,
                                                   const MgScal* __restrict__ sc) {
    // block: kMgT / 64 rows (one per wavefront) of system blockIdx.z for the
    // thread-in-node pair blockIdx.y; that pair's column of b is staged in LDS
    using T = TB<B>;
    constexpr int V = Pk<B>::V;
    extern __shared__ __align__(16) unsigned char mg_smem[];
    T* bl = reinterpret_cast<T*>(mg_smem);   // [Nc]
    const int sys = blockIdx.z, v = blockIdx.y;
    if (!pair_active<B>(sc, sys, v)) return;   // uniform over the block
    const double* bs = b + sys * Nc * B + v * V;
    const int lane = threadIdx.x & 63;
    const int64_t I = blockIdx.x * (int64_t)(kMgT / 64) + (threadIdx.x >> 6);
    const double* A = ainv + (sys * Nc + min(I, Nc - 1)) * Nc;
    // a row's first 1024 entries in flight together, and beside the loads of b
    // (the coarsest solve is a chain of memory round trips)
    constexpr int NA = 16;
    double a[NA];
    const auto row = [&](int64_t J0) {
#pragma unroll
        for (int u = 0; u < NA; ++u) {
            const int64_t J = J0 + u * 64 + lane;
            a[u] = J < Nc ? A[J] : 0.0;
        }
    };
    row(0);
#pragma unroll 4
    for (int64_t J = threadIdx.x; J < Nc; J += kMgT) bl[J] = vld<T>(bs + J * B);
    __syncthreads();
    if (I >= Nc) return;   // whole wavefronts, after the barrier
    T s = 0.0;
    for (int64_t J0 = 0;;) {
#pragma unroll
        for (int u = 0; u < NA; ++u) s += a[u] * bl[min(J0 + u * 64 + lane, Nc - 1)];
        J0 += NA * 64;
        if (J0 >= Nc) break;
        row(J0);
    }
    double out[V];
#pragma unroll
    for (int c = 0; c < V; ++c) {
        double t = comp(s, c);
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) t += __shfl_xor(t, off);
        out[c] = t;
    }
    if (lane == 0) {
        double* xs = x + sys * Nc * B + v * V + I * B;
#pragma unroll
        for (int c = 0; c < V; ++c) xs[c] = out[c];
    }
}

// ---------------------------------------------------------------- PCG kernels
// The direction ping-pongs between two buffers (po: the last iteration's,
// pn: this one's), so that the fused direction + product kernel can read the
// old direction in the halo of a tile while other blocks write the new one.
struct PcgMg {
    LvArgs L;             // the fine operator
    double* x;            // [nsys][N][B] iterate
    double* r;
    double* po;
    double* pn;
    double* q;
    const double* z;
    double* parts;        // [lanes][4][kMgBlocks]
    MgScal* sc;           // [lanes]
    double rtol2;
    int32_t maxit, deflate, nsys;
    // region coarse space (one right-hand side per system), kreg = 0: off;
    // nbr: blocks of the kernels that write the region partials
    int32_t kreg, nbr;
    int32_t p32;          // 1: the direction in FP32 on the tiled 16-right-hand-side path (mixed precision)
    int32_t ring;         // kRing: directions and alphas kept in the ring (x formed later), 0: x updated each iteration
    int32_t* slot;        // the ring's iteration counter
    double* ahist;        // [kRing][lanes]
    const int32_t* reg;   // [nsys][N]
    const double* ry;     // [nsys][kRegMax]
    const double* rcorr;  // [nsys][2]: r.(Z y), mean(Z y)
};

// per-component choice between two V-wide values
__device__ __forceinline__ double pick(double a, double b, bool c0, bool) { return c0 ? a : b; }
__device__ __forceinline__ d2v pick(d2v a, d2v b, bool c0, bool c1) {
    d2v r;
    r.x = c0 ? a.x : b.x;
    r.y = c1 ? a.y : b.y;
    return r;
}

// the PCG scalars of thread-in-node v's right-hand sides as V-wide values
template <int B>
struct LaneScal {
    TB<B> alpha, beta, c;
    bool on0, on1;
    __device__ __forceinline__ LaneScal(const MgScal* sc, int sys, int v) {
        const MgScal& s0 = sc[sys * B + v * Pk<B>::V];
        const MgScal& s1 = sc[sys * B + v * Pk<B>::V + Pk<B>::V - 1];
        on0 = s0.active != 0;
        on1 = s1.active != 0;
        if constexpr (Pk<B>::V == 2) {
            alpha = d2v{s0.alpha, s1.alpha};
            beta = d2v{s0.beta, s1.beta};
            c = d2v{s0.c, s1.c};
        } else {
            alpha = s0.alpha;
            beta = s0.beta;
            c = s0.c;
        }
    }
};

// pn = z - c + beta po (right-hand sides that stopped keep pn); ZF: z in FP32
template <int B, bool ZF = false>
__global__ __launch_bounds__(kMgT) void k_mgp_dir(PcgMg a) {
    using T = TB<B>;
    constexpr int V = Pk<B>::V, BV = Pk<B>::BV;
    const int v = threadIdx.x % BV;
    for (int sys = blockIdx.y; sys < a.nsys; sys += gridDim.y) {
        const LaneScal<B> s(a.sc, sys, v);
        if (!s.on0 && !s.on1) continue;
        const int64_t o = sys * a.L.N * B + v * V;
        QPAT_MG_ELEMS(e, a.L.N * BV) {
            const int64_t at = o + (e / BV) * B;
            T zc = ZF ? vldf<T>(reinterpret_cast<const float*>(a.z) + at) : vld<T>(a.z + at);
            if constexpr (B == 1) {   // the region coarse-space part of z, y_reg(i) - ybar
                if (a.kreg > 0) {
                    const int32_t rg = a.reg[sys * a.L.N + e];
                    zc += (rg >= 0 ? a.ry[sys * kRegMax + rg] : 0.0) - a.rcorr[2 * sys + 1];
                }
            }
            const T pn = zc - s.c + s.beta * vld<T>(a.po + at);
            vst<T>(a.pn + at, s.on0 && s.on1 ? pn : pick(pn, vld<T>(a.pn + at), s.on0, s.on1));
        }
    }
}

// q = A pn, partial pn.q
template <int KIND, int B>
__global__ __launch_bounds__(kMgT) void k_mgp_spmv(PcgMg a) {
    using T = TB<B>;
    constexpr int V = Pk<B>::V;
    __shared__ double sm[kSumLds];
    const int v = threadIdx.x % Pk<B>::BV;
    for (int sys = blockIdx.y; sys < a.nsys; sys += gridDim.y) {
        const double* U = rows_of<KIND>(a.L, sys);
        const int64_t o = sys * a.L.N * B + v * V;
        const double* ps = a.pn + o;
        double* qs = a.q + o;
        T pq = 0.0;
        if (pair_active<B>(a.sc, sys, v)) {
            walk<Pk<B>::BV>(a.L.nx, a.L.ny, a.L.nz, [&](int32_t ix, int32_t iy, int32_t iz, int32_t i, int32_t) {
                const T qi = apply<KIND, B>(a.L, U, VecAt<B, double>{ps}, ix, iy, iz, i);
                vst<T>(qs + i * B, qi);
                pq += vld<T>(ps + i * B) * qi;
            });
        }
        put_sums<B, 0>(a.parts, sys, {pq}, sm);
    }
}

// The new direction z - c + beta po at a node, formed where it is read (ZF: z
// in FP32). reg, ytab: the region coarse-space part of z (one right-hand
// side per system), ytab[g + 1] = y_g - ybar with g = -1 for no region.
template <int B, bool ZF>
struct DirAt {
    const double* z;
    const double* po;
    TB<B> c, beta;
    const int32_t* reg;
    const double* ytab;
    __device__ __forceinline__ TB<B> operator()(int32_t i) const {
        using T = TB<B>;
        T zc = ZF ? vldf<T>(reinterpret_cast<const float*>(z) + i * B) : vld<T>(z + i * B);
        if constexpr (B == 1)
            if (reg) zc += ytab[reg[i] + 1];
        return zc - c + beta * vld<T>(po + i * B);
    }
};

// k_mgp_dir and k_mgp_spmv in one pass: pn = z - c + beta po, q = A pn, partial
// pn.q, every neighbour's direction formed again from z and po. Twice the
// vector reads of the two kernels, but one launch less: for the lattices
// where the launches, not the reads, are the time (fuse_small): 5.5 us
// against 2.9 + 5.3 on 17^3 nodes with 4 right-hand sides.
template <int KIND, int B, bool ZF = false>
__global__ __launch_bounds__(kMgT) void k_mgp_dir_spmv(PcgMg a) {
    using T = TB<B>;
    constexpr int V = Pk<B>::V;
    __shared__ double sm[kSumLds], ytab[kRegMax + 1];
    const int v = threadIdx.x % Pk<B>::BV;
    for (int sys = blockIdx.y; sys < a.nsys; sys += gridDim.y) {
        if (B == 1 && a.kreg > 0) {
            __syncthreads();
            if (threadIdx.x <= kRegMax)
                ytab[threadIdx.x] = (threadIdx.x > 0 ? a.ry[sys * kRegMax + threadIdx.x - 1] : 0.0) - a.rcorr[2 * sys + 1];
            __syncthreads();
        }
        const LaneScal<B> s(a.sc, sys, v);
        const double* U = rows_of<KIND>(a.L, sys);
        const int64_t o = sys * a.L.N * B + v * V;
        double* ps = a.pn + o;
        double* qs = a.q + o;
        T pq = 0.0;
        if (s.on0 || s.on1) {
            const double* zs = ZF ? reinterpret_cast<const double*>(reinterpret_cast<const float*>(a.z) + o) : a.z + o;
            const DirAt<B, ZF> p{zs, a.po + o, s.c, s.beta, B == 1 && a.kreg > 0 ? a.reg + sys * a.L.N : nullptr, ytab};
            walk<Pk<B>::BV>(a.L.nx, a.L.ny, a.L.nz, [&](int32_t ix, int32_t iy, int32_t iz, int32_t i, int32_t) {
                const T pi = p(i);
                const T qi = apply<KIND, B>(a.L, U, p, ix, iy, iz, i);
                vst<T>(ps + i * B, s.on0 && s.on1 ? pi : pick(pi, vld<T>(ps + i * B), s.on0, s.on1));
                vst<T>(qs + i * B, qi);
                pq += pi * qi;
            });
        }
        put_sums<B, 0>(a.parts, sys, {pq}, sm);
    }
}

// x += alpha pn, r -= alpha q (right-hand sides that stopped keep both),
// partial r.r, and the V-cycle's first sweep on the finest level, x0 =
// w D^{-1} r, from the new r where it is at hand
template <int B>
__global__ __launch_bounds__(kMgT) void k_mgp_update(PcgMg a, SmArgs m, double* __restrict__ x0) {
    using T = TB<B>;
    constexpr int V = Pk<B>::V, BV = Pk<B>::BV;
    __shared__ double sm[kSumLds];
    const int v = threadIdx.x % BV;
    for (int sys = blockIdx.y; sys < a.nsys; sys += gridDim.y) {
        const LaneScal<B> s(a.sc, sys, v);
        const int64_t o = sys * a.L.N * B + v * V;
        T rr = 0.0;
        if (s.on0 || s.on1) {
            const double w = m.w[sys * m.nlev + m.lev];
            const double* dinv = m.dinv + sys * a.L.N;
            QPAT_MG_ELEMS(e, a.L.N * BV) {
                const int64_t at = o + (e / BV) * B;
                const double wd = w * dinv[e / BV];
                const T p = vld<T>(a.pn + at), r = vld<T>(a.r + at), x = vld<T>(a.x + at);
                const T rn = pick(r - s.alpha * vld<T>(a.q + at), r, s.on0, s.on1);
                vst<T>(a.x + at, pick(x + s.alpha * p, x, s.on0, s.on1));
                vst<T>(a.r + at, rn);
                vst<T>(x0 + at, wd * rn);
                rr += rn * rn;
            }
        }
        put_sums<B, 1>(a.parts, sys, {rr}, sm);
    }
}

// Deterministic sums of NS slots of one lane's partials, written by nb blocks
// (one block of kMgT threads). The constructor issues every load, take() adds:
// the one-block kernels that use this are a chain of memory round trips and
// little else, and this way the partials come beside the lane's scalars.
template <int NS>
struct Red {
    static constexpr int NL = kMgBlocks / kMgT;
    double v[NS][NL];
    __device__ __forceinline__ Red(const double* parts, int nb, int lane, const int (&slot)[NS]) {
#pragma unroll
        for (int c = 0; c < NS; ++c) {
            const double* p = parts + (lane * 4 + slot[c]) * kMgBlocks;
#pragma unroll
            for (int u = 0; u < NL; ++u) {
                const int b = u * kMgT + static_cast<int>(threadIdx.x);
                v[c][u] = u * kMgT < nb && b < nb ? p[b] : 0.0;
            }
        }
    }
    // the sums, valid in thread 0 (sm: NS doubles a wavefront)
    __device__ __forceinline__ void take(double* sm, double (&out)[NS]) const {
        const int ln = threadIdx.x & 63, wave = threadIdx.x >> 6;
        double s[NS];
#pragma unroll
        for (int c = 0; c < NS; ++c) {
            s[c] = 0.0;
#pragma unroll
            for (int u = 0; u < NL; ++u) s[c] += v[c][u];
        }
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1)
#pragma unroll
            for (int c = 0; c < NS; ++c) s[c] += __shfl_xor(s[c], off);
        if (ln == 0)
#pragma unroll
            for (int c = 0; c < NS; ++c) sm[wave * NS + c] = s[c];
        __syncthreads();
#pragma unroll
        for (int c = 0; c < NS; ++c) {
            out[c] = 0.0;
            if (threadIdx.x == 0)
                for (int w = 0; w < kMgT / 64; ++w) out[c] += sm[w * NS + c];
        }
    }
};

// phase 1 of k_mgp_scalars for one lane that iterates (thread 0 writes)
__device__ __forceinline__ void scalars_rr(const PcgMg& a, const Red<1>& part, int lane, double* sm) {
    MgScal& s = a.sc[lane];
    const double tol = a.rtol2 * s.bnorm2;
    const int iters = s.iters + 1;
    double rr[1];
    part.take(sm, rr);
    if (threadIdx.x == 0) {
        s.rr = rr[0];
        s.iters = iters;
        if (rr[0] <= tol) {
            s.done = 1;
            s.active = 0;
        } else if (iters >= a.maxit) {
            s.active = 0;
        }
    }
}

// one block per lane (blockIdx.y); nb blocks wrote the partials. phase 0:
// alpha = rz / pq; phase 1: rr, convergence, iteration count; phase 2 (after
// the V-cycle): c, beta, rz; phase 3: start of a run (after its first
// V-cycle): c, rz, beta = 0
__global__ __launch_bounds__(kMgT) void k_mgp_scalars(PcgMg a, int nb, int phase) {
    __shared__ double sm[(kMgT / 64) * 3];
    const int lane = blockIdx.y;
    MgScal& s = a.sc[lane];
    const bool mean = phase >= 2 && a.deflate;   // the sums of z and r as well
    const Red<1> p1(a.parts, mean ? 0 : nb, lane, {phase == 1 ? 1 : 0});
    const Red<3> p3(a.parts, mean ? nb : 0, lane, {0, 2, 3});
    const double rz_old = s.rz;
    // the direction ring: each iteration's alpha per lane (0 where the lane did
    // not iterate), and the iteration counter, advanced once at the end of an
    // iteration (phase 2, lane 0's block)
    const bool on = s.active != 0;
    if (a.ring > 0 && threadIdx.x == 0) {
        if (phase == 0 && !on) a.ahist[(*a.slot % a.ring) * gridDim.y + lane] = 0.0;
        if (phase == 2 && lane == 0) *a.slot += 1;
    }
    if (!on) return;
    if (phase == 0) {
        const int slot = a.ring > 0 ? *a.slot % a.ring : 0;
        double pq[1];
        p1.take(sm, pq);
        if (threadIdx.x == 0) {
            s.pq = pq[0];
            const double alpha = pq[0] != 0.0 ? rz_old / pq[0] : 0.0;
            s.alpha = alpha;
            if (a.ring > 0) a.ahist[slot * gridDim.y + lane] = alpha;
        }
    } else if (phase == 1) {
        scalars_rr(a, p1, lane, sm);
    } else {
        double v[3] = {0.0, 0.0, 0.0};
        if (mean) {
            p3.take(sm, v);
        } else {
            double v0[1];
            p1.take(sm, v0);
            v[0] = v0[0];
        }
        double rz = v[0];
        const double z1 = v[1], r1 = v[2];
        if (threadIdx.x == 0) {
            // z = V(r) + Z y; with deflation its mean is mean(V(r)) + ybar, and the
            // direction takes (V(r) - mean V(r)) + (Z y - ybar): the large, nearly
            // constant part of Z y never passes through the sum with V(r)
            double ybar = 0.0;
            if (a.kreg > 0) {
                rz += a.rcorr[2 * lane];
                ybar = a.rcorr[2 * lane + 1];
            }
            const double c = a.deflate ? z1 / static_cast<double>(a.L.N) : 0.0;
            rz -= (c + ybar) * r1;     // r.(z - mean z)
            s.c = c;
            s.beta = (phase == 2 && rz_old != 0.0) ? rz / rz_old : 0.0;
            s.rz = rz;
        }
    }
}

// ---------------------------------------------------------- region coarse space
// Partial sums of Z^T r (one right-hand side per system): every thread adds
// its nodes into kRegMax register accumulators, then fixed-order block sums.
__global__ __launch_bounds__(kMgT) void k_reg_rsum(PcgMg a, double* __restrict__ rparts) {
    __shared__ double sm[(kMgT / 64) * kRegMax];
    for (int sys = blockIdx.y; sys < a.nsys; sys += gridDim.y) {
        if (!a.sc[sys].active) continue;   // uniform over the block
        double acc[kRegMax];
#pragma unroll
        for (int j = 0; j < kRegMax; ++j) acc[j] = 0.0;
        const int32_t* rg = a.reg + sys * a.L.N;
        const double* r = a.r + sys * a.L.N;
        // grid-stride order, four nodes' loads in flight per trip
        const int64_t n = a.L.N, stride = (int64_t)gridDim.x * kMgT;
        for (int64_t i0 = blockIdx.x * (int64_t)kMgT + threadIdx.x; i0 < n; i0 += 4 * stride) {
            int32_t g[4];
            double v[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int64_t i = i0 + q * stride;
                g[q] = i < n ? rg[i] : -1;
                v[q] = i < n ? r[i] : 0.0;
            }
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int j = 0; j < kRegMax; ++j) acc[j] += g[q] == j ? v[q] : 0.0;
        }
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
        for (int j = 0; j < kRegMax; ++j) {
            double t = acc[j];
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) t += __shfl_xor(t, off);
            if (lane == 0) sm[wave * kRegMax + j] = t;
        }
        __syncthreads();
        if (threadIdx.x < kRegMax) {
            double t = 0.0;
            for (int w = 0; w < kMgT / 64; ++w) t += sm[w * kRegMax + threadIdx.x];
            rparts[(sys * kRegMax + threadIdx.x) * kMgBlocks + blockIdx.x] = t;
        }
        __syncthreads();
    }
}

// One right-hand side per system: the PCG update fused with the two passes
// that read its new r next. x += alpha p, r -= alpha q (a system that
// stopped keeps both) and the partial r.r; the V-cycle's first sweep on the
// finest level, x0 = w D^{-1} r (FP64 or FP32: XT); and, with the region
// coarse space, the partial sums of Z^T r. Four nodes' loads in flight per trip (buffer loads
// with 32-bit offsets: N 8 < 2^31; past the end they read 0 and the stores
// drop); few, full blocks (kMgGrid), so that each block's reduction of its
// kRegMax region sums is spread over many nodes.
template <typename XT>
__global__ __launch_bounds__(kMgT, 4) void k_mgp_update_first(PcgMg a, SmArgs s, XT* __restrict__ x0,
                                                           double* __restrict__ rparts) {
    __shared__ double sm[(kMgT / 64) * kRegMax];
    const int64_t n = a.L.N, stride = (int64_t)gridDim.x * kMgT;
    for (int sys = blockIdx.y; sys < a.nsys; sys += gridDim.y) {
        const MgScal& sc = a.sc[sys];
        const bool regions = a.kreg > 0;
        double rr = 0.0, acc[kRegMax];
#pragma unroll
        for (int j = 0; j < kRegMax; ++j) acc[j] = 0.0;
        if (sc.active) {   // uniform over the grid
            const double alpha = sc.alpha, w = s.w[sys * s.nlev];
            const int64_t o = sys * n;
            const uint32_t nb8 = static_cast<uint32_t>(n) * 8u;
            const auto bp = rsrc(a.pn + o, nb8), bq = rsrc(a.q + o, nb8), bd = rsrc(s.dinv + o, nb8);
            const auto bx = rsrc(a.x + o, nb8), br = rsrc(a.r + o, nb8);
            const auto bs = rsrc(x0 + o, static_cast<uint32_t>(n) * static_cast<uint32_t>(sizeof(XT)));
            const auto bg = rsrc(a.reg + (regions ? o : 0), regions ? nb8 / 2 : 0u);
            for (int64_t i0 = blockIdx.x * (int64_t)kMgT + threadIdx.x; i0 < n; i0 += 4 * stride) {
                double pv[4], qv[4], rv[4], xv[4], dv[4];
                int32_t gv[4];
                uint32_t off[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    off[u] = static_cast<uint32_t>(i0 + u * stride) * 8u;   // >= N 8 past the end
                    pv[u] = bload<double>(bp, off[u]);
                    qv[u] = bload<double>(bq, off[u]);
                    rv[u] = bload<double>(br, off[u]);
                    xv[u] = bload<double>(bx, off[u]);
                    dv[u] = bload<double>(bd, off[u]);
                    gv[u] = regions ? bload<int32_t>(bg, off[u] / 2) : -1;
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {   // nodes past the end: all zero, stores dropped
                    const double rn = rv[u] - alpha * qv[u];
                    bstore<double>(bx, off[u], xv[u] + alpha * pv[u]);
                    bstore<double>(br, off[u], rn);
                    bstore<XT>(bs, off[u] / (8u / sizeof(XT)), static_cast<XT>(w * dv[u] * rn));
                    rr += rn * rn;
                    if (regions)
#pragma unroll
                        for (int j = 0; j < kRegMax; ++j) acc[j] += gv[u] == j ? rn : 0.0;
                }
            }
        }
        const double t = group_sum<1>(rr, sm);
        if (threadIdx.x == 0) put(a.parts, sys, 1, t);
        if (regions) {   // fixed-order block sums of the region partials (as k_reg_rsum)
            const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
            for (int j = 0; j < kRegMax; ++j) {
                double v = acc[j];
#pragma unroll
                for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off);
                if (lane == 0) sm[wave * kRegMax + j] = v;
            }
            __syncthreads();
            if (threadIdx.x < kRegMax) {
                double v = 0.0;
                for (int wv = 0; wv < kMgT / 64; ++wv) v += sm[wv * kRegMax + threadIdx.x];
                rparts[(sys * kRegMax + threadIdx.x) * kMgBlocks + blockIdx.x] = v;
            }
            __syncthreads();
        }
    }
}

// y = E^{-1} Z^T r and the corrections r.(Z y), mean(Z y) (deflation) of the
// dot products and the direction; one block per system (blockIdx.y).
// nb > 0: first phase 1 of k_mgp_scalars for the system's one right-hand side,
// from the nb partials that the update left beside those of Z^T r
__global__ __launch_bounds__(kMgT) void k_reg_solve(PcgMg a, int nb, const double* __restrict__ rparts,
                                                    const double* __restrict__ einv, const double* __restrict__ rsize,
                                                    double* __restrict__ ry, double* __restrict__ rcorr) {
    __shared__ double zr[kRegMax], yy[kRegMax];
    const int sys = blockIdx.y;
    if (!a.sc[sys].active) return;   // as it was before this kernel: uniform over the block
    if (nb > 0) {
        __syncthreads();             // every thread has read active
        __shared__ double sm[kMgT / 64];
        scalars_rr(a, Red<1>(a.parts, nb, sys, {1}), sys, sm);
    }
    const int t = threadIdx.x;
    {   // fixed-order block sums of the partials, every region in one pass
        // (slots of regions past kreg hold zeros)
        __shared__ double wsum[(kMgT / 64) * kRegMax];
        double s[kRegMax];
#pragma unroll
        for (int j = 0; j < kRegMax; ++j) s[j] = 0.0;
        for (int b = t; b < a.nbr; b += kMgT)
#pragma unroll
            for (int j = 0; j < kRegMax; ++j) s[j] += rparts[(sys * kRegMax + j) * kMgBlocks + b];
        const int lane = t & 63, wave = t >> 6;
#pragma unroll
        for (int j = 0; j < kRegMax; ++j) {
            double v = s[j];
#pragma unroll
            for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off);
            if (lane == 0) wsum[wave * kRegMax + j] = v;
        }
        __syncthreads();
        if (t < kRegMax) {
            double v = 0.0;
            for (int w = 0; w < kMgT / 64; ++w) v += wsum[w * kRegMax + t];
            zr[t] = t < a.kreg ? v : 0.0;
        }
        __syncthreads();
    }
    if (t < kRegMax) {
        double y = 0.0;
        for (int b = 0; b < a.kreg; ++b) y += einv[(sys * kRegMax + t) * kRegMax + b] * zr[b];
        yy[t] = t < a.kreg ? y : 0.0;
        ry[sys * kRegMax + t] = yy[t];
    }
    __syncthreads();
    if (t == 0) {   // r.(Z y), and with deflation ybar = mean(Z y)
        double c0 = 0.0, c1 = 0.0;
        for (int j = 0; j < a.kreg; ++j) {
            c0 += yy[j] * zr[j];
            c1 += yy[j] * rsize[sys * kRegMax + j];
        }
        rcorr[2 * sys] = c0;
        rcorr[2 * sys + 1] = a.deflate ? c1 / static_cast<double>(a.L.N) : 0.0;
    }
}

// ---- set-up: connected components of the strong couplings (labels converge
// to the smallest node id of each component), region sizes, E = Z^T A Z

// strong coupling of nodes i and j through a_ij
__device__ __forceinline__ bool strong(double aij, double aii, double ajj) {
    return fabs(aij) > kRegTheta * sqrt(fabs(aii * ajj));
}

__global__ __launch_bounds__(kMgT) void k_reg_init(int32_t* __restrict__ lab, int64_t N) {
    for (int64_t i = blockIdx.x * (int64_t)kMgT + threadIdx.x; i < N; i += (int64_t)gridDim.x * kMgT)
        lab[i] = static_cast<int32_t>(i);
}

// hook: every node and the root of its label take the smallest label among
// its strong neighbours
__global__ __launch_bounds__(kMgT) void k_reg_prop(LvArgs L, int32_t* lab, int32_t* __restrict__ flag) {
    const int M1 = L.m + 1;
    for (int64_t i = blockIdx.x * (int64_t)kMgT + threadIdx.x; i < L.N; i += (int64_t)gridDim.x * kMgT) {
        int ix, iy, iz;
        coords(static_cast<int32_t>(i), L.nx, L.ny, ix, iy, iz);
        const double aii = L.U[i * M1];
        const int32_t li = __hip_atomic_load(lab + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        int32_t mi = li;
        for (int j = 0; j < L.m; ++j) {
            const int4 t = L.tab[j];
            if (ix + t.x >= 0 && ix + t.x < L.nx && iy + t.y >= 0 && iy + t.y < L.ny && iz + t.z < L.nz) {
                const int64_t k = i + t.w;
                if (strong(L.U[i * M1 + j + 1], aii, L.U[k * M1]))
                    mi = min(mi, __hip_atomic_load(lab + k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
            }
            if (ix - t.x >= 0 && ix - t.x < L.nx && iy - t.y >= 0 && iy - t.y < L.ny && iz - t.z >= 0) {
                const int64_t k = i - t.w;
                if (strong(L.U[k * M1 + j + 1], aii, L.U[k * M1]))
                    mi = min(mi, __hip_atomic_load(lab + k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
            }
        }
        if (mi < li) {
            atomicMin(lab + li, mi);
            atomicMin(lab + i, mi);
            *flag = 1;
        }
    }
}

// pointer jumping: lab[i] <- lab[lab[i]]
__global__ __launch_bounds__(kMgT) void k_reg_jump(int32_t* lab, int64_t N) {
    for (int64_t i = blockIdx.x * (int64_t)kMgT + threadIdx.x; i < N; i += (int64_t)gridDim.x * kMgT) {
        const int32_t l = __hip_atomic_load(lab + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const int32_t ll = __hip_atomic_load(lab + l, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (ll < l) atomicMin(lab + i, ll);
    }
}

// component sizes; the lanes of a wavefront that share a label add once
// (one component holds most nodes, so per-node atomics would serialise)
__global__ __launch_bounds__(kMgT) void k_reg_count(const int32_t* __restrict__ lab, int32_t* __restrict__ cnt,
                                                    int64_t N) {
    const int lane = threadIdx.x & 63;
    for (int64_t i0 = blockIdx.x * (int64_t)kMgT; i0 < N; i0 += (int64_t)gridDim.x * kMgT) {
        const int64_t i = i0 + threadIdx.x;
        const int32_t l = i < N ? lab[i] : -1;
        unsigned long long todo = __ballot(l >= 0);
        while (todo) {
            const int leader = __ffsll(static_cast<long long>(todo)) - 1;
            const int32_t ll = __shfl(l, leader);
            const unsigned long long same = __ballot(l == ll) & todo;
            if (lane == leader) atomicAdd(cnt + ll, __popcll(same));
            todo &= ~same;
        }
    }
}

// components with at least kRegMin nodes: (root, size) pairs, in any order
__global__ __launch_bounds__(kMgT) void k_reg_roots(const int32_t* __restrict__ lab, const int32_t* __restrict__ cnt,
                                                    int64_t N, int32_t* __restrict__ list, int32_t* __restrict__ n) {
    for (int64_t i = blockIdx.x * (int64_t)kMgT + threadIdx.x; i < N; i += (int64_t)gridDim.x * kMgT) {
        if (lab[i] != i || cnt[i] < kRegMin) continue;
        const int32_t at = atomicAdd(n, 1);
        if (at < kRegList) {
            list[2 * at] = static_cast<int32_t>(i);
            list[2 * at + 1] = cnt[i];
        }
    }
}

__global__ __launch_bounds__(kMgT) void k_reg_assign(const int32_t* __restrict__ lab, int64_t N, int k,
                                                     const int32_t* __restrict__ roots, int32_t* __restrict__ reg) {
    for (int64_t i = blockIdx.x * (int64_t)kMgT + threadIdx.x; i < N; i += (int64_t)gridDim.x * kMgT) {
        int32_t r = -1;
        for (int j = 0; j < k; ++j)
            if (lab[i] == roots[j]) r = j;
        reg[i] = r;
    }
}

// largest |a_ij| (bit pattern of a non-negative double)
__global__ __launch_bounds__(kMgT) void k_reg_absmax(const double* __restrict__ U, int64_t n,
                                                     unsigned long long* __restrict__ out) {
    __shared__ double sm[kMgT / 64];
    double m = 0.0;
    for (int64_t e = blockIdx.x * (int64_t)kMgT + threadIdx.x; e < n; e += (int64_t)gridDim.x * kMgT)
        m = fmax(m, fabs(U[e]));
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) m = fmax(m, __shfl_xor(m, off));
    if ((threadIdx.x & 63) == 0) sm[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kMgT / 64; ++w) m = fmax(m, sm[w]);
        atomicMax(out, static_cast<unsigned long long>(__double_as_longlong(m)));
    }
}

// E = Z^T A Z in fixed point (scale: exact, order-independent integer sums):
// the diagonal entry of every node and each stored upper entry a_ij in both
// (reg i, reg j) and (reg j, reg i)
__global__ __launch_bounds__(kMgT) void k_reg_e(LvArgs L, const int32_t* __restrict__ reg, double scale,
                                                unsigned long long* __restrict__ eint) {
    __shared__ unsigned long long se[kRegMax * kRegMax];
    for (int t = threadIdx.x; t < kRegMax * kRegMax; t += kMgT) se[t] = 0ull;
    __syncthreads();
    const int M1 = L.m + 1;
    auto add = [&](int a, int b, double v) {
        const long long q = llrint(v * scale);
        atomicAdd(se + a * kRegMax + b, static_cast<unsigned long long>(q));
    };
    for (int64_t i = blockIdx.x * (int64_t)kMgT + threadIdx.x; i < L.N; i += (int64_t)gridDim.x * kMgT) {
        const int a = reg[i];
        if (a < 0) continue;
        int ix, iy, iz;
        coords(static_cast<int32_t>(i), L.nx, L.ny, ix, iy, iz);
        add(a, a, L.U[i * M1]);
        for (int j = 0; j < L.m; ++j) {
            const int4 t = L.tab[j];
            if (!(ix + t.x >= 0 && ix + t.x < L.nx && iy + t.y >= 0 && iy + t.y < L.ny && iz + t.z < L.nz)) continue;
            const int b = reg[i + t.w];
            if (b < 0) continue;
            const double v = L.U[i * M1 + j + 1];
            add(a, b, v);
            add(b, a, v);
        }
    }
    __syncthreads();
    for (int t = threadIdx.x; t < kRegMax * kRegMax; t += kMgT)
        if (se[t]) atomicAdd(eint + t, se[t]);
}

// partial sums of b and b.b per lane
template <int B>
__global__ __launch_bounds__(kMgT) void k_mgp_bstats(PcgMg a, const double* __restrict__ b) {
    __shared__ double sm[(kMgT / 64) * 16];
    for (int sys = blockIdx.y; sys < a.nsys; sys += gridDim.y) {
        const int64_t o = sys * a.L.N * B;
        double s1 = 0.0, s2 = 0.0;
        QPAT_MG_ELEMS(e, a.L.N * B) {
            s1 += b[o + e];
            s2 += b[o + e] * b[o + e];
        }
        s1 = group_sum<B>(s1, sm);
        s2 = group_sum<B>(s2, sm);
        if (threadIdx.x < B) {
            put(a.parts, sys * B + threadIdx.x, 2, s1);
            put(a.parts, sys * B + threadIdx.x, 3, s2);
        }
    }
}

// live: where this is the start's last kernel, its answer for the host
__global__ __launch_bounds__(kMgT) void k_mgp_init(PcgMg a, int nb, double inv_delta, Live live) {
    __shared__ double sm[(kMgT / 64) * 2];
    const int lane = blockIdx.y;
    if (a.ring > 0 && lane == 0 && threadIdx.x == 0) *a.slot = 0;   // a run's first iteration: slot 0
    double v[2];
    Red<2>(a.parts, nb, lane, {2, 3}).take(sm, v);
    const double s1 = v[0], s2 = v[1];
    if (threadIdx.x == 0) {
        MgScal& s = a.sc[lane];
        const double mean = a.deflate ? s1 / static_cast<double>(a.L.N) : 0.0;
        s.c = mean;                       // subtracted from b by k_mgp_start
        s.mean = mean * inv_delta;
        s.bnorm2 = s2;
        s.rz = s.pq = s.alpha = s.beta = 0.0;
        s.rr = s.rr0 = s2;
        s.iters = 0;
        s.done = s2 == 0.0 ? 1 : 0;       // b = 0: x = 0
        s.active = s2 == 0.0 ? 0 : 1;
        live.put(lane, s2 != 0.0);
    }
}

// The start of a run without deflation or initial guess in one pass: r = b,
// x = 0 and the partial sums of b and b.b that k_mgp_init reduces. (The
// first direction of the tiled path ignores the old direction, beta = 0.)
// With the direction ring x is not written here: its first formation starts
// from zero.
// A thread takes two right-hand sides of a node, four nodes' loads in flight
// (one value at a time: 174 us on 129^3 nodes with 16 right-hand sides, now
// 105 us; 97^3 71 -> 40).
template <int B>
__global__ __launch_bounds__(kMgT) void k_mgp_start0(PcgMg a, const double* __restrict__ b) {
    using T = TB<B>;
    constexpr int V = Pk<B>::V, BV = Pk<B>::BV, U = 4;
    __shared__ double sm[kSumLds];
    const int v = threadIdx.x % BV;
    const int64_t n = a.L.N * BV, stride = (int64_t)gridDim.x * kMgT;
    for (int sys = blockIdx.y; sys < a.nsys; sys += gridDim.y) {
        const int64_t o = sys * a.L.N * B + v * V;
        T s1 = 0.0, s2 = 0.0;
        for (int64_t e = blockIdx.x * (int64_t)kMgT + threadIdx.x; e < n; e += U * stride) {
            T bv[U];
#pragma unroll
            for (int u = 0; u < U; ++u) bv[u] = vld<T>(b + o + min(e + u * stride, n - BV + v) / BV * B);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (e + u * stride >= n) continue;
                const int64_t at = o + (e + u * stride) / BV * B;
                vst<T>(a.r + at, bv[u]);
                if (a.ring == 0) vst<T>(a.x + at, T(0.0));
                s1 += bv[u];
                s2 += bv[u] * bv[u];
            }
        }
        put_sums<B, 2, 3>(a.parts, sys, {s1, s2}, sm);
    }
}

// b -= mean; r = b; po = 0; x = 0 unless a start is given (and b != 0)
template <int B>
__global__ __launch_bounds__(kMgT) void k_mgp_start(PcgMg a, double* __restrict__ b, int has_x0) {
    const int k = threadIdx.x % B;
    for (int sys = blockIdx.y; sys < a.nsys; sys += gridDim.y) {
        const MgScal& s = a.sc[sys * B + k];
        const double m = s.c;
        const bool keep = has_x0 && s.active;
        const int64_t o = sys * a.L.N * B;
        QPAT_MG_ELEMS(e, a.L.N * B) {
            b[o + e] -= m;
            a.r[o + e] = b[o + e];
            if (!keep) a.x[o + e] = 0.0;
            a.po[o + e] = 0.0;
        }
    }
}

// true residual r = b - A x (compensated), partial r.r (also the start of a run from x0)
template <int KIND, int B>
__global__ __launch_bounds__(kMgT) void k_mgp_true(PcgMg a, const double* __restrict__ b) {
    using T = TB<B>;
    constexpr int V = Pk<B>::V;
    __shared__ double sm[kSumLds];
    const int v = threadIdx.x % Pk<B>::BV;
    const int32_t M1 = a.L.m + 1;
    for (int sys = blockIdx.y; sys < a.nsys; sys += gridDim.y) {
        const double* U = a.L.U + sys * a.L.N * M1;   // upper rows: the compensated sum walks the offset table
        const int64_t o = sys * a.L.N * B + v * V;
        const double* bs = b + o;
        const double* xs = a.x + o;
        double* rs = a.r + o;
        T rr = 0.0;
        walk<Pk<B>::BV>(a.L.nx, a.L.ny, a.L.nz, [&](int32_t ix, int32_t iy, int32_t iz, int32_t i, int32_t) {
            const T bi = vld<T>(bs + i * B);
            T ri;
            if (a.L.m == 7) {   // uniform: the loads of a row all in flight
                if constexpr (V == 2) {
                    ri.x = resid_comp7<B>(a.L, U, xs, bi.x, ix, iy, iz, i);
                    ri.y = resid_comp7<B>(a.L, U, xs + 1, bi.y, ix, iy, iz, i);
                } else {
                    ri = resid_comp7<B>(a.L, U, xs, bi, ix, iy, iz, i);
                }
            } else if constexpr (V == 2) {
                ri.x = resid_comp<B>(a.L, U, xs, bi.x, ix, iy, iz, i);
                ri.y = resid_comp<B>(a.L, U, xs + 1, bi.y, ix, iy, iz, i);
            } else {
                ri = resid_comp<B>(a.L, U, xs, bi, ix, iy, iz, i);
            }
            vst<T>(rs + i * B, ri);
            rr += ri * ri;
        });
        put_sums<B, 1>(a.parts, sys, {rr}, sm);
    }
}

__global__ __launch_bounds__(kMgT) void k_mgp_true_fin(PcgMg a, int nb, int reopen, Live live) {
    __shared__ double sm[kMgT / 64];
    const int lane = blockIdx.y;
    double v[1];
    Red<1>(a.parts, nb, lane, {1}).take(sm, v);
    const double rr = v[0];
    if (threadIdx.x == 0) {
        MgScal& s = a.sc[lane];
        s.rr = rr;
        if (s.iters == 0) s.rr0 = rr;
        const bool ok = rr <= a.rtol2 * s.bnorm2;
        s.done = ok ? 1 : 0;
        const bool on = !ok && reopen && s.iters < a.maxit;
        s.active = on ? 1 : 0;
        live.put(lane, on);
        s.rz = 0.0;   // a reopened run restarts its Krylov space from the true residual
    }
}


// x += alpha_j p_j over the ring slots of iterations f ... s - 1, in that order
// (the fused multiply-adds the update would have made one iteration at a
// time), for every element of the [N][B] iterate; lanes with alpha_j = 0 did
// not iterate then and keep x (their slot holds no direction of theirs). A
// thread takes the V elements of one 16-byte load of a direction (4 in FP32,
// 2 in FP64; B is a multiple of V), every slot's load in flight before the
// sums; the alphas of all slots are staged in LDS.
template <typename PT>
__global__ __launch_bounds__(kMgT) void k_mgp_ring_flush(int64_t n, int B, double* __restrict__ x,
                                                         const char* __restrict__ ring, int64_t stride,
                                                         const double* __restrict__ ahist, int lanes, int f, int s,
                                                         int x_zero) {
    constexpr int V = 16 / sizeof(PT);
    typedef PT PV __attribute__((ext_vector_type(V)));
    typedef double XV __attribute__((ext_vector_type(2)));
    __shared__ double al[kRing * kMgLanes];
    for (int i = threadIdx.x; i < kRing * lanes; i += kMgT) al[i] = ahist[i];
    __syncthreads();
    const int64_t nq = n / V;
    for (int64_t q = blockIdx.x * (int64_t)kMgT + threadIdx.x; q < nq; q += (int64_t)gridDim.x * kMgT) {
        const int64_t e0 = q * V;
        const int lane0 = static_cast<int>(e0 % B);
        PV pv[kRing];
#pragma unroll
        for (int t = 0; t < kRing; ++t) {
            const int sl = (f + t) % kRing;
            // each direction element is read once here: non-temporal
            pv[t] = f + t < s ? __builtin_nontemporal_load(reinterpret_cast<const PV*>(ring + sl * stride +
                                                                                        e0 * (int64_t)sizeof(PT)))
                              : PV{};
        }
        double xv[V];
#pragma unroll
        for (int c = 0; c < V; c += 2) {   // x_zero: the run started from x = 0, not yet stored
            const XV t2 = x_zero ? XV{0.0, 0.0} : *reinterpret_cast<const XV*>(x + e0 + c);
            xv[c] = t2.x;
            xv[c + 1] = t2.y;
        }
#pragma unroll
        for (int t = 0; t < kRing; ++t) {
            if (f + t >= s) break;   // uniform
            const double* at = al + ((f + t) % kRing) * lanes + lane0;
#pragma unroll
            for (int c = 0; c < V; ++c) {
                const double a = at[c];
                xv[c] = a != 0.0 ? xv[c] + a * static_cast<double>(pv[t][c]) : xv[c];
            }
        }
#pragma unroll
        for (int c = 0; c < V; c += 2) *reinterpret_cast<XV*>(x + e0 + c) = XV{xv[c], xv[c + 1]};
    }
}

// pairs of adjacent right-hand sides through buffer descriptors
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2v __attribute__((ext_vector_type(2)));
typedef float f2v __attribute__((ext_vector_type(2)));
__device__ __forceinline__ d2v bload2(__amdgpu_buffer_rsrc_t b, uint32_t off) {
    return __builtin_bit_cast(d2v, __builtin_amdgcn_raw_buffer_load_b128(b, off, 0, 0));
}
// (from FP32 as it is: converted where it is used, so that the load can stay in flight)
__device__ __forceinline__ f2v bload2f(__amdgpu_buffer_rsrc_t b, uint32_t off) {
    return __builtin_bit_cast(f2v, __builtin_amdgcn_raw_buffer_load_b64(b, off, 0, 0));
}
__device__ __forceinline__ d2v as_d2(f2v v) { return d2v{static_cast<double>(v.x), static_cast<double>(v.y)}; }
__device__ __forceinline__ d2v as_d2(d2v v) { return v; }
__device__ __forceinline__ void bstore2_nt(__amdgpu_buffer_rsrc_t b, uint32_t off, d2v v) {
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), b, off, 0, 2);
}
template <bool NT>
__device__ __forceinline__ void bstore2f(__amdgpu_buffer_rsrc_t b, uint32_t off, d2v v) {   // to FP32
    __builtin_amdgcn_raw_buffer_store_b64(
        __builtin_bit_cast(u32x2v, f2v{static_cast<float>(v.x), static_cast<float>(v.y)}), b, off, 0, NT ? 2 : 0);
}

// ------------------------------------------------ LDS-tiled finest-level kernels
// On the finest level of a Kuhn lattice with B >= 8 right-hand sides (the
// K solves) the stencil products run 2.5D-tiled: a work item is a tile of
// kTX x kTY lattice columns over a chunk of planes, and the block sweeps the
// chunk plane by plane, staging each plane of the input vector (with a one-node
// halo) and of the stored operator rows in LDS. Every input value then comes
// from global memory kTHalo / (kTX kTY) times per product (the halo) instead of
// once per row that uses it, and the gathers are LDS reads with immediate
// offsets. The work items of one XCD are contiguous bands of tiles. Byte
// offsets are 32-bit buffer offsets: loads outside the lattice return 0, stores
// there are dropped.
//
// LDS reads are what a plane costs most, so a thread owns two right-hand sides
// of one node (an operator entry is read once for both), and what it read of
// plane z + 1 for node z's upper neighbours stays in its registers for plane
// z + 1 itself and, at the lower neighbours, for plane z + 2: 7 vector values
// and 15 operator entries a node, plane and pair, where one thread a right-hand
// side read 30 (45 with w / a_jj) each. With the plane below in registers, three
// LDS slots need one barrier a plane.
constexpr int kTX = 8, kTY = 8;          // the tile: a thread for every node and pair of right-hand sides
constexpr int kTW = kTX + 2, kTHalo = (kTX + 2) * (kTY + 2);
template <int B>
struct MgTile {
    static constexpr int P = B / 2;                          // pairs per node
    static constexpr int T = kTX * kTY * P;                  // threads
    static constexpr int NS = (kTHalo * P + T - 1) / T;       // staged pairs per thread and plane
    static constexpr int NU = (kTHalo * 4 + T - 1) / T;       // 16-byte loads of operator rows per thread and plane
    static constexpr int RS = kTHalo * B, US = kTHalo * 8;    // doubles of a slot
    static constexpr int OS = kTX * kTY * B;                  // the tile's own nodes
    static constexpr size_t LDS = (size_t)(3 * (RS + US) + 2 * OS) * sizeof(double);
    static constexpr int W = B == 16 ? 4 : 3;                // waves per SIMD that the LDS admits (2, 3 blocks a CU)
};
// the 16-right-hand-side kernels that stage one right-hand side per thread
// (27-point levels)
constexpr int kTT = 512;                 // their threads, and the restriction's
constexpr int kTHX = 12, kTHY = 10;      // their halo'd tile
constexpr int kTHN = kTHX * kTHY;
constexpr int kNpf16 = (kTHN * 16 + kTT - 1) / kTT;   // input elements per thread and plane
enum TileMode { kTDirSpmv = 0, kTResidFirst = 1, kTTrue = 3, kTApply = 5, kTUpdResid = 6, kTProlongSmooth = 7 };
constexpr int kTCW = kTX / 2 + 2, kTC = kTCW * (kTY / 2 + 2);   // coarse columns under the halo'd tile

struct TileArgs {
    int32_t nx, ny, nz;
    int32_t tiles_x, tiles_y, zc, items;
    int32_t ld, col;      // `in` is [N][ld], columns col ... col + B - 1 (ld = B, col = 0 but in kTApply)
    double scale;         // kTApply: out = scale A in
    const double* U;      // [N][8] the Kuhn stencil form
    const double* in;     // the vector staged in LDS (see the modes), [N][B]
    const double* in2;    // kTDirSpmv: the old direction
    const double* b;      // right-hand side (kTResidFirst, kTProlongSmooth, kTTrue)
    const double* dinv;   // [N] (kTResidFirst, kTProlongSmooth, kTUpdResid)
    const double* w;      // the level's Jacobi weight (the same)
    const double* xc;     // kTProlongSmooth: level 1's x, on its lattice
    int32_t cx, cy, cz;
    double* out;
    double* out2;         // kTDirSpmv: the new direction
    double* parts;        // partial sums, [lanes][4][kMgBlocks]
    const MgScal* sc;     // [B]
    // kTDirSpmv with ring_n > 0: the old and new directions are the ring slots
    // of iterations slot - 1 and slot (ring_stride bytes apart)
    const int32_t* slot;
    const char* ring;
    int64_t ring_stride;
    int32_t ring_n;
};

// kTDirSpmv: the PCG direction and product, p = in - c + beta in2 (in = z,
//   in2 = the old direction) staged, out2 = p, out = A p, partial p.out.
// kTResidFirst: the V-cycle's first sweep and residual, x = w D^{-1} in
//   (in = r) staged, out = b - A x with b = r.
// kTTrue: out = b - A in for every right-hand side, partial out.out (out may
//   be null: the partial only).
// kTProlongSmooth: the V-cycle's prolongation into the finest level and its
//   last sweep, x0 = w D^{-1} in + P xc staged (in = b = r, P trilinear), out =
//   x0 + w D^{-1} (b - A x0), partial b.out. Chunks of even length: a coarse
//   plane's values wait in LDS, where each is interpolated once, for the odd
//   fine plane below it; that bilinear sum stays in registers for the even
//   plane on it. On 98 x 41 x 62 nodes with 8 right-hand sides 18.3 us (two
//   kernels: 28), on 97^3 with 16 75 (one right-hand side a thread, its rows by
//   lane broadcasts: 103), on 129^3 with 16 in mixed precision 166 (that form
//   with x0 and A x0 in FP32: 185). The sums of out and b that deflation would
//   need are not taken: K is not deflated.
// kTApply: out = scale A in for every right-hand side (any Kuhn stencil
//   form U, e.g. the derivative of K in the Jacobian product).
// kTUpdResid: the PCG update fused with kTResidFirst: r' = in - alpha in2
//   (in = r, in2 = q = A p) staged, to out2, partial r'.r',
//   and out = r' - A x with the first sweep x = w D^{-1} r' (w / a_jj from
//   LDS per neighbour). r' goes to another buffer than r: neighbouring tiles
//   still read r's halo.
// Z32: z, the V-cycle's output (kTProlongSmooth) and kTDirSpmv's `in`, is FP32
// [N][B].
// P32 (kTProlongSmooth): xc is FP32.
// P32 (kTDirSpmv): the PCG direction p is stored in FP32. The direction kernel
// rounds p before staging it, so q = A p is the FP64 product of exactly the
// stored p, and x later takes alpha times that same p: x and r stay consistent
// (r = b - A x up to FP64 rounding), and the rounding only perturbs the choice
// of the next direction.
template <int MODE, int B, bool Z32 = false, bool P32 = false>
__global__ __launch_bounds__(MgTile<B>::T, MgTile<B>::W) void k_mg_tile(TileArgs g) {
    using TL = MgTile<B>;
    constexpr int P = TL::P, T = TL::T, NS = TL::NS, NU = TL::NU, RS = TL::RS, US = TL::US;
    constexpr uint32_t SZ = sizeof(double);
    constexpr bool UPD = MODE == kTUpdResid;
    // the finest level's residual for the restriction is stored in FP32 (it only
    // feeds the coarse levels of the preconditioner)
    constexpr bool RES32 = MODE == kTResidFirst || UPD;
    constexpr bool PS = MODE == kTProlongSmooth;
    constexpr bool HAS_B = MODE != kTDirSpmv && MODE != kTApply && !UPD;
    extern __shared__ __align__(16) unsigned char mg_smem[];
    __shared__ double sm[(T / 64) * B];
    double* ring = reinterpret_cast<double*>(mg_smem);   // [3][halo node][B]
    double* ust = ring + 3 * RS;                          // [3][halo node][8]
    double* own = ust + 3 * US;                           // UPD: [2][own node][B] r' of the tile's nodes
    double* cring = own;                                  // PS: [coarse column][B] of one coarse plane
    static_assert(kTC <= 2 * kTX * kTY && kTC * P <= T, "the coarse plane's place in LDS, its loads");
    const int tid = threadIdx.x, kp = tid % P;
    constexpr bool ALL = MODE == kTTrue || MODE == kTApply;   // every right-hand side, no PCG scalars
    if constexpr (!ALL) {   // every right-hand side stopped: nothing to do
        bool any = false;
        for (int j = 0; j < B; ++j) any = any || g.sc[j].active != 0;
        if (!any) return;
    }
    // A right-hand side that stopped is carried along with p = q = 0, which leaves
    // its r as it is (the other vectors of it that are written are not read again)
    // Its scalars wait in LDS for the one use a plane: registers are what is short.
    __shared__ double lane_c[2][B];   // kTDirSpmv: c, beta; UPD: alpha
    bool on0 = true, on1 = true;
    if constexpr (MODE == kTDirSpmv || UPD) {
        on0 = g.sc[2 * kp].active != 0;
        on1 = g.sc[2 * kp + 1].active != 0;
        if (tid < B) {
            const MgScal& l = g.sc[tid];
            lane_c[0][tid] = UPD ? (l.active ? l.alpha : 0.0) : l.c;
            lane_c[1][tid] = l.beta;
        }
    }
    const int32_t nx = g.nx, ny = g.ny, nz = g.nz;
    const uint32_t nxy = static_cast<uint32_t>(nx) * ny;
    const uint32_t pv = nxy * B * SZ, pu = nxy * 8 * SZ, pd = nxy * SZ, pin = nxy * g.ld * SZ;
    const double w = (PS || MODE == kTResidFirst || UPD) ? *g.w : 0.0;
    // descriptors stay uniform over the wavefront (a per-lane size would turn
    // every access into a loop over the distinct values)
    // (the plane clamped and no branch: a step stays one basic block, so its
    // sections keep their order)
    auto plane = [&](const auto* base, int pl, uint32_t stride, uint32_t bytes) {
        return rsrc(base + (int64_t)min(max(pl, 0), nz - 1) * stride, pl >= 0 && pl < nz ? bytes : 0u);
    };
    if constexpr (MODE == kTDirSpmv) {
        if (g.ring_n > 0) {   // this iteration's slot and the one before (uniform)
            const int32_t sl = *g.slot;
            g.in2 = reinterpret_cast<const double*>(g.ring + ((sl + g.ring_n - 1) % g.ring_n) * g.ring_stride);
            g.out2 = reinterpret_cast<double*>(const_cast<char*>(g.ring + (sl % g.ring_n) * g.ring_stride));
        }
    }
    static_assert(!Z32 || MODE == kTDirSpmv || PS, "z: the direction + product and the last sweep");
    static_assert(!P32 || MODE == kTDirSpmv || PS, "FP32 direction or coarse x");
    constexpr bool ZIN = Z32 && MODE == kTDirSpmv;
    const int hc = (tid / P / kTX + 1) * kTW + tid / P % kTX + 1;   // halo node of the thread's own node
    // LDS, from the thread's node and pair: vector values, operator row
    const double* rb = ring + hc * B + 2 * kp;
    const double* ub = ust + hc * 8;
    auto val_at = [&](int sl, int d) { return *reinterpret_cast<const d2v*>(rb + sl * RS + d * B); };
    auto off_of = [](int q) constexpr { return (q >> 1) * kTW + (q & 1); };   // in-plane offset of mask q (x 1, y 2)
    std::conditional_t<ZIN, f2v, d2v> fr[NS];
    std::conditional_t<P32, f2v, d2v> f2[NS];
    std::conditional_t<P32, f2v, d2v> cv;   // PS: the thread's pair of the next coarse plane
    d2v cy[NS];   // PS: the bilinear sum of the last coarse plane at the staged nodes
    d2v fu[NU];
    double f2d[NS];   // kTResidFirst, PS, UPD: 1 / a_ii of the staged nodes
    d2v a0 = 0.0, a1 = 0.0;

    const int32_t xcd = blockIdx.x & 7, slot = blockIdx.x >> 3, per = gridDim.x >> 3;
    const int32_t wx = (g.items + 7) / 8;
    const int32_t it_end = min(g.items, (xcd + 1) * wx);
    const int32_t tiles = g.tiles_x * g.tiles_y;
    for (int32_t item = xcd * wx + slot; item < it_end; item += per) {
        const int32_t ch = item / tiles, t2 = item % tiles;
        const int32_t x0 = (t2 % g.tiles_x) * kTX, y0 = (t2 / g.tiles_x) * kTY;
        const int32_t zb = ch * g.zc, ze = min(zb + g.zc, nz);
        // node of halo node h, or -1 outside the lattice
        auto node_of = [&](int h) {
            const int gx = x0 - 1 + h % kTW, gy = y0 - 1 + h / kTW;
            return h < kTHalo && gx >= 0 && gx < nx && gy >= 0 && gy < ny ? gy * nx + gx : -1;
        };
        uint32_t fo[NS], uo[NU], oo;
#pragma unroll
        for (int u = 0; u < NS; ++u) {
            const int n = node_of((tid + u * T) / P);
            fo[u] = n >= 0 ? (static_cast<uint32_t>(n) * g.ld + g.col + 2 * kp) * SZ : kOut;
        }
#pragma unroll
        for (int v = 0; v < NU; ++v) {
            const int e = tid + v * T, n = node_of(e / 4);
            uo[v] = n >= 0 ? (static_cast<uint32_t>(n) * 8 + 2 * (e % 4)) * SZ : kOut;
        }
        {
            const int n = node_of(hc);
            oo = n >= 0 ? (static_cast<uint32_t>(n) * B + 2 * kp) * SZ : kOut;
        }
        const bool in = oo != kOut;
        // the pair's offset in an FP32 array, its node's in an [N] array (ld = B): kOut
        // stays past the end of both (kOut / 2 and kOut / B bytes are as many as a
        // plane of 2^31 bytes of pairs can have there)
        auto half = [](uint32_t o) { return o / 2; };
        auto node8 = [](uint32_t o) { return o / (B * 8) * 8; };
        // PS: coarse plane Z; the bilinear sum of the coarse plane in LDS at halo node h
        uint32_t co = kOut;
        if constexpr (PS) {
            const int X = x0 / 2 - 1 + tid / P % kTCW, Y = y0 / 2 - 1 + tid / P / kTCW;
            if (tid < kTC * P && X >= 0 && X < g.cx && Y >= 0 && Y < g.cy)
                co = (static_cast<uint32_t>(Y * g.cx + X) * B + 2 * kp) * SZ;
        }
        auto load_coarse = [&](int Z) {
            const uint32_t cxy = static_cast<uint32_t>(g.cx) * g.cy * B;
            const int64_t at = static_cast<int64_t>(min(max(Z, 0), g.cz - 1)) * cxy;
            const uint32_t n = Z >= 0 && Z < g.cz ? cxy : 0u;
            if constexpr (P32)
                cv = bload2f(rsrc(reinterpret_cast<const float*>(g.xc) + at, n * 4u), half(co));
            else
                cv = bload2(rsrc(g.xc + at, n * 8u), co);
        };
        auto put_coarse = [&] {
            if (tid < kTC * P) *reinterpret_cast<d2v*>(cring + 2 * tid) = as_d2(cv);
        };
        // x0 and y0 are even: a halo node's place among the coarse columns does not
        // depend on the tile. The weights are 1 or 1/2 an axis: with the even
        // neighbour read twice every case is a quarter of four terms.
        auto bil = [&](int u) {
            const int h = min((tid + u * T) / P, kTHalo - 1), hx = h % kTW, hy = h / kTW;
            const double* q = cring + (((hy + 1) >> 1) * kTCW + ((hx + 1) >> 1)) * B + 2 * kp;
            const int dx = hx & 1 ? 0 : B, dy = hy & 1 ? 0 : kTCW * B;
            const auto at = [&](int o) { return *reinterpret_cast<const d2v*>(q + o); };
            return 0.25 * ((at(0) + at(dx)) + (at(dy) + at(dy + dx)));
        };
        auto fetch = [&](int pl, auto EVEN) {
            if constexpr (PS && decltype(EVEN)::value) load_coarse(pl / 2 + 1);
            if constexpr (ZIN) {
                const auto bi = plane(reinterpret_cast<const float*>(g.in), pl, nxy * g.ld, pin / 2);
#pragma unroll
                for (int u = 0; u < NS; ++u) fr[u] = bload2f(bi, half(fo[u]));
            } else {
                const auto bi = plane(g.in, pl, nxy * g.ld, pin);
#pragma unroll
                for (int u = 0; u < NS; ++u) fr[u] = bload2(bi, fo[u]);
            }
            if constexpr (MODE == kTDirSpmv && P32) {   // the old direction, FP32
                const auto b2 = plane(reinterpret_cast<const float*>(g.in2), pl, nxy * B, pv / 2);
#pragma unroll
                for (int u = 0; u < NS; ++u) f2[u] = bload2f(b2, half(fo[u]));
            } else if constexpr (MODE == kTDirSpmv || UPD) {
                const auto b2 = plane(g.in2, pl, nxy * B, pv);
#pragma unroll
                for (int u = 0; u < NS; ++u) f2[u] = bload2(b2, fo[u]);
            }
            if constexpr (PS || MODE == kTResidFirst || UPD) {
                const auto bd = plane(g.dinv, pl, nxy, pd);
#pragma unroll
                for (int u = 0; u < NS; ++u) f2d[u] = bload<double>(bd, node8(fo[u]));
            }
            const auto bu = plane(g.U, pl, nxy * 8, pu);
#pragma unroll
            for (int v = 0; v < NU; ++v) fu[v] = bload2(bu, uo[v]);
        };
        d2v bn = 0.0;   // the right-hand side of the next plane
        auto loadb = [&](int z) { bn = bload2(plane(g.b, z, nxy * B, pv), oo); };
        if constexpr (HAS_B) loadb(zb);
        // PS: an odd plane reads the coarse plane above it in LDS, the even plane after
        // it puts the next one there
        auto store = [&](int sl, int pl, auto EVEN) {
            d2v lc0 = 0.0, lc1 = 0.0;
            if constexpr (MODE == kTDirSpmv || UPD) {
                lc0 = *reinterpret_cast<const d2v*>(&lane_c[0][2 * kp]);
                lc1 = *reinterpret_cast<const d2v*>(&lane_c[1][2 * kp]);
            }
#pragma unroll
            for (int u = 0; u < NS; ++u) {
                const d2v in1 = as_d2(fr[u]);
                d2v val = in1, in2 = 0.0;
                if constexpr (MODE == kTDirSpmv || UPD) in2 = as_d2(f2[u]);
                // beta = 0 (a run's first direction) never reads the old direction's values
                if constexpr (MODE == kTDirSpmv) {
                    const bool st = fo[u] != kOut;
                    val.x = st && on0 ? (lc1.x != 0.0 ? in1.x - lc0.x + lc1.x * in2.x : in1.x - lc0.x) : 0.0;
                    val.y = st && on1 ? (lc1.y != 0.0 ? in1.y - lc0.y + lc1.y * in2.y : in1.y - lc0.y) : 0.0;
                }
                if constexpr (P32 && MODE == kTDirSpmv)
                    val = d2v{static_cast<double>(static_cast<float>(val.x)), static_cast<double>(static_cast<float>(val.y))};
                if constexpr (MODE == kTResidFirst) val = w * f2d[u] * in1;
                if constexpr (PS) {
                    val = w * f2d[u] * in1;
                    if constexpr (decltype(EVEN)::value) {
                        val += cy[u];
                    } else {
                        const d2v up = bil(u);
                        val += 0.5 * (cy[u] + up);
                        cy[u] = up;
                    }
                }
                if constexpr (UPD) {   // w D^{-1} r' for the products, r' of the tile's own nodes beside it
                    const d2v rn = in1 - lc0 * in2;
                    const int h = (tid + u * T) / P, hx = h % kTW - 1, hy = h / kTW - 1;
                    if (hx >= 0 && hx < kTX && hy >= 0 && hy < kTY)
                        *reinterpret_cast<d2v*>(own + (pl & 1) * TL::OS + (hy * kTX + hx) * B + 2 * kp) = rn;
                    val = (w * f2d[u]) * rn;
                }
                if (tid + u * T < kTHalo * P) *reinterpret_cast<d2v*>(ring + sl * RS + 2 * (tid + u * T)) = val;
            }
#pragma unroll
            for (int v = 0; v < NU; ++v)
                if (tid + v * T < kTHalo * 4) *reinterpret_cast<d2v*>(ust + sl * US + 2 * (tid + v * T)) = fu[v];
            if constexpr (PS && decltype(EVEN)::value) put_coarse();
        };
        // Kept between planes: the current plane's values at the node and its three
        // upper in-plane neighbours (cur), r' there (rc), and the sum over the four
        // neighbours in the plane below (part; kTTrue: compensated, part + pcomp)
        auto own_at = [&](int pl) { return *reinterpret_cast<const d2v*>(own + (pl & 1) * TL::OS + 2 * tid); };
        d2v cur[4], part = 0.0, pcomp = 0.0, rc = 0.0;
        // the sum over the lower neighbours of the next plane's node: the values at
        // this plane's node and its three lower neighbours
        CompSum b0(0.0), b1(0.0);
        auto below_start = [&] {
            part = 0.0;
            b0 = b1 = CompSum(0.0);
        };
        auto below_term = [&](double c, d2v x) {
            if constexpr (MODE == kTTrue) {
                b0.sub(c, x.x);
                b1.sub(c, x.y);
            } else {
                part = d2v{fma(c, x.x, part.x), fma(c, x.y, part.y)};
            }
        };
        auto below_end = [&] {
            part = d2v{b0.s, b1.s};
            pcomp = d2v{b0.c, b1.c};
        };
        // plane z in slot sz, plane z + 1 in slot sp
        auto step = [&](int z, auto SZ0, auto SP0, auto EVEN) {   // EVEN: z - zb is
            constexpr int sz = decltype(SZ0)::value, sp = decltype(SP0)::value;
            store(sp, z + 1, std::integral_constant<bool, !decltype(EVEN)::value>{});
            __syncthreads();
            if (z + 1 < ze) fetch(z + 2, EVEN);
            const d2v bc = bn;   // loaded one step earlier
            if constexpr (HAS_B) {
                if (z + 1 < ze) loadb(z + 1);
            }
            double dc = 0.0;
            if constexpr (PS) dc = bload<double>(plane(g.dinv, z, nxy, pd), node8(oo));
            const d2v xc = cur[0];
            d2v sum = part;
            CompSum c0(0.0), c1(0.0);
            if constexpr (MODE == kTTrue) {
                c0.s = part.x;
                c0.c = pcomp.x;
                c1.s = part.y;
                c1.c = pcomp.y;
            }
            auto term = [&](double c, d2v x) {
                if constexpr (MODE == kTTrue) {
                    c0.sub(c, x.x);
                    c1.sub(c, x.y);
                } else {
                    sum = d2v{fma(c, x.x, sum.x), fma(c, x.y, sum.y)};
                }
            };
            const auto row = [&](int q) { return *reinterpret_cast<const d2v*>(ub + sz * US + 2 * q); };
            // The stencil form's entry of offset mask m is m. The sections' operands
            // are not live together (128 registers).
            {   // this plane, upper half
                const d2v u01 = row(0), u23 = row(1);
                const double um[4] = {u01.x, u01.y, u23.x, u23.y};
#pragma unroll
                for (int q = 0; q < 4; ++q) term(um[q], cur[q]);
            }
            __builtin_amdgcn_sched_barrier(0);
            // this plane, lower half, and the next plane's sum over it
            below_start();
            below_term(ub[sz * US + 4], xc);
#pragma unroll
            for (int q = 1; q < 4; ++q) {
                const d2v lo = val_at(sz, -off_of(q));
                term(ub[sz * US - off_of(q) * 8 + q], lo);
                below_term(ub[sz * US - off_of(q) * 8 + 4 + q], lo);
            }
            if constexpr (MODE == kTTrue) below_end();
            __builtin_amdgcn_sched_barrier(0);
            const d2v rz = rc;
            if constexpr (UPD) rc = own_at(z + 1);   // read in the step that staged it: two slots do
            {   // the plane above
                const d2v u45 = row(2), u67 = row(3);
                const double um[4] = {u45.x, u45.y, u67.x, u67.y};
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    cur[q] = val_at(sp, off_of(q));
                    term(um[q], cur[q]);
                }
            }
            d2v rtrue = 0.0;
            if constexpr (MODE == kTTrue) {
                c0.add(bc.x);
                c1.add(bc.y);
                rtrue = d2v{c0.value(), c1.value()};
            }
            // RES32: float [N][B] planes; kTTrue with out = null: only the partial out.out
            const auto bo = RES32 || (PS && Z32)
                                  ? rsrc(reinterpret_cast<const float*>(g.out) + (int64_t)z * nxy * B, pv / 2)
                                  : plane(g.out, z, nxy * B, g.out ? pv : 0u);
            const d2v zero = 0.0;
            d2v o;
            if constexpr (MODE == kTDirSpmv) {
                o = sum;
                a0 += in ? xc * sum : zero;
                if constexpr (P32)   // xc is already an FP32 value
                    bstore2f<true>(plane(reinterpret_cast<const float*>(g.out2), z, nxy * B, pv / 2), half(oo), xc);
                else
                    bstore2_nt(plane(g.out2, z, nxy * B, pv), oo, xc);   // p: next read by the next iteration
            } else if constexpr (MODE == kTApply) {
                o = g.scale * sum;
            } else if constexpr (UPD) {
                o = rz - sum;
                a1 += in ? rz * rz : zero;
                bstore2_nt(plane(g.out2, z, nxy * B, pv), oo, rz);
            } else if constexpr (PS) {
                o = xc + w * dc * (bc - sum);
                if constexpr (Z32) o = d2v{held_as<float>(o.x), held_as<float>(o.y)};
                a0 += in ? bc * o : zero;
            } else {
                o = MODE == kTTrue ? rtrue : bc - sum;
                if constexpr (MODE == kTTrue) a1 += in ? o * o : zero;
            }
            if constexpr (RES32)
                bstore2f<false>(bo, half(oo), o);   // read next
            else if constexpr (PS && Z32)
                bstore2f<true>(bo, half(oo), o);
            else
                bstore2_nt(bo, oo, o);
        };
        using Even = std::true_type;
        using Odd = std::false_type;
        __syncthreads();   // the last planes of the item before are read
        if constexpr (PS) {   // zb is even: plane zb - 1 lies between coarse planes zb / 2 - 1 and zb / 2
            load_coarse(zb / 2 - 1);
            put_coarse();
            load_coarse(zb / 2);
            __syncthreads();
#pragma unroll
            for (int u = 0; u < NS; ++u) cy[u] = bil(u);
            __syncthreads();
            put_coarse();
        }
        fetch(zb - 1, Odd{});
        if constexpr (PS) __syncthreads();
        store(0, zb - 1, Odd{});
        fetch(zb, Even{});
        if constexpr (PS) __syncthreads();
        store(1, zb, Even{});
        fetch(zb + 1, Odd{});
        __syncthreads();
        if constexpr (UPD) rc = own_at(zb);
        below_start();
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            below_term(ub[-off_of(q) * 8 + 4 + q], val_at(0, -off_of(q)));
            cur[q] = val_at(1, off_of(q));
        }
        if constexpr (MODE == kTTrue) below_end();
        // plane z - zb + 1 lives in slot (z - zb + 1) % 3. A wavefront at most one
        // barrier ahead writes plane z + 2 over plane z - 1, which no step reads
        using I0 = std::integral_constant<int, 0>;
        using I1 = std::integral_constant<int, 1>;
        using I2 = std::integral_constant<int, 2>;
        if constexpr (PS) {   // six steps: the parities too are known at compile time
            for (int z = zb; z < ze; z += 6) {
                step(z, I1{}, I2{}, Even{});
                if (z + 1 < ze) step(z + 1, I2{}, I0{}, Odd{});
                if (z + 2 < ze) step(z + 2, I0{}, I1{}, Even{});
                if (z + 3 < ze) step(z + 3, I1{}, I2{}, Odd{});
                if (z + 4 < ze) step(z + 4, I2{}, I0{}, Even{});
                if (z + 5 < ze) step(z + 5, I0{}, I1{}, Odd{});
            }
        } else {
            for (int z = zb; z < ze; z += 3) {
                step(z, I1{}, I2{}, Even{});
                if (z + 1 < ze) step(z + 1, I2{}, I0{}, Even{});
                if (z + 2 < ze) step(z + 2, I0{}, I1{}, Even{});
            }
        }
    }
    auto out_sum = [&](d2v v, int slot_) {
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            double t = comp(v, c);
#pragma unroll
            for (int off = 32; off >= P; off >>= 1) t += __shfl_xor(t, off);
            if ((tid & 63) < P) sm[(tid >> 6) * B + 2 * kp + c] = t;
        }
        __syncthreads();
        if (tid < B) {
            double t = 0.0;
            for (int wv = 0; wv < T / 64; ++wv) t += sm[wv * B + tid];
            put(g.parts, tid, slot_, t);
        }
        __syncthreads();
    };
    if constexpr (MODE == kTDirSpmv || PS) out_sum(a0, 0);
    if constexpr (MODE == kTTrue || UPD) out_sum(a1, 1);
}

// ------------------------------------------------ LDS-tiled restriction
// Finest to first coarse level of the K hierarchy (trilinear weights, B >= 8
// right-hand sides): a work item is a tile of kRX x RY coarse columns over a
// chunk of coarse planes. The block stages each fine plane of the tile's
// support, (2 kRX + 1) x (2 RY + 1) nodes, in LDS with row-contiguous loads
// (double-buffered: the next plane's loads are in flight during the sums)
// and forms the in-plane 3 x 3 weighted sums from LDS; the weights along z
// (1/2 for planes 2K - 1 and 2K + 1, 1 for 2K) are applied as the planes
// stream by, so a fine plane is read once per chunk, the chunk's first plane
// twice. Fine nodes off the lattice load as 0 (their weight is 0).
constexpr int kRX = 8;
template <int B>
struct MgRst {
    static constexpr int RY = kTT / B / kRX;                  // coarse rows per tile (one coarse node per B threads)
    static constexpr int FX = 2 * kRX + 1, FY = 2 * RY + 1;   // fine support of the tile
    static constexpr int NPF = (FX * FY * B + kTT - 1) / kTT;  // fine values per thread and plane
    static constexpr size_t LDS = (size_t)2 * NPF * kTT * sizeof(double);
};

struct RstArgs {
    int32_t nx, ny, nz;      // fine lattice
    int32_t cx, cy, cz;      // coarse lattice
    int32_t tiles_x, tiles_y, zc, items;
    const void* r;           // fine residual [Nf][B], FP64 or (R32) FP32
    const double* dinv;      // coarse 1 / a_ii [Nc]
    const double* w;         // coarse level's Jacobi weight
    double* bc;              // coarse right-hand side [Nc][B]
    double* xc;              // coarse first sweep w D^{-1} bc [Nc][B]
    const MgScal* sc;        // [B]
};

template <int B, bool R32, bool O32 = false>
__global__ __launch_bounds__(kTT) void k_mg_restrict_tile(RstArgs g) {
    using TR = MgRst<B>;
    constexpr int RY = TR::RY, FX = TR::FX, FY = TR::FY, NPF = TR::NPF, RS = NPF * kTT;
    constexpr uint32_t SZ = sizeof(double);
    extern __shared__ __align__(16) unsigned char mg_smem[];
    double* buf = reinterpret_cast<double*>(mg_smem);   // [2][RS]: [support node][B]
    const int tid = threadIdx.x, k = tid % B, cn = tid / B;
    bool any = false;
    for (int j = 0; j < B; ++j) any = any || g.sc[j].active != 0;
    if (!any) return;   // every right-hand side stopped
    const bool act = g.sc[k].active != 0;
    const int32_t nx = g.nx, ny = g.ny, nz = g.nz;
    constexpr uint32_t RZ = R32 ? 4 : 8;   // bytes per fine value
    const uint32_t nxy = static_cast<uint32_t>(nx) * ny, pv = nxy * B * RZ;
    const int64_t cxy = (int64_t)g.cx * g.cy;
    const double wc = *g.w;   // system 0 of the coarse level (the caller passes that entry)
    const int lx = cn % kRX, ly = cn / kRX;
    const int c0 = ((2 * ly + 1) * FX + 2 * lx + 1) * B + k;   // LDS index of the node's centre fine node

    const int32_t xcd = blockIdx.x & 7, slot = blockIdx.x >> 3, per = gridDim.x >> 3;
    const int32_t wx = (g.items + 7) / 8;
    const int32_t it_end = min(g.items, (xcd + 1) * wx);
    const int32_t tiles = g.tiles_x * g.tiles_y;
    double fr[NPF];
    for (int32_t item = xcd * wx + slot; item < it_end; item += per) {
        const int32_t ch = item / tiles, t2 = item % tiles;
        const int32_t X0 = (t2 % g.tiles_x) * kRX, Y0 = (t2 / g.tiles_x) * RY;
        const int32_t Kb = ch * g.zc, Ke = min(Kb + g.zc, g.cz);
        uint32_t fo[NPF];
#pragma unroll
        for (int u = 0; u < NPF; ++u) {
            const int e = tid + u * kTT, nl = e / B;
            const int gx = 2 * X0 - 1 + nl % FX, gy = 2 * Y0 - 1 + nl / FX;
            const bool in = nl < FX * FY && gx >= 0 && gx < nx && gy >= 0 && gy < ny;
            fo[u] = in ? (static_cast<uint32_t>(gy * nx + gx) * B + e % B) * RZ : kOut;
        }
        auto fetch = [&](int pl) {
            const bool in = pl >= 0 && pl < nz;
            const auto br = rsrc(static_cast<const char*>(g.r) + (in ? (int64_t)pl * pv : 0), in ? pv : 0u);
#pragma unroll
            for (int u = 0; u < NPF; ++u) {
                if constexpr (R32)
                    fr[u] = static_cast<double>(bload<float>(br, fo[u]));
                else
                    fr[u] = bload<double>(br, fo[u]);
            }
        };
        auto store = [&](int sl) {
#pragma unroll
            for (int u = 0; u < NPF; ++u) buf[sl * RS + tid + u * kTT] = fr[u];
        };
        auto psum = [&](int sl) {   // in-plane weights 1/2, 1, 1/2 along x and y
            const double* f = buf + sl * RS + c0;
            double rows[3];
#pragma unroll
            for (int dy = -1; dy <= 1; ++dy) {
                const double* q = f + dy * FX * B;
                rows[dy + 1] = 0.5 * (q[-B] + q[B]) + q[0];
            }
            return 0.5 * (rows[0] + rows[2]) + rows[1];
        };
        const int32_t Ix = X0 + lx, Iy = Y0 + ly;
        const bool own = act && Ix < g.cx && Iy < g.cy;
        const int p0 = 2 * Kb - 1, p1 = 2 * Ke - 1;
        fetch(p0);
        store(0);
        double acc = 0.0;
        for (int p = p0; p <= p1; ++p) {
            __syncthreads();
            if (p < p1) fetch(p + 1);
            const double s = psum((p - p0) & 1);
            if (((p - p0) & 1) == 0) {   // odd plane p = 2K - 1 or 2K + 1
                if (p > p0) {            // closes coarse plane K = (p - 1) / 2
                    const double v = acc + 0.5 * s;
                    if (own) {
                        const int64_t I = (int64_t)((p - 1) / 2) * cxy + (int64_t)Iy * g.cx + Ix;
                        if constexpr (O32) {   // the coarse level's vectors in FP32
                            reinterpret_cast<float*>(g.bc)[I * B + k] = static_cast<float>(v);
                            reinterpret_cast<float*>(g.xc)[I * B + k] = static_cast<float>(wc * g.dinv[I] * v);
                        } else {
                            g.bc[I * B + k] = v;
                            g.xc[I * B + k] = wc * g.dinv[I] * v;
                        }
                    }
                }
                acc = 0.5 * s;
            } else {
                acc += s;
            }
            if (p < p1) store((p + 1 - p0) & 1);
        }
        __syncthreads();   // the next item's first store overwrites slot 0
    }
}

// ------------------------------------------------ LDS-tiled 27-point kernels
// The first coarse level of the K hierarchy with 16 right-hand sides: the
// same 2.5D tiling as the finest level (the input vector's planes in LDS),
// with the Galerkin operator's 27-point rows stored whole (FP32, 32 a node:
// diagonal, 13 upper, 13 lower entries, zero where the partner is off the
// lattice, padding). The 16 lanes of a node load its row as two 128-byte
// lines, lane k holding entries k and 16 + k, and every entry reaches the
// row's lanes by a DPP row broadcast, so the operator never passes through
// LDS and the partner rows are never gathered.
constexpr int64_t kTile27Min = 16384;   // smaller levels keep the walk kernels (launch-bound anyway)
constexpr int64_t kRow27Min = 131072;   // M_delta: whole 27-point rows pay off from about this size on
enum Tile27Mode { kT27Resid = 0, kT27Smooth = 1 };

// whole 27-point rows from the stored half (diagonal, 13 upper, 13 lower
// entries; zero where the partner is off the lattice), entry e of node i
__device__ __forceinline__ double row27(const LvArgs& L, const double* __restrict__ U, int64_t i, int ix, int iy, int iz,
                                        int e) {
    if (e == 0) return U[i * 14];
    if (e > 26) return 0.0;
    const int j = e < 14 ? e - 1 : e - 14, sg = e < 14 ? 1 : -1, code = 14 + j;
    const int dx = sg * (code % 3 - 1), dy = sg * ((code / 3) % 3 - 1), dz = sg * (code / 9 - 1);
    const bool in = ix + dx >= 0 && ix + dx < L.nx && iy + dy >= 0 && iy + dy < L.ny && iz + dz >= 0 && iz + dz < L.nz;
    const int64_t r = e < 14 ? i : i + dx + (int64_t)L.nx * (dy + (int64_t)L.ny * dz);
    return in ? U[r * 14 + 1 + j] : 0.0;
}

// entry-major [27][N] per system (the one-right-hand-side walk kernels, row kind 4)
__global__ __launch_bounds__(kMgT) void k_mg_fullrows27(LvArgs L, double* __restrict__ Uf) {
    const int sys = blockIdx.y;
    const double* U = L.U + (int64_t)sys * L.N * 14;
    double* F = Uf + (int64_t)sys * L.N * 27;
    for (int64_t i = blockIdx.x * (int64_t)kMgT + threadIdx.x; i < L.N; i += (int64_t)gridDim.x * kMgT) {
        int ix, iy, iz;
        coords(static_cast<int32_t>(i), L.nx, L.ny, ix, iy, iz);
#pragma unroll
        for (int e = 0; e < 27; ++e) F[e * L.N + i] = row27(L, U, i, ix, iy, iz, e);
    }
}

// node-major [N][16] FP32 pairs (entry k, entry k + 16): the tiled kernels; 16
// threads a node (49^3 nodes 13 us; by way of FP64 rows, a thread a node, 75)
__global__ __launch_bounds__(kMgT) void k_mg_pairs27(LvArgs L, float* __restrict__ P) {
    for (int64_t t = blockIdx.x * (int64_t)kMgT + threadIdx.x; t < L.N * 16; t += (int64_t)gridDim.x * kMgT) {
        const int64_t i = t / 16;
        const int k = static_cast<int>(t % 16);
        int ix, iy, iz;
        coords(static_cast<int32_t>(i), L.nx, L.ny, ix, iy, iz);
        *reinterpret_cast<float2*>(P + 2 * t) = make_float2(static_cast<float>(row27(L, L.U, i, ix, iy, iz, k)),
                                                            static_cast<float>(row27(L, L.U, i, ix, iy, iz, k + 16)));
    }
}

// lane J of each 16-lane row, to the whole row
template <int J>
__device__ __forceinline__ double row_bcast(double v) {
    // one 64-bit DPP move (row_newbcast takes 64-bit operands); every lane is
    // written (row broadcast, full masks), so the old value is never used
    return __builtin_amdgcn_update_dpp(0.0, v, 0x150 + J, 0xF, 0xF, true);
}

// two FP32 row entries stored side by side, loaded as one 64-bit value, so that
// one 64-bit DPP row broadcast delivers both
__device__ __forceinline__ float pair_lo(double p) {
    return __builtin_bit_cast(float, static_cast<uint32_t>(__builtin_bit_cast(uint64_t, p)));
}
__device__ __forceinline__ float pair_hi(double p) {
    return __builtin_bit_cast(float, static_cast<uint32_t>(__builtin_bit_cast(uint64_t, p) >> 32));
}

// sum over the row's entries held as FP32 pairs: pair k = (entry k, entry k + 16),
// 16 broadcasts for the 27 entries, the products in FP64
template <int... K>
__device__ __forceinline__ void bcast16(double pr, double (&bc)[16], std::integer_sequence<int, K...>) {
    ((bc[K] = row_bcast<K>(pr)), ...);
}
template <int J>
__device__ __forceinline__ double pair27p(double s, const double (&bc)[16], const double* rb, int sz, int sp, int sl) {
    constexpr int code = 14 + J;
    constexpr int dx = code % 3 - 1, dy = (code / 3) % 3 - 1, dz = code / 9 - 1;
    constexpr int d = (dy * kTHX + dx) * 16;
    const int up = dz ? sp : sz, lo = dz ? sl : sz;
    const double cu = static_cast<double>(pair_lo(bc[1 + J]));
    double cl;
    if constexpr (14 + J < 16)
        cl = static_cast<double>(pair_lo(bc[14 + J]));
    else
        cl = static_cast<double>(pair_hi(bc[J - 2]));
    return fma(cl, rb[lo - d], fma(cu, rb[up + d], s));
}
template <int... J>
__device__ __forceinline__ double apply27p(double pr, const double* rb, int sz, int sp, int sl,
                                           std::integer_sequence<int, J...>) {
    double bc[16];
    bcast16(pr, bc, std::make_integer_sequence<int, 16>{});
    double s = static_cast<double>(pair_lo(bc[0])) * rb[sz];
    ((s = pair27p<J>(s, bc, rb, sz, sp, sl)), ...);
    return s;
}

struct Tile27Args {
    int32_t nx, ny, nz;
    int32_t tiles_x, tiles_y, zc, items;
    const float* Uf27p;   // the rows as [N][16] FP32 pairs
    const double* x;      // staged vector [N][16]
    const double* b;      // [N][16]
    const double* dinv;   // [N] (kT27Smooth)
    const double* w;      // the level's Jacobi weight (kT27Smooth)
    double* out;          // kT27Resid: b - A x; kT27Smooth: x + w D^{-1} (b - A x)
    const MgScal* sc;     // [16]
};

template <int MODE, bool V32 = false>
__global__ __launch_bounds__(kTT, 4) void k_mg_tile27(Tile27Args g) {
    constexpr int B = 16;
    constexpr int NPF = kNpf16, RS = NPF * kTT;
    constexpr int TX = kTHX - 2, TY = kTHY - 2;
    constexpr int NO = (TX * TY * B + kTT - 1) / kTT;   // output slots per thread
    constexpr uint32_t SZ = sizeof(double);
    extern __shared__ __align__(16) unsigned char mg_smem[];
    double* ring = reinterpret_cast<double*>(mg_smem);   // [3][RS]: [halo node][B]
    const int tid = threadIdx.x, k = tid % B;
    bool any = false;
    for (int j = 0; j < B; ++j) any = any || g.sc[j].active != 0;
    if (!any) return;   // every right-hand side stopped
    const bool act = g.sc[k].active != 0;
    const int32_t nx = g.nx, ny = g.ny, nz = g.nz;
    const uint32_t nxy = static_cast<uint32_t>(nx) * ny;
    const uint32_t pv = nxy * B * SZ, pd = nxy * SZ;
    const double w = MODE == kT27Smooth ? *g.w : 0.0;
    auto plane = [&](const double* base, int pl, uint32_t stride, uint32_t bytes) {
        const bool in = pl >= 0 && pl < nz;
        return rsrc(base + (in ? (int64_t)pl * stride : 0), in ? bytes : 0u);
    };
    // x, b and out of the level: V32 keeps them in FP32 (offsets halve)
    auto vplane = [&](const double* base, int pl) {
        if constexpr (V32) {
            const bool in = pl >= 0 && pl < nz;
            return rsrc(reinterpret_cast<const float*>(base) + (in ? (int64_t)pl * nxy * B : 0), in ? pv / 2 : 0u);
        } else {
            return plane(base, pl, nxy * B, pv);
        }
    };
    auto vload = [&](__amdgpu_buffer_rsrc_t br, uint32_t o) -> double {
        if constexpr (V32)
            return static_cast<double>(bload<float>(br, o == kOut ? kOut : o / 2));
        else
            return bload<double>(br, o);
    };
    int32_t oc[NO];
#pragma unroll
    for (int u = 0; u < NO; ++u) {
        const int nl = (tid + u * kTT) / B;
        oc[u] = nl < TX * TY ? (nl / TX + 1) * kTHX + nl % TX + 1 : kTHX + 1;
    }
    double fr[NPF];
    const int32_t xcd = blockIdx.x & 7, slot = blockIdx.x >> 3, per = gridDim.x >> 3;
    const int32_t wx = (g.items + 7) / 8;
    const int32_t it_end = min(g.items, (xcd + 1) * wx);
    const int32_t tiles = g.tiles_x * g.tiles_y;
    for (int32_t item = xcd * wx + slot; item < it_end; item += per) {
        const int32_t ch = item / tiles, t2 = item % tiles;
        const int32_t x0 = (t2 % g.tiles_x) * TX, y0 = (t2 / g.tiles_x) * TY;
        const int32_t zb = ch * g.zc, ze = min(zb + g.zc, nz);
        uint32_t fo[NPF], oo[NO], od[NO];
#pragma unroll
        for (int u = 0; u < NPF; ++u) {
            const int nl = (tid + u * kTT) / B;
            const int gx = x0 - 1 + nl % kTHX, gy = y0 - 1 + nl / kTHX;
            const bool fin = nl < kTHN && gx >= 0 && gx < nx && gy >= 0 && gy < ny;
            fo[u] = fin ? (static_cast<uint32_t>(gy * nx + gx) * B + k) * SZ : kOut;
        }
#pragma unroll
        for (int u = 0; u < NO; ++u) {
            const int nl = (tid + u * kTT) / B;
            const int ox = x0 + nl % TX, oy = y0 + nl / TX;
            const bool oin = nl < TX * TY && ox < nx && oy < ny;
            oo[u] = oin ? (static_cast<uint32_t>(oy * nx + ox) * B + k) * SZ : kOut;
            od[u] = oin ? static_cast<uint32_t>(oy * nx + ox) * SZ : kOut;
        }
        auto fetch = [&](int pl) {
            const auto bx = vplane(g.x, pl);
#pragma unroll
            for (int u = 0; u < NPF; ++u) fr[u] = vload(bx, fo[u]);
        };
        auto store = [&](int sl) {
#pragma unroll
            for (int u = 0; u < NPF; ++u) ring[sl * RS + tid + u * kTT] = fr[u];
        };
        // the operator rows and b of plane z, loaded a plane ahead
        double ua[NO], bn[NO];
        auto load_node = [&](int z) {
            const auto bb = vplane(g.b, z);
            // the pair (entry k, entry k + 16) as 8 bytes: the layout of a [N][16] vector
            const auto bq = plane(reinterpret_cast<const double*>(g.Uf27p), z, nxy * B, pv);
#pragma unroll
            for (int u = 0; u < NO; ++u) {
                ua[u] = bload<double>(bq, oo[u]);
                bn[u] = vload(bb, oo[u]);
            }
        };
        load_node(zb);
        auto step = [&](int z, auto SZ0, auto SP0, auto SL0) {
            constexpr int sz = decltype(SZ0)::value, sp = decltype(SP0)::value, sl = decltype(SL0)::value;
            store(sp);
            __syncthreads();
            if (z + 1 < ze) fetch(z + 2);
            double ca[NO], bc[NO], dc[NO];
#pragma unroll
            for (int u = 0; u < NO; ++u) {
                ca[u] = ua[u];
                bc[u] = bn[u];
            }
            if (z + 1 < ze) load_node(z + 1);
            if constexpr (MODE == kT27Smooth) {   // 1 / a_ii of this plane (one value per node)
                const auto bd = plane(g.dinv, z, nxy, pd);
#pragma unroll
                for (int u = 0; u < NO; ++u) dc[u] = bload<double>(bd, od[u]);
            }
            const auto bo = vplane(g.out, z);   // uniform descriptor; stopped lanes store nowhere
#pragma unroll
            for (int u = 0; u < NO; ++u) {
                if (tid + u * kTT >= TX * TY * B) continue;   // whole waves past the tile skip
                const double* rb = ring + oc[u] * B + k;
                const double ax = apply27p(ca[u], rb, sz * RS, sp * RS, sl * RS, std::make_integer_sequence<int, 13>{});
                double o = bc[u] - ax;
                if constexpr (MODE == kT27Smooth) o = rb[sz * RS] + w * dc[u] * o;
                if constexpr (V32)
                    bstore<float>(bo, act && oo[u] != kOut ? oo[u] / 2 : kOut, static_cast<float>(o));
                else
                    bstore<double>(bo, act ? oo[u] : kOut, o);
            }
            __syncthreads();
        };
        fetch(zb - 1);
        store(0);
        fetch(zb);
        store(1);
        fetch(zb + 1);
        using I0 = std::integral_constant<int, 0>;
        using I1 = std::integral_constant<int, 1>;
        using I2 = std::integral_constant<int, 2>;
        for (int z = zb; z < ze; z += 3) {   // plane z - zb + 1 lives in slot (z - zb + 1) % 3
            step(z, I1{}, I2{}, I0{});
            if (z + 1 < ze) step(z + 1, I2{}, I0{}, I1{});
            if (z + 2 < ze) step(z + 2, I0{}, I1{}, I2{});
        }
    }
}

inline LvArgs lv_args(const MgLevel& L) {
    LvArgs a;
    a.U = L.U;
    a.tab = L.tab;
    a.m = L.m;
    a.nx = L.nx;
    a.ny = L.ny;
    a.nz = L.nz;
    a.N = L.N;
    a.kind = L.kind;
    a.Uf = L.Uf;
    a.Uf32 = L.Uf32;
    return a;
}

// a multiple of 8 blocks (the XCD row split), at most cap (<= kMgBlocks)
inline dim3 vgrid(int64_t n, int cap = kMgGrid) { return dim3((grid_for(n, kMgT, cap) + 7) & ~7); }

#define QPAT_MG_KIND(kind, B, KERNEL, ...)                                 \
    switch (kind) {                                                         \
        case 1: hipLaunchKernelGGL((KERNEL<1, B>), __VA_ARGS__); break;     \
        case 2: hipLaunchKernelGGL((KERNEL<2, B>), __VA_ARGS__); break;     \
        case 3: hipLaunchKernelGGL((KERNEL<3, B>), __VA_ARGS__); break;     \
        case 4:                                                             \
            if constexpr (B == 1) hipLaunchKernelGGL((KERNEL<4, 1>), __VA_ARGS__); \
            break;                                                          \
        case 5:                                                             \
            if constexpr (B == 1) hipLaunchKernelGGL((KERNEL<5, 1>), __VA_ARGS__); \
            break;                                                          \
        case 6:                                                             \
            if constexpr (B == 1) hipLaunchKernelGGL((KERNEL<6, 1>), __VA_ARGS__); \
            break;                                                          \
        default: hipLaunchKernelGGL((KERNEL<0, B>), __VA_ARGS__); break;    \
    }

// Dense inverse of an SPD matrix (Cholesky), in place; false if not positive definite.
bool spd_inverse(std::vector<double>& A, int n) {
    std::vector<double> L(A);
    for (int j = 0; j < n; ++j) {
        double d = L[(size_t)j * n + j];
        for (int k = 0; k < j; ++k) d -= L[(size_t)j * n + k] * L[(size_t)j * n + k];
        if (!(d > 0.0)) return false;
        d = std::sqrt(d);
        L[(size_t)j * n + j] = d;
        for (int i = j + 1; i < n; ++i) {
            double s = L[(size_t)i * n + j];
            for (int k = 0; k < j; ++k) s -= L[(size_t)i * n + k] * L[(size_t)j * n + k];
            L[(size_t)i * n + j] = s / d;
        }
    }
    // columns of the inverse: solve L L^T x = e_c
    std::vector<double> y(n);
    for (int col = 0; col < n; ++col) {
        for (int i = 0; i < n; ++i) {
            double s = i == col ? 1.0 : 0.0;
            for (int k = 0; k < i; ++k) s -= L[(size_t)i * n + k] * y[k];
            y[i] = s / L[(size_t)i * n + i];
        }
        for (int i = n - 1; i >= 0; --i) {
            double s = y[i];
            for (int k = i + 1; k < n; ++k) s -= L[(size_t)k * n + i] * y[k];
            y[i] = s / L[(size_t)i * n + i];
        }
        for (int i = 0; i < n; ++i) A[(size_t)i * n + col] = y[i];
    }
    // the columns carry independent rounding: make the inverse exactly
    // symmetric, as the preconditioner it is part of must be
    for (int i = 0; i < n; ++i)
        for (int j = i + 1; j < n; ++j) {
            const double v = 0.5 * (A[(size_t)i * n + j] + A[(size_t)j * n + i]);
            A[(size_t)i * n + j] = A[(size_t)j * n + i] = v;
        }
    return true;
}

template <int B, bool DOTS>
void launch_smooth(int kind, dim3 g, hipStream_t st, const SmArgs& a, const double* b, const double* x, double* y,
                   double* parts) {
    switch (kind) {
        case 1: hipLaunchKernelGGL((k_mg_smooth<1, B, DOTS>), g, dim3(kMgT), 0, st, a, b, x, y, parts); break;
        case 2: hipLaunchKernelGGL((k_mg_smooth<2, B, DOTS>), g, dim3(kMgT), 0, st, a, b, x, y, parts); break;
        case 3: hipLaunchKernelGGL((k_mg_smooth<3, B, DOTS>), g, dim3(kMgT), 0, st, a, b, x, y, parts); break;
        case 4:
            if constexpr (B == 1) hipLaunchKernelGGL((k_mg_smooth<4, 1, DOTS>), g, dim3(kMgT), 0, st, a, b, x, y, parts);
            break;
        case 5:
            if constexpr (B == 1) hipLaunchKernelGGL((k_mg_smooth<5, 1, DOTS>), g, dim3(kMgT), 0, st, a, b, x, y, parts);
            break;
        case 6:
            if constexpr (B == 1) hipLaunchKernelGGL((k_mg_smooth<6, 1, DOTS>), g, dim3(kMgT), 0, st, a, b, x, y, parts);
            break;
        default: hipLaunchKernelGGL((k_mg_smooth<0, B, DOTS>), g, dim3(kMgT), 0, st, a, b, x, y, parts); break;
    }
}

// one grid row per system (blockIdx.y) for one right-hand side per thread: the
// systems' sweeps then run side by side instead of one after the other in
// each block (the one-right-hand-side kernels are latency-bound)
inline dim3 sys_rows(dim3 g, int B, int nsys) { return dim3(g.x, B == 1 ? nsys : 1); }

// grid of the stencil and V-cycle kernels of a level with n nodes
template <int B>
dim3 sgrid(int64_t n, int nsys = 1) {
    // one right-hand side per thread (the M_delta solves) is latency-bound: more blocks
    return sys_rows(vgrid(n * Pk<B>::BV, B == 1 ? kMgBlocks : kMgGrid), B, nsys);
}

// the direction ring of the tiled iterations, as the direction kernel reads it
struct RingArg {
    const int32_t* slot = nullptr;
    const char* base = nullptr;
    int64_t stride = 0;
    int32_t n = 0;
};

template <int MODE, int B, bool Z32 = false, bool P32 = false>
void launch_tile(const MgState& M, const TileGeo& t, hipStream_t st, const double* in, const double* in2,
                 const double* b, double* out, double* out2, RingArg ring = {}) {
    if constexpr (B >= 8) {   // tile_setup turns the tiling on only there
        const MgLevel& L = M.lv[0];
        TileArgs g{};
        g.nx = L.nx;
        g.ny = L.ny;
        g.nz = L.nz;
        g.tiles_x = t.tiles_x;
        g.tiles_y = t.tiles_y;
        g.zc = t.zc;
        g.items = t.items;
        g.ld = B;
        g.col = 0;
        g.scale = 1.0;
        g.U = L.U;
        g.in = in;
        g.in2 = in2;
        g.b = b;
        g.dinv = L.dinv;
        g.w = M.w;   // system 0, level 0
        g.out = out;
        g.out2 = out2;
        g.parts = M.parts;
        g.sc = M.sc;
        g.slot = ring.slot;
        g.ring = ring.base;
        g.ring_stride = ring.stride;
        g.ring_n = ring.n;
        hipLaunchKernelGGL((k_mg_tile<MODE, B, Z32, P32>), dim3(t.blocks), dim3(MgTile<B>::T), MgTile<B>::LDS, st, g);
    }
}

template <int B>
TileArgs ps_args(const MgState& M, const TileGeo& t, const double* r, const double* x1, double* z) {
    const MgLevel& L = M.lv[0];
    const MgLevel& C = M.lv[1];
    TileArgs g{};
    g.nx = L.nx;
    g.ny = L.ny;
    g.nz = L.nz;
    g.tiles_x = t.tiles_x;
    g.tiles_y = t.tiles_y;
    g.zc = t.ps_zc;
    g.items = t.ps_items;
    g.ld = B;
    g.U = L.U;
    g.in = r;
    g.b = r;
    g.dinv = L.dinv;
    g.w = M.w;   // system 0, level 0
    g.xc = x1;
    g.cx = C.nx;
    g.cy = C.ny;
    g.cz = C.nz;
    g.out = z;
    g.parts = M.parts;
    g.sc = M.sc;
    return g;
}

// coarse level l: out = b - A x (kT27Resid) or x + w D^{-1} (b - A x) (kT27Smooth)
template <int MODE>
void launch_tile27(const MgState& M, const TileGeo& t, int l, hipStream_t st, const double* x, const double* b,
                   double* out, bool v32 = false) {
    const MgLevel& L = M.lv[l];
    const TileGeo::Lv27& q = t.t27[l];
    Tile27Args g;
    g.nx = L.nx;
    g.ny = L.ny;
    g.nz = L.nz;
    g.tiles_x = q.tx;
    g.tiles_y = q.ty;
    g.zc = q.zc;
    g.items = q.items;
    g.Uf27p = L.Uf27p;
    g.x = x;
    g.b = b;
    g.dinv = L.dinv;
    g.w = M.w + l;   // system 0, level l
    g.out = out;
    g.sc = M.sc;
    const size_t lds = (size_t)3 * kNpf16 * kTT * sizeof(double);
    if (v32)   // the level's vectors in FP32, as its rows
        hipLaunchKernelGGL((k_mg_tile27<MODE, true>), dim3(q.blocks), dim3(kTT), lds, st, g);
    else
        hipLaunchKernelGGL((k_mg_tile27<MODE, false>), dim3(q.blocks), dim3(kTT), lds, st, g);
}
inline bool tiled27(const TileGeo& t, int l) { return l >= 1 && l < kMgMaxLevels && t.t27[l].on; }

// level 0: z = x0 + w D^{-1} (r - A x0), x0 = w D^{-1} r + P x1 (fused). z is
// FP32, in the first half of its FP64 array, with 16 right-hand sides; c32:
// level 1's x in FP32
template <int B>
void launch_ps(const MgState& M, const TileGeo& t, hipStream_t st, const double* r, const double* x1, double* z,
               bool c32) {
    if constexpr (B >= 8) {   // tile_setup turns the tiling on only there
        const TileArgs g = ps_args<B>(M, t, r, x1, z);
        const dim3 grid(t.ps_blocks), blk(MgTile<B>::T);
        if (B == 16 && c32)
            hipLaunchKernelGGL((k_mg_tile<kTProlongSmooth, B, B == 16, B == 16>), grid, blk, MgTile<B>::LDS, st, g);
        else
            hipLaunchKernelGGL((k_mg_tile<kTProlongSmooth, B, B == 16>), grid, blk, MgTile<B>::LDS, st, g);
    }
}

// level l's residual to level l + 1's b and first sweep xc (tiled; trilinear)
template <int B>
void launch_restrict(const MgState& M, const TileGeo& t, int l, hipStream_t st, double* xc, bool v1 = false) {
    if constexpr (B >= 8) {
        const MgLevel& L = M.lv[l];
        const MgLevel& C = M.lv[l + 1];
        const TileGeo::Rst& q = t.rst[l];
        RstArgs g;
        g.nx = L.nx;
        g.ny = L.ny;
        g.nz = L.nz;
        g.cx = C.nx;
        g.cy = C.ny;
        g.cz = C.nz;
        g.tiles_x = q.tx;
        g.tiles_y = q.ty;
        g.zc = q.zc;
        g.items = q.items;
        g.r = L.r;
        g.dinv = C.dinv;
        g.w = M.w + l + 1;   // system 0, level l + 1
        g.bc = C.b;
        g.xc = xc;
        g.sc = M.sc;
        // the finest level's residual comes from the tiled kernels in FP32; v1:
        // level 1's vectors are FP32 too (written here from level 0, read here
        // towards level 2)
        if (l == 0 && v1)
            hipLaunchKernelGGL((k_mg_restrict_tile<B, true, true>), dim3(q.blocks), dim3(kTT), MgRst<B>::LDS, st, g);
        else if (l == 0 || (l == 1 && v1))
            hipLaunchKernelGGL((k_mg_restrict_tile<B, true>), dim3(q.blocks), dim3(kTT), MgRst<B>::LDS, st, g);
        else
            hipLaunchKernelGGL((k_mg_restrict_tile<B, false>), dim3(q.blocks), dim3(kTT), MgRst<B>::LDS, st, g);
    }
}

// The finest-level tiling for block size B: on for the Kuhn stencil of one
// system with B >= 8 whose plane offsets fit 32 bits; the z-chunk length
// balances the work items over the blocks resident per XCD.
// ---- autotuning of the tiled z-chunk length
// The cost model ranks z-chunk lengths by (item waves per XCD) x (planes + 2).
// With opts.autotune the lowest-cost candidates (at most kTuneCands distinct
// lengths) are timed on the device, each by one untimed and kTuneReps timed
// launches of the kernel on scratch vectors, in kTuneRounds interleaved rounds
// (each candidate keeps its fastest round: the first launches of a process run
// on a GPU that is still raising its clocks). The model's first candidate is
// kept unless another is faster by more than kTuneMargin, so timing noise of a
// few percent cannot move the choice away from the model's. The choice is
// cached per process by (kernel, lattice size, block), so a second context on
// the same lattice reuses it; timings taken while other streams load the GPU
// (concurrent batched instances) are noisier but only pick among the model's
// own candidates.
constexpr int kTuneCands = 4, kTuneReps = 3, kTuneRounds = 2;
constexpr float kTuneMargin = 0.02f;

// index of the candidate to keep from their times (model order)
inline size_t tune_pick(const std::vector<float>& ms) {
    size_t best = 0;
    for (size_t i = 1; i < ms.size(); ++i)
        if (ms[i] < ms[0] * (1.f - kTuneMargin) && ms[i] < ms[best]) best = i;
    return best;
}
using TuneKey = std::tuple<int, int, int, int, int>;   // kernel, nx, ny, nz, B
std::mutex g_tune_mu;
std::map<TuneKey, int32_t> g_tune;

// the candidate chunk lengths (even: only even lengths), lowest model cost first
inline std::vector<int64_t> chunk_candidates(int64_t nz, int64_t tiles, int64_t conc, bool even) {
    std::vector<std::pair<int64_t, int64_t>> cz;   // (cost, zc)
    for (int64_t nch = 1; nch <= nz; ++nch) {
        int64_t zc = (nz + nch - 1) / nch;
        if (even) zc += zc & 1;
        const int64_t items = tiles * ((nz + zc - 1) / zc);
        const int64_t cost = (((items + 7) / 8 + conc - 1) / conc) * (zc + 2);
        bool seen = false;
        for (auto& e : cz) seen = seen || e.second == zc;
        if (!seen) cz.emplace_back(cost, zc);
    }
    std::stable_sort(cz.begin(), cz.end(), [](const auto& a, const auto& b) { return a.first < b.first; });
    std::vector<int64_t> out;
    for (size_t i = 0; i < cz.size() && (int)i < kTuneCands; ++i) out.push_back(cz[i].second);
    return out;
}

// mean time (ms) of kTuneReps launches after one untimed launch
template <typename F>
qpat_status time_launches(qpat_ctx* c, F&& launch, float* ms) {
    hipEvent_t e0 = nullptr, e1 = nullptr;
    QPAT_HIP(c, hipEventCreate(&e0));
    QPAT_HIP(c, hipEventCreate(&e1));
    launch();
    QPAT_HIP(c, hipEventRecord(e0, c->stream));
    for (int r = 0; r < kTuneReps; ++r) launch();
    QPAT_HIP(c, hipEventRecord(e1, c->stream));
    QPAT_HIP(c, hipGetLastError());
    QPAT_HIP(c, hipEventSynchronize(e1));
    QPAT_HIP(c, hipEventElapsedTime(ms, e0, e1));
    *ms /= kTuneReps;
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    return QPAT_OK;
}

template <int B>
qpat_status tile_geometry(qpat_ctx* c, MgState& M, TileGeo& t) {
    const MgLevel& L = M.lv[0];
    if constexpr (B >= 8) {
        if (M.nsys != 1 || L.kind != 1 || L.N * B * (int64_t)sizeof(double) >= (int64_t(1) << 31)) return QPAT_OK;
        static_assert(MgTile<B>::LDS <= 159 * 1024, "tiled multigrid LDS budget");
        const void* fns[] = {reinterpret_cast<const void*>(&k_mg_tile<kTDirSpmv, B>),
                             reinterpret_cast<const void*>(&k_mg_tile<kTResidFirst, B>),
                             reinterpret_cast<const void*>(&k_mg_tile<kTTrue, B>),
                             reinterpret_cast<const void*>(&k_mg_tile<kTApply, B>),
                             reinterpret_cast<const void*>(&k_mg_tile<kTUpdResid, B>),
                             reinterpret_cast<const void*>(&k_mg_tile<kTProlongSmooth, B, B == 16>),
                             reinterpret_cast<const void*>(&k_mg_tile<kTProlongSmooth, B, B == 16, B == 16>),
                             reinterpret_cast<const void*>(&k_mg_tile<kTDirSpmv, B, true>),
                             reinterpret_cast<const void*>(&k_mg_tile<kTDirSpmv, B, true, true>)};
        for (const void* f : fns)   // dynamic LDS beyond the default limit is allowed per kernel
            QPAT_HIP(c, hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)MgTile<B>::LDS));
        int occ = 1, cus = 256;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, reinterpret_cast<const void*>(&k_mg_tile<kTUpdResid, B>), MgTile<B>::T, MgTile<B>::LDS) != hipSuccess) occ = 1;
        if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, c->device) != hipSuccess) cus = 256;
        // blocks resident per XCD; each leaves one partial sum
        const int64_t conc = std::min<int64_t>((int64_t)std::max(occ, 1) * std::max(cus / 8, 1), kMgBlocks / 8);
        const int64_t tx = (L.nx + kTX - 1) / kTX, ty = (L.ny + kTY - 1) / kTY;
        int64_t best = -1, best_zc = L.nz;
        for (int64_t nch = 1; nch <= L.nz; ++nch) {
            const int64_t zc = (L.nz + nch - 1) / nch;
            const int64_t items = tx * ty * ((L.nz + zc - 1) / zc);
            const int64_t cost = (((items + 7) / 8 + conc - 1) / conc) * (zc + 2);
            if (best < 0 || cost < best) {
                best = cost;
                best_zc = zc;
            }
        }
        t.tiles_x = static_cast<int32_t>(tx);
        t.tiles_y = static_cast<int32_t>(ty);
        auto set_zc = [&](int64_t zc) {
            t.zc = static_cast<int32_t>(zc);
            t.items = static_cast<int32_t>(tx * ty * ((L.nz + zc - 1) / zc));
            t.blocks = static_cast<int32_t>(8 * std::min<int64_t>(conc, (t.items + 7) / 8));
        };
        set_zc(best_zc);
        t.zc_model = t.zc;
        t.on = true;
        if (c->opts.autotune) {
            // time the two kernels of every PCG iteration that share this geometry, the
            // direction + product and the fused update + first residual (FP64 forms), on
            // the PCG's scratch vectors with every lane active
            const TuneKey key{0, L.nx, L.ny, L.nz, B};
            int32_t zc_t = 0;
            {
                std::lock_guard<std::mutex> lk(g_tune_mu);
                auto it = g_tune.find(key);
                if (it != g_tune.end()) zc_t = it->second;
            }
            if (!zc_t) {
                MgScal* sc_t = nullptr;
                QPAT_TRY(dalloc(c, &sc_t, B));
                std::vector<MgScal> hs(B);
                for (auto& h : hs) {
                    std::memset(&h, 0, sizeof h);
                    h.active = 1;
                    h.alpha = 0.5;
                    h.beta = 0.5;   // nonzero: the direction kernel reads the old direction
                }
                QPAT_HIP(c, hipMemcpyAsync(sc_t, hs.data(), B * sizeof(MgScal), hipMemcpyHostToDevice, c->stream));
                for (double* v : {M.pa, M.pb, M.pq, M.pr, M.pr2})
                    QPAT_HIP(c, hipMemsetAsync(v, 0, L.N * B * sizeof(double), c->stream));
                const std::vector<int64_t> cands = chunk_candidates(L.nz, tx * ty, conc, false);
                std::vector<float> cms(cands.size(), 0.f);
                for (int round = 0; round < kTuneRounds; ++round)
                for (size_t ci = 0; ci < cands.size(); ++ci) {
                    set_zc(cands[ci]);
                    TileArgs g{};
                    g.nx = L.nx;
                    g.ny = L.ny;
                    g.nz = L.nz;
                    g.tiles_x = t.tiles_x;
                    g.tiles_y = t.tiles_y;
                    g.zc = t.zc;
                    g.items = t.items;
                    g.ld = B;
                    g.col = 0;
                    g.U = L.U;
                    g.dinv = L.dinv;
                    g.w = M.w;
                    g.parts = M.parts;
                    g.sc = sc_t;
                    TileArgs gd = g, gu = g;
                    gd.in = M.pa;    // z
                    gd.in2 = M.pb;   // old direction
                    gd.out = M.pq;   // q
                    gd.out2 = M.pr;  // new direction
                    gu.in = M.pr;    // r
                    gu.in2 = M.pq;   // q
                    gu.out = M.lv[0].r;
                    gu.out2 = M.pr2;
                    const dim3 grid(t.blocks);
                    float ms_d = 0.f, ms_u = 0.f;
                    QPAT_TRY(time_launches(c, [&] {
                        hipLaunchKernelGGL((k_mg_tile<kTDirSpmv, B>), grid, dim3(MgTile<B>::T), MgTile<B>::LDS, c->stream, gd);
                    }, &ms_d));
                    QPAT_TRY(time_launches(c, [&] {
                        hipLaunchKernelGGL((k_mg_tile<kTUpdResid, B>), grid, dim3(MgTile<B>::T), MgTile<B>::LDS, c->stream, gu);
                    }, &ms_u));
                    cms[ci] = round == 0 ? ms_d + ms_u : std::min(cms[ci], ms_d + ms_u);
                }
                zc_t = static_cast<int32_t>(cands[tune_pick(cms)]);
                std::lock_guard<std::mutex> lk(g_tune_mu);
                g_tune.emplace(key, zc_t);
            }
            set_zc(zc_t);
            t.tuned = true;
        }
        // restrictions to levels 1, 2, ... (coarse level of at least kTile27Min nodes): the
        // same balance with (2 zc + 1) fine planes per item
        const MgLevel& C = M.lv[1];
        const void* fr = reinterpret_cast<const void*>(&k_mg_restrict_tile<B, true>);
        for (const void* f : {fr, reinterpret_cast<const void*>(&k_mg_restrict_tile<B, false>),
                              reinterpret_cast<const void*>(&k_mg_restrict_tile<B, true, true>)})
            QPAT_HIP(c, hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)MgRst<B>::LDS));
        int rocc = 1;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&rocc, fr, kTT, MgRst<B>::LDS) != hipSuccess) rocc = 1;
        const int64_t rconc = (int64_t)std::max(rocc, 1) * (cus / 8);
        for (int l = 0; l + 1 < (int)M.lv.size() && l < kMgMaxLevels; ++l) {
            const MgLevel& Q = M.lv[l + 1];
            if (l > 0 && Q.N < kTile27Min) break;
            const int64_t rtx = (Q.nx + kRX - 1) / kRX, rty = (Q.ny + MgRst<B>::RY - 1) / MgRst<B>::RY;
            int64_t rbest = -1, rzc = Q.nz;
            for (int64_t nch = 1; nch <= Q.nz; ++nch) {
                const int64_t zc = (Q.nz + nch - 1) / nch;
                const int64_t items = rtx * rty * ((Q.nz + zc - 1) / zc);
                const int64_t cost = (((items + 7) / 8 + rconc - 1) / rconc) * (2 * zc + 2);
                if (rbest < 0 || cost < rbest) {
                    rbest = cost;
                    rzc = zc;
                }
            }
            TileGeo::Rst& q = t.rst[l];
            q.tx = static_cast<int32_t>(rtx);
            q.ty = static_cast<int32_t>(rty);
            q.zc = static_cast<int32_t>(rzc);
            q.items = static_cast<int32_t>(rtx * rty * ((Q.nz + rzc - 1) / rzc));
            q.blocks = static_cast<int32_t>(8 * std::min<int64_t>(rconc, (q.items + 7) / 8));
            q.on = true;
        }
        {   // the fused prolongation + last sweep: the same tiles, even chunks
            int64_t best_ps = -1, zc_ps = L.nz + (L.nz & 1);
            for (int64_t nch = 1; nch <= L.nz; ++nch) {
                int64_t zc = (L.nz + nch - 1) / nch;
                zc += zc & 1;
                const int64_t items = tx * ty * ((L.nz + zc - 1) / zc);
                const int64_t cost = (((items + 7) / 8 + conc - 1) / conc) * (zc + 2);
                if (best_ps < 0 || cost < best_ps) {
                    best_ps = cost;
                    zc_ps = zc;
                }
            }
            auto set_ps = [&](int64_t zc) {
                t.ps_zc = static_cast<int32_t>(zc);
                t.ps_items = static_cast<int32_t>(tx * ty * ((L.nz + zc - 1) / zc));
                t.ps_blocks = static_cast<int32_t>(8 * std::min<int64_t>(conc, (t.ps_items + 7) / 8));
            };
            set_ps(zc_ps);
            t.ps_zc_model = t.ps_zc;
            if (c->opts.autotune) {
                const TuneKey key{1, L.nx, L.ny, L.nz, B};
                int32_t zc_t = 0;
                {
                    std::lock_guard<std::mutex> lk(g_tune_mu);
                    auto it = g_tune.find(key);
                    if (it != g_tune.end()) zc_t = it->second;
                }
                if (!zc_t) {
                    // scratch: r in pa, z in pq, lanes all active in a private scalar array
                    MgScal* sc_t = nullptr;
                    QPAT_TRY(dalloc(c, &sc_t, B));
                    std::vector<MgScal> hs(B);
                    for (auto& h : hs) {
                        std::memset(&h, 0, sizeof h);
                        h.active = 1;
                    }
                    QPAT_HIP(c, hipMemcpyAsync(sc_t, hs.data(), B * sizeof(MgScal), hipMemcpyHostToDevice, c->stream));
                    QPAT_HIP(c, hipMemsetAsync(M.pa, 0, L.N * B * sizeof(double), c->stream));
                    QPAT_HIP(c, hipMemsetAsync(C.x, 0, C.N * B * sizeof(double), c->stream));
                    const std::vector<int64_t> cands = chunk_candidates(L.nz, tx * ty, conc, true);
                    std::vector<float> cms(cands.size(), 0.f);
                    for (int round = 0; round < kTuneRounds; ++round)
                    for (size_t ci = 0; ci < cands.size(); ++ci) {
                        set_ps(cands[ci]);
                        TileArgs g = ps_args<B>(M, t, M.pa, C.x, M.pq);
                        g.sc = sc_t;
                        float ms = 0.f;
                        QPAT_TRY(time_launches(c, [&] {
                            hipLaunchKernelGGL((k_mg_tile<kTProlongSmooth, B, B == 16>), dim3(t.ps_blocks),
                                               dim3(MgTile<B>::T), MgTile<B>::LDS, c->stream, g);
                        }, &ms));
                        cms[ci] = round == 0 ? ms : std::min(cms[ci], ms);
                    }
                    zc_t = static_cast<int32_t>(cands[tune_pick(cms)]);
                    std::lock_guard<std::mutex> lk(g_tune_mu);
                    g_tune.emplace(key, zc_t);
                }
                set_ps(zc_t);
            }
        }
        if constexpr (B == 16) {   // the coarse levels' 27-point kernels
            const void* f27[4] = {reinterpret_cast<const void*>(&k_mg_tile27<kT27Resid>),
                                  reinterpret_cast<const void*>(&k_mg_tile27<kT27Smooth>),
                                  reinterpret_cast<const void*>(&k_mg_tile27<kT27Resid, true>),
                                  reinterpret_cast<const void*>(&k_mg_tile27<kT27Smooth, true>)};
            constexpr size_t lds27 = (size_t)3 * kNpf16 * kTT * sizeof(double);
            for (const void* f : f27)
                QPAT_HIP(c, hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds27));
            int occ27 = 1;
            if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ27, f27[1], kTT, lds27) != hipSuccess) occ27 = 1;
            const int64_t conc27 = (int64_t)std::max(occ27, 1) * (cus / 8);
            for (int l = 1; l < (int)M.lv.size() && l < kMgMaxLevels; ++l) {
                const MgLevel& Q = M.lv[l];
                if (!Q.Uf27p) continue;
                const int64_t tx27 = (Q.nx + kTHX - 3) / (kTHX - 2), ty27 = (Q.ny + kTHY - 3) / (kTHY - 2);
                int64_t best27 = -1, zc27 = Q.nz;
                for (int64_t nch = 1; nch <= Q.nz; ++nch) {
                    const int64_t zc = (Q.nz + nch - 1) / nch;
                    const int64_t items = tx27 * ty27 * ((Q.nz + zc - 1) / zc);
                    const int64_t cost = (((items + 7) / 8 + conc27 - 1) / conc27) * (zc + 2);
                    if (best27 < 0 || cost < best27) {
                        best27 = cost;
                        zc27 = zc;
                    }
                }
                TileGeo::Lv27& g27 = t.t27[l];
                g27.tx = static_cast<int32_t>(tx27);
                g27.ty = static_cast<int32_t>(ty27);
                g27.zc = static_cast<int32_t>(zc27);
                g27.items = static_cast<int32_t>(tx27 * ty27 * ((Q.nz + zc27 - 1) / zc27));
                g27.blocks = static_cast<int32_t>(8 * std::min<int64_t>(conc27, (g27.items + 7) / 8));
                g27.on = true;
            }
        }
    }
    return QPAT_OK;
}

// M.tiles[B], on the first call that succeeds
template <int B>
qpat_status tile_setup(qpat_ctx* c, MgState& M) {
    if (M.tiles[B].ready) return QPAT_OK;
    const ScopedArrays scratch(c);
    TileGeo t;
    QPAT_TRY(tile_geometry<B>(c, M, t));
    t.ready = true;
    M.tiles[B] = t;
    return QPAT_OK;
}

// row kind of the V-cycle's kernels on a level
inline int vkind(const MgLevel& L) { return L.vkind >= 0 ? L.vkind : L.kind; }

// The tiled path (K) fuses the PCG update with the V-cycle's first residual and
// the prolongation with its last finest-level sweep. That leaves z in FP32
// with 16 right-hand sides.
static_assert(kMgNu == 1, "the tiled kernels take one sweep each way");
template <int B>
inline bool z32_path(const TileGeo& tg) {
    return B == 16 && tg.on;
}

// One right-hand side per system (M_delta), walk kernels with the FP32 Kuhn
// rows and one sweep each way: the finest level's V-cycle vectors (x0, its
// residual, z) are FP32, in the first half of their FP64 arrays. Every kernel
// that touches them has that form: the PCG update's first sweep (or the first
// sweep from zero), the residual, the restriction, the prolongation into
// level 0, the last sweep (whose dot products use z as stored) and the
// direction. The PCG's own vectors (x, r, p, q) stay FP64.
template <int B>
inline bool f32v0_path(const MgState& M, const TileGeo& tg) {
    return B == 1 && M.opdep && !tg.on && M.lv.size() > 1 && M.lv[0].vkind == 5 &&
           M.lv[0].N * 8 < (int64_t(1) << 31);
}

// Level 1 keeps the V-cycle's vectors (x, its ping-pong partner, r, b) in FP32,
// in the first half of their FP64 arrays, where every kernel that touches them
// has that form: 16 right-hand sides, the tiled restrictions into and out of
// level 1, its tiled 27-point residual and sweep, the prolongation into it and
// the fused prolongation + last sweep above it (preconditioner work only).
template <int B>
inline bool v32_path(const MgState& M, const TileGeo& tg) {
    return z32_path<B>(tg) && M.lv.size() > 2 && tiled27(tg, 1) && tg.rst[0].on &&
           tg.rst[1].on;
}

// the smoother arguments of level l
inline SmArgs level_args(const MgState& M, int l) {
    SmArgs a;
    a.L = lv_args(M.lv[l]);
    a.dinv = M.lv[l].dinv;
    a.w = M.w;
    a.nlev = static_cast<int>(M.lv.size());
    a.lev = l;
    a.nsys = M.nsys;
    a.sc = M.sc;
    return a;
}

// Small levels: the time of a kernel is its launch and its first memory round
// trips, and two passes in one launch (k_mgp_dir_spmv, k_mg_resid_restrict)
// beat the two with fewer reads. In threads of the walk kernels; a Jacobian
// pair (separate -> fused) on 17^3 nodes with 4 right-hand sides 1449 -> 1302
// us, 33^3 with 4 2250 -> 2210, 41^3 with 1 2578 -> 2498; M_delta's kernels
// read their transfer weights as well: 17^3 838 -> 793, 25^3 1756 -> 1742,
// 33^3 1484 -> 1583. The coarse levels' 27-point rows are formed up to 8 times
// over at more cost: six solves side by side, 25^3 - 61^3, never 11.15 ms, up
// to 20000 threads 11.02, up to 80000 11.62 (17^3 with 16 right-hand sides,
// 39000 threads, 16.7 us against 5.9 + 5.6).
constexpr int64_t kFuseK = 80000, kFuseM = 32768, kFuseCoarse = 20000;
template <int B>
inline bool fuse_small(int64_t n, int nsys, int lev = 0) {
    return n * Pk<B>::BV * nsys <= (lev > 0 ? kFuseCoarse : nsys == 1 ? kFuseK : kFuseM);
}

// level l's residual to level l + 1's b and first sweep xc, in one launch
// (f0: level 0's vectors in FP32)
template <int B>
void launch_resid_restrict(const MgState& M, int l, hipStream_t st, const double* b, const double* x, double* xc,
                           bool f0) {
    const MgLevel& L = M.lv[l];
    const MgLevel& C = M.lv[l + 1];
    const SmArgs f = level_args(M, l), c = level_args(M, l + 1);
    const dim3 g = sys_rows(dim3((unsigned)((C.N * Pk<B>::BV * 32 + kMgT - 1) / kMgT)), B, M.nsys);
    const auto go = [&](auto kind, auto opw, auto x_) {
        hipLaunchKernelGGL((k_mg_resid_restrict<decltype(kind)::value, B, decltype(opw)::value,
                                                std::remove_const_t<std::remove_pointer_t<decltype(x_)>>>),
                           g, dim3(kMgT), 0, st, f, c, b, x_, C.b, xc, L.Wc);
    };
    using std::integral_constant;
    const auto kinds = [&](auto opw) {
        switch (vkind(L)) {
            case 1: go(integral_constant<int, 1>{}, opw, x); break;
            case 2: go(integral_constant<int, 2>{}, opw, x); break;
            case 3: go(integral_constant<int, 3>{}, opw, x); break;
            case 4: if constexpr (B == 1) go(integral_constant<int, 4>{}, opw, x); break;
            case 5: if constexpr (B == 1) go(integral_constant<int, 5>{}, opw, x); break;
            case 6: if constexpr (B == 1) go(integral_constant<int, 6>{}, opw, x); break;
            default: go(integral_constant<int, 0>{}, opw, x); break;
        }
    };
    if constexpr (B == 1) {   // M_delta: operator-dependent weights
        if (f0)
            go(integral_constant<int, 5>{}, std::true_type{}, reinterpret_cast<const float*>(x));
        else if (M.opdep)
            kinds(std::true_type{});
        else
            kinds(std::false_type{});
    } else {
        kinds(std::false_type{});
    }
}

// One V-cycle on every lane: z = V(r), r = level 0's b. The last sweep also
// leaves the partial sum r.z (M_delta: and sum z, sum r). On a tiled finest
// level the first sweep w D^{-1} r is never stored: the residual kernel stages
// it and the prolongation recomputes it. Level 0 takes 2 kMgNu - 1 ping-pong
// sweeps (an odd number), so z ends in level 0's t.
// first_done: the PCG update already wrote the finest level's first sweep
// look: asked once the way down and the coarsest solve are launched, so that the
// device has work while the host waits for the answer and launches the rest (asked
// behind level 0 alone, a pair on 41 x 34 x 29 nodes with 16 right-hand sides took
// 2577 - 2585 us against 2567 without the question or with it here; an idle way
// down costs a zero right-hand side some 15 us); false ends the cycle there.
// Returns whether it was completed.
template <int B>
bool vcycle(const MgState& M, hipStream_t st, const TileGeo& tg, hipEvent_t* ev = nullptr, const double* b0 = nullptr,
            bool resid_done = false, bool first_done = false, const std::function<bool()>& look = {}) {
    const int nl = static_cast<int>(M.lv.size());
    const bool v1 = v32_path<B>(M, tg);   // level 1's vectors in FP32
    const bool f0 = f32v0_path<B>(M, tg);  // level 0's vectors in FP32 (one right-hand side)
    const double* r0 = b0 ? b0 : M.lv[0].b;   // level 0's right-hand side (the PCG residual)
    std::vector<double*> xl(nl), tl(nl);
    for (int l = 0; l < nl; ++l) {
        xl[l] = M.lv[l].x;
        tl[l] = M.lv[l].t;
    }
    auto sm = [&](int l) { return level_args(M, l); };
    for (int l = 0; l < nl - 1; ++l) {
        const MgLevel& L = M.lv[l];
        const MgLevel& C = M.lv[l + 1];
        const SmArgs a = sm(l);
        const dim3 g = sgrid<B>(L.N, M.nsys);
        const double* bl = l == 0 ? r0 : L.b;
        if (l == 0 && !tg.on && !first_done && f0)
            hipLaunchKernelGGL((k_mg_first<B, float>), sys_rows(vgrid(L.N * B), B, M.nsys), dim3(kMgT), 0, st, a, r0,
                               reinterpret_cast<float*>(xl[0]));
        else if (l == 0 && !tg.on && !first_done)
            hipLaunchKernelGGL(k_mg_first<B>, sys_rows(vgrid(L.N * B), B, M.nsys), dim3(kMgT), 0, st, a, r0, xl[0]);
        if (l == 0 && ev) (void)hipEventRecord(ev[0], st);
        const bool tiled = (l == 0 && tg.on) || (B == 16 && tiled27(tg, l)) ||
                           (tg.on && l < kMgMaxLevels && tg.rst[l].on && !M.opdep);
        if (!tiled && !ev && fuse_small<B>(L.N, M.nsys, l)) {   // residual and restriction in one launch
            launch_resid_restrict<B>(M, l, st, bl, xl[l], xl[l + 1], l == 0 && f0);
            continue;
        }
        if (l == 0 && tg.on && resid_done)
            ;   // the PCG update produced level 0's residual (kTUpdResid)
        else if (l == 0 && tg.on)
            launch_tile<kTResidFirst, B>(M, tg, st, r0, nullptr, r0, L.r, nullptr);
        else if (B == 16 && tiled27(tg, l))
            launch_tile27<kT27Resid>(M, tg, l, st, xl[l], L.b, L.r, v1 && l == 1);
        else if (l == 0 && f0) {
            if constexpr (B == 1)
                hipLaunchKernelGGL((k_mg_resid<5, 1, float>), g, dim3(kMgT), 0, st, a, bl,
                                   reinterpret_cast<const float*>(xl[0]), reinterpret_cast<float*>(L.r));
        } else
            QPAT_MG_KIND(vkind(L), B, k_mg_resid, g, dim3(kMgT), 0, st, a, bl, xl[l], L.r);
        if (l == 0 && ev) (void)hipEventRecord(ev[1], st);
        if (tg.on && l < kMgMaxLevels && tg.rst[l].on && !M.opdep)
            launch_restrict<B>(M, tg, l, st, xl[l + 1], v1);
        else if (M.opdep && l == 0 && f0)
            hipLaunchKernelGGL((k_mg_restrict<B, true, float>), sgrid<B>(C.N, M.nsys), dim3(kMgT), 0, st, sm(l + 1),
                               L.nx, L.ny, L.nz, reinterpret_cast<const float*>(L.r), C.b, xl[l + 1], L.Wc);
        else if (M.opdep)
            hipLaunchKernelGGL((k_mg_restrict<B, true>), sgrid<B>(C.N, M.nsys), dim3(kMgT), 0, st, sm(l + 1), L.nx,
                               L.ny, L.nz, L.r, C.b, xl[l + 1], L.Wc);
        else
            hipLaunchKernelGGL((k_mg_restrict<B, false>), sgrid<B>(C.N, M.nsys), dim3(kMgT), 0, st, sm(l + 1), L.nx, L.ny,
                               L.nz, L.r, C.b, xl[l + 1], static_cast<const float*>(nullptr));
    }
    const MgLevel& K = M.lv[nl - 1];
    hipLaunchKernelGGL(k_mg_dense<B>,
                       dim3((unsigned)((K.N + kMgT / 64 - 1) / (kMgT / 64)), (unsigned)Pk<B>::BV, (unsigned)M.nsys),
                       dim3(kMgT), K.N * sizeof(TB<B>), st, K.N, M.nsys, M.ainv, K.b, xl[nl - 1], M.sc);
    if (look && !look()) return false;
    for (int l = nl - 2; l >= 0; --l) {
        const MgLevel& L = M.lv[l];
        const MgLevel& C = M.lv[l + 1];
        const SmArgs a = sm(l);
        const dim3 g = sgrid<B>(L.N, M.nsys);
        const double* bl = l == 0 ? r0 : L.b;
        if (l == 0 && tg.on) {   // prolongation fused into the last sweep
            if (ev) (void)hipEventRecord(ev[2], st);
            launch_ps<B>(M, tg, st, r0, xl[1], tl[0], v1);
            if (ev) (void)hipEventRecord(ev[3], st);
            std::swap(xl[0], tl[0]);
            continue;
        }
        if (M.opdep && l == 0 && f0)   // into level 0's FP32 x0
            hipLaunchKernelGGL((k_mg_prolong<B, true, true>), g, dim3(kMgT), 0, st, a, C.nx, C.ny, C.nz,
                               xl[l + 1], xl[l], L.Wc);
        else if (M.opdep)
            hipLaunchKernelGGL((k_mg_prolong<B, true>), g, dim3(kMgT), 0, st, a, C.nx, C.ny, C.nz,
                               xl[l + 1], xl[l], L.Wc);
        else if (l == 1 && v1)   // into level 1's FP32 x
            hipLaunchKernelGGL((k_mg_prolong<B, false, true>), g, dim3(kMgT), 0, st, a, C.nx, C.ny,
                               C.nz, xl[l + 1], xl[l], static_cast<const float*>(nullptr));
        else
            hipLaunchKernelGGL((k_mg_prolong<B, false>), g, dim3(kMgT), 0, st, a, C.nx, C.ny, C.nz, xl[l + 1],
                               xl[l], static_cast<const float*>(nullptr));
        for (int k = 0; k < kMgNu; ++k) {
            const bool last = l == 0 && k == kMgNu - 1;
            if (last && ev) (void)hipEventRecord(ev[2], st);
            if (last && f0) {
                if constexpr (B == 1)
                    hipLaunchKernelGGL((k_mg_smooth<5, 1, true, float>), g, dim3(kMgT), 0, st, a, bl,
                                       reinterpret_cast<const float*>(xl[0]), reinterpret_cast<float*>(tl[0]),
                                       M.parts);
            } else if (last)
                launch_smooth<B, true>(vkind(L), g, st, a, bl, xl[l], tl[l], M.parts);
            else if (B == 16 && tiled27(tg, l))
                launch_tile27<kT27Smooth>(M, tg, l, st, xl[l], L.b, tl[l], v1 && l == 1);
            else
                launch_smooth<B, false>(vkind(L), g, st, a, bl, xl[l], tl[l], nullptr);
            if (last && ev) (void)hipEventRecord(ev[3], st);
            std::swap(xl[l], tl[l]);
        }
    }
    return true;
}

// blocks of the V-cycle's last finest-level sweep, which leave r.z
template <int B>
inline int last_blocks(const MgState& M, const TileGeo& tg) {
    if (tg.on) return tg.ps_blocks;
    return static_cast<int>(sgrid<B>(M.lv[0].N).x);
}

MgState*& state_of(qpat_ctx* c, Op op) { return op == Op::K ? c->mgk : c->mg; }

template <int B>
PcgMg pcg_args(qpat_ctx* c, Op op) {
    const MgState& M = *state_of(c, op);
    PcgMg a;
    a.L = lv_args(M.lv[0]);
    a.x = c->x64;
    a.r = M.pr;
    a.po = M.pa;
    a.pn = M.pb;
    a.q = M.pq;
    a.z = M.lv[0].t;   // where the V-cycle leaves z
    a.parts = M.parts;
    a.sc = M.sc;
    const double rtol = op == Op::K ? c->opts.pcg_rtol : c->opts.prior_rtol;
    a.rtol2 = rtol * rtol;
    a.maxit = c->opts.pcg_maxit;
    a.deflate = op == Op::Prior ? c->opts.prior_deflate : 0;
    a.nsys = M.nsys;
    a.nbr = static_cast<int32_t>(vgrid(c->N, kMgGrid).x);   // k_reg_rsum, k_mgp_update_first
    a.kreg = B == 1 ? M.kreg : 0;
    a.p32 = op == Op::K && c->opts.precision == 1 ? 1 : 0;
    a.reg = M.reg;
    a.ry = M.ry;
    a.rcorr = M.rcorr;
    a.ring = 0;   // solve_B turns the direction ring on for the tiled iterations
    a.slot = M.pslot;
    a.ahist = M.ahist;
    return a;
}

// the region coarse-space part of the preconditioner for the current r
// (sums_done: the PCG update already left the partial sums of Z^T r and of
// r.r, and the scalars of the latter are due)
template <int B>
void region_solve(const MgState& M, const PcgMg& a, hipStream_t st, bool sums_done = false) {
    if (a.kreg <= 0) return;
    // each block reduces kRegMax sums: fewer, fuller blocks than the walk kernels
    if (!sums_done)
        hipLaunchKernelGGL(k_reg_rsum, sys_rows(vgrid(a.L.N, kMgGrid), B, a.nsys), dim3(kMgT), 0, st, a, M.rparts);
    hipLaunchKernelGGL(k_reg_solve, dim3(1, a.nsys), dim3(kMgT), 0, st, a, sums_done ? a.nbr : 0, M.rparts, M.einv,
                       M.rsize, M.ry, M.rcorr);
}

// one iteration after the first direction: direction and product, alpha,
// update, rr, V-cycle (with r.z), beta. Iterations alternate
// the two direction buffers (par); chunks of iterations have even length.
// ev (profiling): 8 events, recorded around the direction + product, the
// update, and the finest-level residual and last sweep of the V-cycle.
template <int B>
void iteration(const MgState& M, PcgMg a, const TileGeo& tg, hipStream_t st, int par, hipEvent_t* ev = nullptr) {
    if (par) std::swap(a.po, a.pn);
    const dim3 g = sgrid<B>(a.L.N, a.nsys), lanes(1, a.nsys * B);
    if (ev) (void)hipEventRecord(ev[0], st);
    const bool p32 = a.p32 && z32_path<B>(tg);   // mixed precision: the direction in FP32
    RingArg ring;   // the direction ring: the slots of this iteration and the one before
    if (a.ring > 0) {
        ring.slot = a.slot;
        ring.base = reinterpret_cast<const char*>(M.pring);
        ring.stride = a.L.N * B * (p32 ? 4 : 8);
        ring.n = a.ring;
    }
    if (tg.on && p32) {
        launch_tile<kTDirSpmv, B, true, true>(M, tg, st, a.z, a.po, nullptr, a.q, a.pn, ring);
    } else if (tg.on && z32_path<B>(tg)) {   // z from the fused prolongation + last sweep, FP32
        launch_tile<kTDirSpmv, B, true>(M, tg, st, a.z, a.po, nullptr, a.q, a.pn, ring);
    } else if (tg.on) {
        launch_tile<kTDirSpmv, B>(M, tg, st, a.z, a.po, nullptr, a.q, a.pn, ring);
    } else {
        const bool zf = f32v0_path<B>(M, tg);   // z in FP32
        if (fuse_small<B>(a.L.N, a.nsys)) {
            if constexpr (B == 1) {
                if (zf && a.L.kind == 3)
                    hipLaunchKernelGGL((k_mgp_dir_spmv<3, 1, true>), g, dim3(kMgT), 0, st, a);
                else
                    QPAT_MG_KIND(a.L.kind, B, k_mgp_dir_spmv, g, dim3(kMgT), 0, st, a);
            } else {
                QPAT_MG_KIND(a.L.kind, B, k_mgp_dir_spmv, g, dim3(kMgT), 0, st, a);
            }
        } else {
            if (zf)
                hipLaunchKernelGGL((k_mgp_dir<B, true>), g, dim3(kMgT), 0, st, a);
            else
                hipLaunchKernelGGL(k_mgp_dir<B>, g, dim3(kMgT), 0, st, a);
            QPAT_MG_KIND(a.L.kind, B, k_mgp_spmv, g, dim3(kMgT), 0, st, a);
        }
    }
    if (ev) (void)hipEventRecord(ev[1], st);
    hipLaunchKernelGGL(k_mgp_scalars, lanes, dim3(kMgT), 0, st, a, tg.on ? tg.blocks : (int)g.x, 0);
    if (ev) (void)hipEventRecord(ev[2], st);
    const bool upd1 = B == 1 && !tg.on && a.L.N * 8 < (int64_t(1) << 31);
    if (tg.on) {   // r, x and the V-cycle's first sweep + residual in one pass; r alternates buffers
        double* r_old = par ? M.pr2 : M.pr;
        double* r_new = par ? M.pr : M.pr2;
        launch_tile<kTUpdResid, B>(M, tg, st, r_old, a.q, nullptr, M.lv[0].r, r_new);
        a.r = r_new;
    } else if (upd1 && f32v0_path<B>(M, tg)) {   // one right-hand side: update, first sweep (FP32), region sums
        hipLaunchKernelGGL(k_mgp_update_first<float>, sys_rows(vgrid(a.L.N, kMgGrid), B, a.nsys), dim3(kMgT), 0, st,
                           a, level_args(M, 0), reinterpret_cast<float*>(M.lv[0].x), M.rparts);
    } else if (upd1) {   // one right-hand side: update, first sweep and region sums in one pass over r
        hipLaunchKernelGGL(k_mgp_update_first<double>, sys_rows(vgrid(a.L.N, kMgGrid), B, a.nsys), dim3(kMgT), 0, st,
                           a, level_args(M, 0), M.lv[0].x, M.rparts);
    } else {
        hipLaunchKernelGGL(k_mgp_update<B>, g, dim3(kMgT), 0, st, a, level_args(M, 0), M.lv[0].x);
    }
    if (ev) (void)hipEventRecord(ev[3], st);
    const int nb1 = tg.on ? tg.blocks : upd1 ? a.nbr : (int)g.x;
    const bool reg1 = upd1 && a.kreg > 0;   // k_reg_solve takes the scalars with it
    if (!reg1) hipLaunchKernelGGL(k_mgp_scalars, lanes, dim3(kMgT), 0, st, a, nb1, 1);
    region_solve<B>(M, a, st, upd1);
    vcycle<B>(M, st, tg, ev ? ev + 4 : nullptr, a.r, tg.on, !tg.on);
    hipLaunchKernelGGL(k_mgp_scalars, lanes, dim3(kMgT), 0, st, a, last_blocks<B>(M, tg), 2);
}

// true residual r = b - A x of every lane, partial r.r (write_r false, tiled path:
// the partial only)
template <int B>
void true_residual(const MgState& M, const PcgMg& a, const TileGeo& tg, const double* b, hipStream_t st,
                   bool write_r = true) {
    if (tg.on)
        launch_tile<kTTrue, B>(M, tg, st, a.x, nullptr, b, write_r ? a.r : nullptr, nullptr);
    else
        QPAT_MG_KIND(a.L.kind, B, k_mgp_true, sgrid<B>(a.L.N, a.nsys), dim3(kMgT), 0, st, a, b);
}

template <int B>
qpat_status solve_B(qpat_ctx* c, Op op, SolveStats* st, bool has_x0) {
    MgState& M = *state_of(c, op);
    hipStream_t sm = c->stream;
    const int S = M.nsys * B;
    const dim3 g = sgrid<B>(c->N, M.nsys), lanes(1, S);
    PcgMg a = pcg_args<B>(c, op);
    QPAT_TRY(tile_setup<B>(c, M));
    const TileGeo tg = M.tiles[B];
    // The tiled iterations keep their directions and alphas in a ring and form
    // x = x + sum alpha_j p_j (k_mgp_ring_flush) before x is read: the update
    // then neither reads nor writes x nor reads p.
    if (tg.on) {
        const size_t n = (size_t)kRing * c->N * M.bmax;   // FP64-sized slots
        QPAT_TRY(dalloc_once(c, &M.ahist, (size_t)kRing * kMgLanes));
        QPAT_TRY(dalloc_once(c, &M.pslot, 1));
        if (!M.pring) {   // finite values in the slots of lanes that stopped (their alpha is 0)
            QPAT_TRY(dalloc(c, &M.pring, n));
            QPAT_HIP(c, hipMemsetAsync(M.pring, 0, n * sizeof(double), sm));
        }
        a.ring = kRing;
        a.slot = M.pslot;
        a.ahist = M.ahist;
    }
    int ring_s = 0, ring_f = 0;   // iterations launched in this solve; those already added to x
    // the one-pass start leaves x unwritten with the ring: the first formation starts from zero
    bool x_zero = a.ring > 0 && tg.on && !a.deflate && !has_x0;
    auto ring_flush = [&]() -> qpat_status {
        if (a.ring == 0 || (ring_s == ring_f && !x_zero)) return QPAT_OK;
        const int64_t n = c->N * (int64_t)B;
        const bool p32r = a.p32 && z32_path<B>(tg);
        const int64_t stride = n * (p32r ? 4 : 8);
        const char* base = reinterpret_cast<const char*>(M.pring);
        if (B % (p32r ? 4 : 2) != 0) return fail(c, QPAT_ERR_STATE, "multigrid: direction ring with %d right-hand sides", B);
        if (p32r)
            hipLaunchKernelGGL(k_mgp_ring_flush<float>, vgrid(n, kMgBlocks), dim3(kMgT), 0, sm, n, B, a.x, base, stride,
                               M.ahist, S, ring_f, ring_s, x_zero ? 1 : 0);
        else
            hipLaunchKernelGGL(k_mgp_ring_flush<double>, vgrid(n, kMgBlocks), dim3(kMgT), 0, sm, n, B, a.x, base, stride,
                               M.ahist, S, ring_f, ring_s, x_zero ? 1 : 0);
        ring_f = ring_s;
        x_zero = false;
        QPAT_HIP(c, hipGetLastError());
        return QPAT_OK;
    };
    const Live live = live_begin(c);
    if (tg.on && !a.deflate && !has_x0) {   // one pass over b
        const dim3 gs = vgrid(c->N * Pk<B>::BV / 4 + 1, kMgBlocks);
        hipLaunchKernelGGL(k_mgp_start0<B>, gs, dim3(kMgT), 0, sm, a, c->b64);
        hipLaunchKernelGGL(k_mgp_init, lanes, dim3(kMgT), 0, sm, a, (int)gs.x, c->delta > 0 ? 1.0 / c->delta : 0.0,
                           live);
    } else {
        hipLaunchKernelGGL(k_mgp_bstats<B>, g, dim3(kMgT), 0, sm, a, c->b64);
        hipLaunchKernelGGL(k_mgp_init, lanes, dim3(kMgT), 0, sm, a, (int)g.x, c->delta > 0 ? 1.0 / c->delta : 0.0,
                           has_x0 ? Live{} : live);
        hipLaunchKernelGGL(k_mgp_start<B>, g, dim3(kMgT), 0, sm, a, c->b64, has_x0 ? 1 : 0);
    }
    if (has_x0) {   // r = b - A x0; lanes that x0 already solves stop here
        true_residual<B>(M, a, tg, c->b64, sm);
        hipLaunchKernelGGL(k_mgp_true_fin, lanes, dim3(kMgT), 0, sm, a, tg.on ? tg.blocks : (int)g.x, 1, live);
    }
    QPAT_HIP(c, hipGetLastError());
    auto fetch = [&]() -> qpat_status {
        QPAT_HIP(c, hipMemcpyAsync(M.sc_host, M.sc, S * sizeof(MgScal), hipMemcpyDeviceToHost, sm));
        QPAT_HIP(c, hipStreamSynchronize(sm));
        return QPAT_OK;
    };
    auto any_active = [&]() {
        for (int i = 0; i < S; ++i)
            if (M.sc_host[i].active) return true;
        return false;
    };
    std::vector<int> reopened(S, 0);   // per lane: restarts after a failed true-residual check
    bool fetched = false;              // sc_host holds the lanes' last state
    bool idle = false;                 // every right-hand side is 0
    // A solve's first V-cycle and chunk go out without a copy of the scalars: a
    // lane with nothing to do is inactive on the device already, and what the
    // chunk lengths need of the start (rr0) comes back with the first check. Each
    // such check is a copy, a wait and an idle device while the next chunk is
    // launched. Only whether any lane iterates at all is asked, behind the
    // V-cycle's way down: right-hand sides of zero (J 0) or a start that solves
    // them end there (M_delta^{-1} 0 on 128^3 voxels 115 us, 670 with the first
    // chunk; on 16^3 82, 200; a pair's two solves are no slower for it).
    for (int restart = 0; restart < 4; ++restart) {
        if (restart > 0) {
            QPAT_TRY(fetch());
            if (!any_active()) {
                fetched = true;
                break;
            }
            for (int i = 0; i < S; ++i) reopened[i] += M.sc_host[i].active ? 1 : 0;
        }
        // the tiled check below stores no r (its lanes almost always stop there):
        // a lane it reopened restarts from the true residual formed here
        if (restart > 0 && tg.on) true_residual<B>(M, a, tg, c->b64, sm);
        // first direction of a run: z = V(r) (+ Z y), p = z - c
        region_solve<B>(M, a, sm);
        if (restart == 0) {
            if (!vcycle<B>(M, sm, tg, nullptr, nullptr, false, false, [&] { return any_live(c, S); })) {
                QPAT_TRY(ring_flush());   // x = 0 where the start left it unwritten
                fetched = idle = !has_x0; // b = 0: nothing to learn from the scalars
                break;
            }
        } else {
            vcycle<B>(M, sm, tg);
        }
        hipLaunchKernelGGL(k_mgp_scalars, lanes, dim3(kMgT), 0, sm, a,
                           last_blocks<B>(M, tg), 3);
        QPAT_HIP(c, hipGetLastError());
        // Iterations run in chunks of even length between host checks. The
        // first is kMgChunk0 long; later ones cover the iterations that the
        // slowest lane still needs at its contraction rate over the last
        // chunk (within [2, 16]), so few iterations run after convergence. PCG
        // converges superlinearly towards the end of a run, where that rate
        // overestimates the need: a third or later chunk is therefore kept to
        // half the iterations the run has done, which bounds the iterations
        // launched after convergence (each still costs its launches) by that
        // half, at the price of a host check more on runs that long.
        int chunk = kMgChunk0, nchunk = 0;
        std::vector<int> iters_before(S, 0), iters_start(S, 0);
        std::vector<double> rr_before(S, 0.0);
        for (int i = 0; restart > 0 && i < S; ++i) {   // from the check above
            iters_before[i] = iters_start[i] = M.sc_host[i].iters;
            rr_before[i] = M.sc_host[i].rr;
        }
        for (;;) {
            if (nchunk > 0) {
                QPAT_TRY(fetch());
                if (!any_active()) break;
                if (nchunk == 1 && restart == 0)
                    for (int i = 0; i < S; ++i) rr_before[i] = M.sc_host[i].rr0;
                double need = 0.0;
                for (int i = 0; i < S; ++i) {
                    const MgScal& h = M.sc_host[i];
                    if (!h.active) continue;
                    const int done_its = h.iters - iters_before[i];
                    const double target = a.rtol2 * h.bnorm2;
                    if (done_its <= 0 || !(rr_before[i] > 0.0) || !(h.rr > 0.0) || h.rr >= rr_before[i]) {
                        need = 16.0;
                        continue;
                    }
                    const double rate = std::log(h.rr / rr_before[i]) / done_its;   // < 0
                    need = std::max(need, std::log(target / h.rr) / rate);
                }
                const int n = static_cast<int>(std::ceil(need));
                chunk = std::min(16, std::max(2, n + (n & 1)));
                if (nchunk >= 2) {
                    int run_its = 0;
                    for (int i = 0; i < S; ++i) run_its = std::max(run_its, M.sc_host[i].iters - iters_start[i]);
                    const int half = run_its / 2;
                    chunk = std::min(chunk, std::max(2, half + (half & 1)));
                }
                for (int i = 0; i < S; ++i) {
                    iters_before[i] = M.sc_host[i].iters;
                    rr_before[i] = M.sc_host[i].rr;
                }
            }
            ++nchunk;
            // the chunk writes ring slots ring_s ... ring_s + chunk - 1: those not yet in x must survive
            if (a.ring > 0 && ring_s + chunk - ring_f > kRing) QPAT_TRY(ring_flush());
            ring_s += chunk;
            const bool prof = c->prof_on;
            if (prof) {
                if (M.ev.size() < (size_t)8 * chunk) {
                    const size_t old = M.ev.size();
                    M.ev.resize((size_t)8 * chunk);
                    for (size_t e = old; e < M.ev.size(); ++e) QPAT_HIP(c, hipEventCreate(&M.ev[e]));
                }
                for (int i = 0; i < chunk; ++i) iteration<B>(M, a, tg, sm, i & 1, &M.ev[8 * i]);
                QPAT_HIP(c, hipGetLastError());
                QPAT_TRY(fetch());
                // iterations after every lane stopped do no work: count the live ones
                const int base = op == Op::K ? 4 : 8;
                for (int i = 0; i < chunk; ++i) {
                    int lanes_on = 0;
                    for (int l = 0; l < S; ++l) lanes_on += (M.sc_host[l].iters - iters_before[l]) > i;
                    if (lanes_on == 0) break;
                    for (int kk = 0; kk < 4; ++kk) {
                        if (kk == 2 && tg.on) continue;   // the update's kernel did it
                        float t = 0.f;
                        QPAT_HIP(c, hipEventElapsedTime(&t, M.ev[8 * i + 2 * kk], M.ev[8 * i + 2 * kk + 1]));
                        qpat_kstat& ks = c->prof[base + kk];
                        ks.launches += 1;
                        ks.lanes += lanes_on;
                        ks.total_ms += t;
                        ks.min_ms = ks.launches == 1 ? t : std::min(ks.min_ms, (double)t);
                        ks.max_ms = std::max(ks.max_ms, (double)t);
                    }
                }
                continue;
            }
            if (c->opts.use_graphs) {
                // the chunk as graphs of 16, 8, 4 and 2 iterations (its binary
                // digits; every chunk is even), so that a solver captures at most
                // four graphs whatever chunk lengths its right-hand sides take
                for (int len = 16; len >= 2; len /= 2) {
                    if (!(chunk & len)) continue;
                    // every by-value argument of the captured kernels that can change
                    // between runs: the region count is recomputed at each prior set-up
                    char key[128];
                    snprintf(key, sizeof key, "%d/%d/%.17g/%d/%d/%d/%d", B, len, a.rtol2, a.maxit, a.deflate, a.kreg,
                             a.p32);
                    auto it = M.graphs.find(key);
                    hipGraphExec_t ex = nullptr;
                    if (it != M.graphs.end()) {
                        ex = it->second;
                    } else {
                        if (!M.cap) QPAT_HIP(c, hipStreamCreateWithFlags(&M.cap, hipStreamNonBlocking));
                        hipGraph_t gr = nullptr;
                        QPAT_HIP(c, hipStreamBeginCapture(M.cap, hipStreamCaptureModeThreadLocal));
                        for (int i = 0; i < len; ++i) iteration<B>(M, a, tg, M.cap, i & 1);
                        QPAT_HIP(c, hipStreamEndCapture(M.cap, &gr));
                        QPAT_HIP(c, hipGraphInstantiate(&ex, gr, nullptr, nullptr, 0));
                        QPAT_HIP(c, hipGraphDestroy(gr));
                        M.graphs[key] = ex;
                    }
                    QPAT_HIP(c, hipGraphLaunch(ex, sm));
                }
            } else {
                for (int i = 0; i < chunk; ++i) iteration<B>(M, a, tg, sm, i & 1);
            }
            QPAT_HIP(c, hipGetLastError());
        }
        // confirm on the true residual; a failed check restarts from the true residual
        QPAT_TRY(ring_flush());
        true_residual<B>(M, a, tg, c->b64, sm, !tg.on);
        hipLaunchKernelGGL(k_mgp_true_fin, lanes, dim3(kMgT), 0, sm, a, tg.on ? tg.blocks : (int)g.x, restart < 3 ? 1 : 0,
                           Live{});
        QPAT_HIP(c, hipGetLastError());
    }
    if (!fetched) QPAT_TRY(fetch());
    for (int i = 0; i < S; ++i) {
        const MgScal& s = M.sc_host[i];
        if (op == Op::Prior)   // the output kernel of the prior solve adds mean(b)/delta
            QPAT_HIP(c, hipMemcpyAsync(&c->scal[i].mean, &M.sc[i].mean, sizeof(double), hipMemcpyDeviceToDevice, sm));
        if (idle) {
            st->add(0, 0.0, 0, true);
            continue;
        }
        const double rel = s.bnorm2 > 0 ? std::sqrt(s.rr / s.bnorm2) : 0.0;
        st->add(s.iters, rel, reopened[i], s.done != 0);
    }
    return QPAT_OK;
}

}  // namespace

static void mg_drop(qpat_ctx* c, Op op) {
    MgState*& M = state_of(c, op);
    if (!M) return;
    for (auto& kv : M->graphs) (void)hipGraphExecDestroy(kv.second);
    for (hipEvent_t e : M->ev) (void)hipEventDestroy(e);
    if (M->cap) (void)hipStreamDestroy(M->cap);
    if (M->sc_host) (void)hipHostFree(M->sc_host);
    delete M;
    M = nullptr;
}

void mg_destroy(qpat_ctx* c) {
    mg_drop(c, Op::K);
    mg_drop(c, Op::Prior);
}

bool mg_available(const qpat_ctx* c, Op op) {
    const bool want = op == Op::K ? c->opts.pcg_precond == 1 : c->opts.prior_precond == 1;
    const double* U = op == Op::K ? c->KU64 : c->MU64;
    // 32-bit element offsets in the kernels: [N][m+1] operator rows, [N][B] vectors
    return want && c->lat.on && c->opts.operator_format == 1 && U &&
           (int64_t)(c->lat.m + 1) * c->N * 8 < (int64_t(1) << 31) && c->N * kMaxRhs < (int64_t(1) << 31);
}

bool mg_ready(qpat_ctx* c, Op op) {
    const MgState* M = state_of(c, op);
    return mg_available(c, op) && M && M->current;
}

// Region coarse space of the finest level of M (one system at a time): labels
// of the strong-coupling components, the kRegMax largest regions with at
// least kRegMin nodes (with deflation: after the largest), E = Z^T A Z (exact
// integer sums) and its inverse.
static qpat_status region_setup(qpat_ctx* c, MgState& M) {
    const MgLevel& F = M.lv[0];
    const int64_t N = F.N;
    const int M1 = F.m + 1;
    QPAT_TRY(dalloc_once(c, &M.reg, M.nsys * N));
    QPAT_TRY(dalloc_once(c, &M.einv, M.nsys * kRegMax * kRegMax));
    QPAT_TRY(dalloc_once(c, &M.rsize, M.nsys * kRegMax));
    QPAT_TRY(dalloc_once(c, &M.rparts, (int64_t)M.nsys * kRegMax * kMgBlocks));
    QPAT_TRY(dalloc_once(c, &M.ry, M.nsys * kRegMax));
    QPAT_TRY(dalloc_once(c, &M.rcorr, 2 * M.nsys));
    const ScopedArrays scratch(c);
    int32_t *lab = nullptr, *cnt = nullptr, *flag = nullptr, *list = nullptr, *roots = nullptr;
    unsigned long long *eint = nullptr, *amax = nullptr;
    QPAT_TRY(dalloc(c, &lab, N));
    QPAT_TRY(dalloc(c, &cnt, N));
    QPAT_TRY(dalloc(c, &flag, 2));
    QPAT_TRY(dalloc(c, &list, 2 * kRegList));
    QPAT_TRY(dalloc(c, &roots, kRegMax));
    QPAT_TRY(dalloc(c, &eint, kRegMax * kRegMax));
    QPAT_TRY(dalloc(c, &amax, 1));
    hipStream_t st = c->stream;
    const dim3 g(grid_for(N, kMgT, 4096)), b(kMgT);
    std::vector<double> einv_h(M.nsys * kRegMax * kRegMax, 0.0), size_h(M.nsys * kRegMax, 0.0);
    M.kreg = 0;
    for (int sys = 0; sys < M.nsys; ++sys) {
        LvArgs L = lv_args(F);
        L.U = F.U + sys * N * M1;
        hipLaunchKernelGGL(k_reg_init, g, b, 0, st, lab, N);
        for (int round = 0;; ++round) {
            if (round > 4096) return fail(c, QPAT_ERR_DEVICE, "region labels did not settle");
            QPAT_HIP(c, hipMemsetAsync(flag, 0, sizeof(int32_t), st));
            hipLaunchKernelGGL(k_reg_prop, g, b, 0, st, L, lab, flag);
            hipLaunchKernelGGL(k_reg_jump, g, b, 0, st, lab, N);
            hipLaunchKernelGGL(k_reg_jump, g, b, 0, st, lab, N);
            int32_t fh = 0;
            QPAT_HIP(c, hipMemcpyAsync(&fh, flag, sizeof fh, hipMemcpyDeviceToHost, st));
            QPAT_HIP(c, hipStreamSynchronize(st));
            if (!fh) break;
        }
        QPAT_HIP(c, hipMemsetAsync(cnt, 0, N * sizeof(int32_t), st));
        hipLaunchKernelGGL(k_reg_count, g, b, 0, st, lab, cnt, N);
        QPAT_HIP(c, hipMemsetAsync(flag + 1, 0, sizeof(int32_t), st));
        hipLaunchKernelGGL(k_reg_roots, g, b, 0, st, lab, cnt, N, list, flag + 1);
        int32_t nl = 0;
        QPAT_HIP(c, hipMemcpyAsync(&nl, flag + 1, sizeof nl, hipMemcpyDeviceToHost, st));
        QPAT_HIP(c, hipStreamSynchronize(st));
        nl = std::min(nl, kRegList);
        std::vector<int32_t> lh(2 * std::max(nl, 1));
        if (nl > 0)
            QPAT_HIP(c, hipMemcpyAsync(lh.data(), list, 2 * nl * sizeof(int32_t), hipMemcpyDeviceToHost, st));
        QPAT_HIP(c, hipStreamSynchronize(st));
        std::vector<std::pair<int32_t, int32_t>> cand;   // (size, root)
        for (int i = 0; i < nl; ++i) cand.push_back({lh[2 * i + 1], lh[2 * i]});
        std::sort(cand.begin(), cand.end(), [](const auto& x, const auto& y) {
            return x.first != y.first ? x.first > y.first : x.second < y.second;
        });
        // With deflation the constant vector is solved exactly; the largest
        // region's indicator is then nearly that vector, and keeping it makes
        // the coarse correction all but repeat the deflated direction (PCG
        // stagnated near rtol 1e-12 with it); the other regions span its
        // complement part anyway.
        const int skip = c->opts.prior_deflate && !cand.empty() ? 1 : 0;
        cand.erase(cand.begin(), cand.begin() + skip);
        int k = std::min<int>(kRegMax, static_cast<int>(cand.size()));
        int32_t rt[kRegMax] = {};
        for (int j = 0; j < k; ++j) rt[j] = cand[j].second;
        QPAT_HIP(c, hipMemcpyAsync(roots, rt, sizeof rt, hipMemcpyHostToDevice, st));
        hipLaunchKernelGGL(k_reg_assign, g, b, 0, st, lab, N, k, roots, M.reg + sys * N);
        // E in fixed point: every sum of |contributions| stays below 2^62
        QPAT_HIP(c, hipMemsetAsync(amax, 0, sizeof(unsigned long long), st));
        hipLaunchKernelGGL(k_reg_absmax, g, b, 0, st, L.U, N * M1, amax);
        unsigned long long ab = 0;
        QPAT_HIP(c, hipMemcpyAsync(&ab, amax, sizeof ab, hipMemcpyDeviceToHost, st));
        QPAT_HIP(c, hipStreamSynchronize(st));
        double maxabs;
        std::memcpy(&maxabs, &ab, sizeof maxabs);
        if (k > 0 && maxabs > 0.0 && std::isfinite(maxabs)) {
            const double bound = static_cast<double>(N) * (2 * F.m + 1) * maxabs;
            const double scale = std::ldexp(1.0, static_cast<int>(std::floor(62.0 - std::log2(bound))));
            QPAT_HIP(c, hipMemsetAsync(eint, 0, kRegMax * kRegMax * sizeof(unsigned long long), st));
            hipLaunchKernelGGL(k_reg_e, g, b, 0, st, L, M.reg + sys * N, scale, eint);
            std::vector<unsigned long long> eh(kRegMax * kRegMax);
            QPAT_HIP(c, hipMemcpyAsync(eh.data(), eint, eh.size() * sizeof(unsigned long long), hipMemcpyDeviceToHost,
                                       st));
            QPAT_HIP(c, hipStreamSynchronize(st));
            std::vector<double> E((size_t)k * k);
            for (int i = 0; i < k; ++i)
                for (int j = 0; j < k; ++j)
                    E[(size_t)i * k + j] = static_cast<double>(static_cast<long long>(eh[i * kRegMax + j])) / scale;
            if (!spd_inverse(E, k)) k = 0;   // not positive definite in fixed point: no region space
            for (int i = 0; i < k; ++i) {
                size_h[sys * kRegMax + i] = cand[i].first;
                for (int j = 0; j < k; ++j) einv_h[(sys * kRegMax + i) * kRegMax + j] = E[(size_t)i * k + j];
            }
        } else {
            k = 0;
        }
        if (k == 0) hipLaunchKernelGGL(k_reg_assign, g, b, 0, st, lab, N, 0, roots, M.reg + sys * N);
        M.nreg[sys] = k;
        M.kreg = std::max(M.kreg, k);
    }
    QPAT_HIP(c, hipMemcpyAsync(M.einv, einv_h.data(), einv_h.size() * sizeof(double), hipMemcpyHostToDevice, st));
    QPAT_HIP(c, hipMemcpyAsync(M.rsize, size_h.data(), size_h.size() * sizeof(double), hipMemcpyHostToDevice, st));
    QPAT_HIP(c, hipGetLastError());
    QPAT_HIP(c, hipStreamSynchronize(st));
    return QPAT_OK;
}

// Inverse of the coarsest level's SPD matrix by the sweep operator
// (Gauss-Jordan elimination without pivoting) taken kGj pivots at a time: with
// D = S_KK the block of pivots,
//   T_KK = -D^{-1}, T_IK = S_IK D^{-1}, T_KJ = D^{-1} S_KJ, T_IJ = S_IJ - S_IK D^{-1} S_KJ,
// and after every block the matrix is minus its inverse. Every pivot is a
// Schur-complement diagonal, so positive for an SPD matrix; one that is not
// sets bad[sys].
// A block owns a kGj x kGj tile and forms it with FP64 MFMAs, one 16 x 16
// quadrant a wavefront; the block of the next pivots' tile then inverts it, so
// a step is one launch and one block's inversion (every block inverting D for
// itself made a step of order 729 18 us, of which 11 were the inversions).
// Order 729: 24 launches; one launch a pivot (729 of them, 4.1 us each) took 3 ms
// of every forward solve's set-up.
constexpr int kGj = 32;
typedef double mg_d4 __attribute__((ext_vector_type(4)));

// quadrant (qr, qc) of X Y for two kGj x kGj tiles in LDS; the 16x16x4 FP64 MFMA takes
// A[l % 16][l / 16], B[l / 16][l % 16] from lane l and leaves D[l / 16 + 4 q][l % 16]
__device__ __forceinline__ mg_d4 gj_product(const double (*X)[kGj + 1], const double (*Y)[kGj + 1], int qr, int qc,
                                            mg_d4 acc) {
    const int lane = threadIdx.x & 63, i = lane % 16, k = lane / 16;
#pragma unroll
    for (int kk = 0; kk < kGj; kk += 4)
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(X[16 * qr + i][kk + k], Y[kk + k][16 * qc + i], acc, 0, 0, 0);
    return acc;
}

// A 16 x 16 symmetric positive definite tile to its inverse by one wavefront,
// in the registers a MFMA leaves it in (lane l: rows l / 16 + 4 q of column
// l % 16): Gauss-Jordan elimination, the pivot's column by row broadcasts, its
// row by one permute. False where a pivot is not positive.
template <int K>
__device__ __forceinline__ void gj16_pivot(double (&a)[4], bool& ok) {
    constexpr int gk = K % 4, qk = K / 4;   // row K: lanes 16 gk ..., element qk
    const int g = (threadIdx.x & 63) >> 4, c = threadIdx.x & 15;
    const double rk = __shfl(a[qk], gk * 16 + c);
    const uint64_t bits = __builtin_bit_cast(uint64_t, a[qk]);
    const uint32_t lo = __builtin_amdgcn_readlane(static_cast<uint32_t>(bits), gk * 16 + K);
    const uint32_t hi = __builtin_amdgcn_readlane(static_cast<uint32_t>(bits >> 32), gk * 16 + K);
    const double p = __builtin_bit_cast(double, static_cast<uint64_t>(hi) << 32 | lo);
    const double inv = 1.0 / p, r = rk * inv;
    ok = ok && p > 0.0 && std::isfinite(inv);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const double ck = row_bcast<K>(a[q]);
        const double other = c == K ? -ck * inv : a[q] - ck * r;
        a[q] = q == qk && g == gk ? (c == K ? inv : r) : other;
    }
}
template <int... K>
__device__ __forceinline__ bool gj16(double (&a)[4], std::integer_sequence<int, K...>) {
    bool ok = true;
    (gj16_pivot<K>(a, ok), ...);
    return ok;
}

// D[0] to -D[0]^{-1} by a block, d the thread's four elements of it. One
// wavefront does it with nobody to wait for: the inverse of the upper left
// 16 x 16 tile, the Schur complement's, and the products between them by MFMA,
// the tiles passing through LDS (32 pivots with a block barrier for every two
// were most of a step's 14.6 us; 11.5 now).
__device__ __forceinline__ bool gj_invert(double (&D)[2][kGj][kGj + 1], double (&d)[4]) {
    const int r0 = threadIdx.x / 8, c0 = threadIdx.x % 8 * 4;
    bool ok = true;
    if (threadIdx.x < 64) {
        const int g = threadIdx.x >> 4, c = threadIdx.x & 15;
        const auto pass = [] {   // the wavefront's LDS writes are seen by its other lanes
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        };
        using Pivots = std::make_integer_sequence<int, 16>;
        double i11[4], i22[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) i11[q] = D[0][g + 4 * q][c];
        ok = gj16(i11, Pivots{});
#pragma unroll
        for (int q = 0; q < 4; ++q) D[1][g + 4 * q][c] = i11[q];
        pass();
        mg_d4 w = {0.0, 0.0, 0.0, 0.0}, s, z = {0.0, 0.0, 0.0, 0.0}, t;   // W = A_21 A_11^{-1}
#pragma unroll
        for (int k = 0; k < 16; k += 4) w = __builtin_amdgcn_mfma_f64_16x16x4f64(D[0][16 + c][k + g], D[1][k + g][c], w, 0, 0, 0);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            D[1][16 + g + 4 * q][c] = w[q];
            s[q] = D[0][16 + g + 4 * q][16 + c];
        }
        pass();
#pragma unroll
        for (int k = 0; k < 16; k += 4)   // the Schur complement A_22 - W A_12
            s = __builtin_amdgcn_mfma_f64_16x16x4f64(-D[1][16 + c][k + g], D[0][k + g][16 + c], s, 0, 0, 0);
#pragma unroll
        for (int q = 0; q < 4; ++q) i22[q] = s[q];
        ok = gj16(i22, Pivots{}) && ok;
#pragma unroll
        for (int q = 0; q < 4; ++q) D[1][16 + g + 4 * q][16 + c] = i22[q];
        pass();
#pragma unroll
        for (int k = 0; k < 16; k += 4)   // Z = (Schur complement)^{-1} W
            z = __builtin_amdgcn_mfma_f64_16x16x4f64(D[1][16 + c][16 + k + g], D[1][16 + k + g][c], z, 0, 0, 0);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            D[0][16 + g + 4 * q][c] = z[q];
            D[0][c][16 + g + 4 * q] = z[q];
            D[0][16 + g + 4 * q][16 + c] = -i22[q];
            t[q] = -i11[q];
        }
        pass();
#pragma unroll
        for (int k = 0; k < 16; k += 4)   // -A_11^{-1} - W^T Z
            t = __builtin_amdgcn_mfma_f64_16x16x4f64(-D[1][16 + k + g][c], D[0][16 + k + g][c], t, 0, 0, 0);
#pragma unroll
        for (int q = 0; q < 4; ++q) D[0][g + 4 * q][c] = t[q];
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 4; ++q) d[q] = D[0][r0][c0 + q];
    static_assert(kGj == 32, "two tiles of 16");
    return ok;
}

// P[sys] = -D^{-1} of the first block of pivots (beyond n: an identity block)
__global__ __launch_bounds__(kMgT) void k_gj_first(const double* __restrict__ Sall, int n, double* __restrict__ P,
                                                   int* __restrict__ bad) {
    __shared__ double D[2][kGj][kGj + 1];
    const int sys = blockIdx.x, r0 = threadIdx.x / 8, c0 = threadIdx.x % 8 * 4;
    double d[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int c = c0 + q;
        D[0][r0][c] = r0 < n && c < n ? Sall[((int64_t)sys * n + r0) * n + c] : (r0 == c ? 1.0 : 0.0);
    }
    __syncthreads();
    if (!gj_invert(D, d) && threadIdx.x == 0) bad[sys] = 1;
#pragma unroll
    for (int q = 0; q < 4; ++q) P[(sys * kGj + r0) * kGj + c0 + q] = d[q];
}

// step K from S to T with P = -D^{-1} of its pivots; leaves the next step's in Pn
__global__ __launch_bounds__(kMgT) void k_gj(const double* __restrict__ Sall, double* __restrict__ Tall, int n, int K,
                                             const double* __restrict__ Pall, double* __restrict__ Pn,
                                             int* __restrict__ bad) {
    __shared__ double D[2][kGj][kGj + 1], X[kGj][kGj + 1], Y[kGj][kGj + 1];
    const int I = blockIdx.y, J = blockIdx.x, sys = blockIdx.z;
    const int64_t nn = (int64_t)n * n;
    const double* S = Sall + sys * nn;
    double* T = Tall + sys * nn;
    auto at = [&](int r, int c) { return r < n && c < n ? S[(int64_t)r * n + c] : 0.0; };
    const int r0 = threadIdx.x / 8, c0 = threadIdx.x % 8 * 4;
    const int wave = threadIdx.x >> 6, qr = wave / 2, qc = wave % 2, lane = threadIdx.x & 63;
    mg_d4 t;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        D[0][r0][c0 + q] = Pall[(sys * kGj + r0) * kGj + c0 + q];
        X[r0][c0 + q] = at(I * kGj + r0, K * kGj + c0 + q);
        Y[r0][c0 + q] = at(K * kGj + r0, J * kGj + c0 + q);
        t[q] = at(I * kGj + 16 * qr + lane / 16 + 4 * q, J * kGj + 16 * qc + lane % 16);
    }
    __syncthreads();
    mg_d4 out;
    if (I == K && J == K) {
#pragma unroll
        for (int q = 0; q < 4; ++q) out[q] = D[0][16 * qr + lane / 16 + 4 * q][16 * qc + lane % 16];
    } else if (I == K) {   // D^{-1} S_KJ
        out = -gj_product(D[0], Y, qr, qc, mg_d4{0.0, 0.0, 0.0, 0.0});
    } else {
        const mg_d4 w = gj_product(X, D[0], qr, qc, mg_d4{0.0, 0.0, 0.0, 0.0});   // -S_IK D^{-1}
        if (J == K) {
            out = -w;
        } else {
#pragma unroll
            for (int q = 0; q < 4; ++q) D[1][16 * qr + lane / 16 + 4 * q][16 * qc + lane % 16] = w[q];
            __syncthreads();   // uniform over the block
            out = gj_product(D[1], Y, qr, qc, t);
        }
    }
    const bool next = I == K + 1 && J == K + 1;
    if (next) __syncthreads();   // D is read no more
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int lr = 16 * qr + lane / 16 + 4 * q, lc = 16 * qc + lane % 16, r = I * kGj + lr, c = J * kGj + lc;
        if (r < n && c < n) T[(int64_t)r * n + c] = out[q];
        if (next) D[0][lr][lc] = r < n && c < n ? out[q] : (lr == lc ? 1.0 : 0.0);
    }
    if (!next) return;
    __syncthreads();
    double d[4];
    if (!gj_invert(D, d) && threadIdx.x == 0) bad[sys] = 1;
#pragma unroll
    for (int q = 0; q < 4; ++q) Pn[(sys * kGj + r0) * kGj + c0 + q] = d[q];
}

// out = -(T + T^T) / 2: the preconditioner must be exactly symmetric
__global__ __launch_bounds__(kMgT) void k_gj_out(const double* __restrict__ T, double* __restrict__ out, int n) {
    const int64_t nn = (int64_t)n * n, e = blockIdx.x * (int64_t)kMgT + threadIdx.x;
    if (e >= nn) return;
    const double* t = T + blockIdx.y * nn;
    out[blockIdx.y * nn + e] = -0.5 * (t[e] + t[(e % n) * n + e / n]);
}

// the coarsest level's 27-point rows as a dense matrix
__global__ __launch_bounds__(kMgT) void k_dense_fill(LvArgs L, double* __restrict__ A) {
    const int64_t n = L.N, e = blockIdx.x * (int64_t)kMgT + threadIdx.x;
    if (e >= n * n) return;
    const int sys = blockIdx.y;
    const double* U = L.U + (int64_t)sys * n * 14;
    const int i = static_cast<int>(e / n), j = static_cast<int>(e % n);
    int ix, iy, iz, jx, jy, jz;
    coords(i, L.nx, L.ny, ix, iy, iz);
    coords(j, L.nx, L.ny, jx, jy, jz);
    const int dx = jx - ix, dy = jy - iy, dz = jz - iz;
    double v = 0.0;
    if (dx >= -1 && dx <= 1 && dy >= -1 && dy <= 1 && dz >= -1 && dz <= 1) {
        const int code = dx + 3 * dy + 9 * dz;   // > 0: an upper entry of row i, < 0: of row j
        v = code >= 0 ? U[(int64_t)i * 14 + code] : U[(int64_t)j * 14 - code];
    }
    A[sys * n * n + e] = v;
}

// The Jacobi weights from the Gershgorin bounds g: on the finest level, on the
// coarse ones. bad[nsys] = 1 where a bound is not positive and finite.
__global__ void k_mg_weights(const uint64_t* __restrict__ gmax, int nsys, int nl, double fine, double coarse,
                             double* __restrict__ w, int* __restrict__ bad) {
    const int i = threadIdx.x;
    if (i >= nsys * nl) return;
    const double g = __longlong_as_double(static_cast<long long>(gmax[i]));
    if (!(g > 0.0) || !std::isfinite(g)) bad[nsys] = 1;
    w[i] = (i % nl == 0 ? fine : coarse) / g;
}

__global__ void k_zero_words(uint32_t* p, int n) {
    if (threadIdx.x < (unsigned)n) p[threadIdx.x] = 0;
}

// M.ainv = the inverses of the coarsest level's systems (asynchronous; M.bad tells)
void dense_spd_inverse(const MgState& M, hipStream_t st) {
    const MgLevel& K = M.lv.back();
    const int n = static_cast<int>(K.N), steps = (n + kGj - 1) / kGj;
    const dim3 ge((unsigned)(((int64_t)n * n + kMgT - 1) / kMgT), (unsigned)M.nsys);
    // the steps alternate between M.ainv and M.ainv_t and end in the latter
    double* src = steps % 2 ? M.ainv : M.ainv_t;
    double* dst = steps % 2 ? M.ainv_t : M.ainv;
    hipLaunchKernelGGL(k_dense_fill, ge, dim3(kMgT), 0, st, lv_args(K), src);
    double* P[2] = {M.apiv, M.apiv + M.nsys * kGj * kGj};
    hipLaunchKernelGGL(k_gj_first, dim3(M.nsys), dim3(kMgT), 0, st, src, n, P[0], M.bad);
    for (int k = 0; k < steps; ++k) {
        hipLaunchKernelGGL(k_gj, dim3(steps, steps, M.nsys), dim3(kMgT), 0, st, src, dst, n, k, P[k & 1], P[~k & 1], M.bad);
        std::swap(src, dst);
    }
    hipLaunchKernelGGL(k_gj_out, ge, dim3(kMgT), 0, st, src, M.ainv, n);
}

// The levels of op's hierarchy and their arrays; *useful = false where the lattice has none
static qpat_status mg_alloc(qpat_ctx* c, Op op, int nsys, MgState& M, bool* useful) {
    *useful = true;
    M.nsys = nsys;
    M.bmax = op == Op::K ? kMaxRhs : 1;
    MgLevel L0;
    L0.nx = c->lat.nx;
    L0.ny = c->lat.ny;
    L0.nz = c->lat.nz;
    L0.N = c->N;
    L0.m = c->lat.m;
    L0.tab = reinterpret_cast<const int4*>(c->lat_tab);
    bool kuhn = c->lat.m == 7;
    for (int j = 0; kuhn && j < 7; ++j)
        kuhn = c->lat.dx[j] == kKx[j] && c->lat.dy[j] == kKy[j] && c->lat.dz[j] == kKz[j];
    L0.kind = kuhn ? 1 : 0;
    M.lv.push_back(L0);
    // stop at the first coarse level small enough for a dense inverse (the
    // levels below it cost a launch each for almost no work)
    while (std::max(M.lv.back().nx, std::max(M.lv.back().ny, M.lv.back().nz)) > kMgCoarse &&
           !(M.lv.size() >= 2 && M.lv.back().N <= kMgDenseK)) {
        const MgLevel& F = M.lv.back();
        MgLevel C;
        C.nx = F.nx > 2 ? F.nx / 2 + 1 : F.nx;
        C.ny = F.ny > 2 ? F.ny / 2 + 1 : F.ny;
        C.nz = F.nz > 2 ? F.nz / 2 + 1 : F.nz;
        if (C.nx == F.nx && C.ny == F.ny && C.nz == F.nz) break;
        C.N = (int64_t)C.nx * C.ny * C.nz;
        C.m = 13;
        C.kind = 2;
        M.lv.push_back(C);
    }
    const int nl = static_cast<int>(M.lv.size());
    const int64_t Nc = M.lv.back().N;
    if (Nc > (op == Op::K ? kMgDenseK : 4096) || nl < 2) {   // no useful hierarchy: keep Jacobi-PCG
        *useful = false;
        return QPAT_OK;
    }
    const int64_t V = (int64_t)nsys * M.bmax;
    for (int l = 0; l < nl; ++l) {
        MgLevel& L = M.lv[l];
        if (l > 0) {
            int32_t tab[4 * 13];
            for (int j = 0; j < 13; ++j) {
                const int code = 14 + j;
                const int dx = code % 3 - 1, dy = (code / 3) % 3 - 1, dz = code / 9 - 1;
                tab[4 * j] = dx;
                tab[4 * j + 1] = dy;
                tab[4 * j + 2] = dz;
                tab[4 * j + 3] = dx + L.nx * (dy + L.ny * dz);
            }
            QPAT_TRY(dalloc(c, &L.tab_own, 13));
            QPAT_HIP(c, hipMemcpyAsync(L.tab_own, tab, sizeof tab, hipMemcpyHostToDevice, c->stream));
            L.tab = L.tab_own;
            QPAT_TRY(dalloc(c, &L.U, nsys * L.N * 14));
            QPAT_TRY(dalloc(c, &L.b, V * L.N));
        }
        QPAT_TRY(dalloc(c, &L.dinv, nsys * L.N));
        QPAT_TRY(dalloc(c, &L.x, V * L.N));
        QPAT_TRY(dalloc(c, &L.t, V * L.N));
        QPAT_TRY(dalloc(c, &L.r, V * L.N));
        if (op == Op::Prior && l + 1 < nl) {
            if (WPack{L.nx, L.ny, L.nz}.size() >= (int64_t(1) << 31))
                return fail(c, QPAT_ERR_ARG, "multigrid: lattice %d x %d x %d too large for the prior's transfers",
                            L.nx, L.ny, L.nz);
            QPAT_TRY(dalloc(c, &L.W, nsys * L.N * 8));
            QPAT_TRY(dalloc(c, &L.Wc, nsys * WPack{L.nx, L.ny, L.nz}.size()));
        }
        if (op == Op::Prior && l == 0 && L.kind == 1) {   // entry-major upper rows (kind 3) and in FP32 (kind 5)
            QPAT_TRY(dalloc(c, &L.Uf, nsys * L.N * kUpRow));
            QPAT_TRY(dalloc(c, &L.Uf32, nsys * L.N * kUpRow));
        }
        if (op == Op::K && l >= 1 && l < kMgMaxLevels && M.bmax == 16 && M.lv[0].kind == 1 &&
            L.N >= kTile27Min && L.N * 32 * (int64_t)sizeof(double) < (int64_t(1) << 31))
            QPAT_TRY(dalloc(c, &L.Uf27p, L.N * 32));
        if (op == Op::Prior && l >= 1 && l + 1 < nl && L.N >= kRow27Min) {   // entry-major rows (kind 4)
            QPAT_TRY(dalloc(c, &L.Uf, nsys * L.N * 27));
            QPAT_TRY(dalloc(c, &L.Uf32, nsys * L.N * 27));   // and in FP32 for the V-cycle (kind 6)
        }
    }
    QPAT_TRY(dalloc(c, &M.w, nsys * nl));
    QPAT_TRY(dalloc(c, &M.gmax, nsys * nl));
    QPAT_TRY(dalloc(c, &M.ainv, nsys * Nc * Nc));
    QPAT_TRY(dalloc(c, &M.ainv_t, nsys * Nc * Nc));
    QPAT_TRY(dalloc(c, &M.apiv, 2 * nsys * kGj * kGj));
    QPAT_TRY(dalloc(c, &M.bad, nsys + 1));
    QPAT_TRY(dalloc(c, &M.pr, V * c->N));
    QPAT_TRY(dalloc(c, &M.pr2, V * c->N));
    QPAT_TRY(dalloc(c, &M.pa, V * c->N));
    QPAT_TRY(dalloc(c, &M.pb, V * c->N));
    QPAT_TRY(dalloc(c, &M.pq, V * c->N));
    QPAT_TRY(dalloc(c, &M.parts, (int64_t)kMgLanes * 4 * kMgBlocks));
    QPAT_TRY(dalloc(c, &M.sc, kMgLanes));
    QPAT_HIP(c, hipMemsetAsync(M.sc, 0, kMgLanes * sizeof(MgScal), c->stream));
    QPAT_HIP(c, hipHostMalloc((void**)&M.sc_host, kMgLanes * sizeof(MgScal), hipHostMallocDefault));
    M.lv[0].b = M.pr;   // the V-cycle acts on the PCG residual
    return QPAT_OK;
}

// Hierarchy for the current operator (after its assembly and stencil form).
// Called after every assembly: when the options turn multigrid off, an older
// hierarchy is marked stale so that turning it on again cannot pick it up.
qpat_status mg_setup(qpat_ctx* c, Op op) {
    MgState*& Mp = state_of(c, op);
    if (Mp) Mp->current = false;
    if (!mg_available(c, op)) return QPAT_OK;
    const int nsys = op == Op::K ? 1 : 2;
    if (!Mp) {
        const size_t mark = c->allocs.size();
        Mp = new MgState();
        bool useful = false;
        const qpat_status st = mg_alloc(c, op, nsys, *Mp, &useful);
        if (st != QPAT_OK || !useful) {   // a whole hierarchy or none (none: Jacobi-PCG)
            mg_drop(c, op);
            QPAT_TRY(dfree_from(c, mark));
            return st;
        }
    }
    MgState& M = *Mp;
    const int nl = static_cast<int>(M.lv.size());
    M.lv[0].U = op == Op::K ? c->KU64 : c->MU64;
    M.opdep = op == Op::Prior;
    if (M.lv[0].Uf) {   // M_delta's walk kernels
        M.lv[0].kind = 1;
        hipLaunchKernelGGL(k_mg_fullrows, dim3(grid_for(M.lv[0].N, kMgT, 4096), nsys), dim3(kMgT), 0, c->stream,
                           lv_args(M.lv[0]), M.lv[0].Uf);
        if (M.lv[0].Uf32)
            hipLaunchKernelGGL(k_to_f32, dim3(grid_for(nsys * M.lv[0].N * kUpRow, kMgT, 4096)), dim3(kMgT), 0,
                               c->stream, M.lv[0].Uf, M.lv[0].Uf32, nsys * M.lv[0].N * kUpRow);
    }
    for (int l = 0; l + 1 < nl; ++l) {
        const MgLevel& F = M.lv[l];
        const MgLevel& C = M.lv[l + 1];
        if (M.opdep) {   // prolongation weights from this level's operator, by parity class
            const dim3 g(grid_for(F.N, kMgT, 4096), nsys);
            hipLaunchKernelGGL(k_mg_pweights<0>, g, dim3(kMgT), 0, c->stream, lv_args(F), F.W);
            hipLaunchKernelGGL(k_mg_pweights<1>, g, dim3(kMgT), 0, c->stream, lv_args(F), F.W);
            hipLaunchKernelGGL(k_mg_pweights<2>, g, dim3(kMgT), 0, c->stream, lv_args(F), F.W);
            hipLaunchKernelGGL(k_mg_pweights<3>, g, dim3(kMgT), 0, c->stream, lv_args(F), F.W);
            // the transfers read the weights in FP32, packed; the Galerkin product
            // below uses the same rounded values, so A_c = P^T A P holds for the P applied
            hipLaunchKernelGGL(k_mg_wpack, g, dim3(kMgT), 0, c->stream, lv_args(F), F.W, F.Wc);
        }
        const dim3 gr((unsigned)((C.N + kRapNodes - 1) / kRapNodes), nsys);
        if (F.m <= 7)
            hipLaunchKernelGGL(k_mg_rap<7>, gr, dim3(kMgT), 0, c->stream, lv_args(F), M.opdep ? F.W : nullptr, C.U, C.nx,
                               C.ny, C.nz);
        else
            hipLaunchKernelGGL(k_mg_rap<13>, gr, dim3(kMgT), 0, c->stream, lv_args(F), M.opdep ? F.W : nullptr, C.U, C.nx,
                               C.ny, C.nz);
    }
    for (int l = 1; l < nl; ++l)
        if (M.lv[l].Uf27p) {
            hipLaunchKernelGGL(k_mg_pairs27, dim3(grid_for(M.lv[l].N * 16, kMgT, 4096)), dim3(kMgT), 0, c->stream,
                               lv_args(M.lv[l]), M.lv[l].Uf27p);
        } else if (M.lv[l].Uf) {
            hipLaunchKernelGGL(k_mg_fullrows27, dim3(grid_for(M.lv[l].N, kMgT, 4096), nsys), dim3(kMgT), 0, c->stream,
                               lv_args(M.lv[l]), M.lv[l].Uf);
            if (M.lv[l].Uf32)
                hipLaunchKernelGGL(k_to_f32, dim3(grid_for(nsys * M.lv[l].N * 27, kMgT, 4096)), dim3(kMgT), 0,
                                   c->stream, M.lv[l].Uf, M.lv[l].Uf32, nsys * M.lv[l].N * 27);
        }
    hipLaunchKernelGGL(k_zero_words, dim3(1), dim3(kMgT), 0, c->stream, reinterpret_cast<uint32_t*>(M.gmax),
                       2 * nsys * nl);
    hipLaunchKernelGGL(k_zero_words, dim3(1), dim3(kMgT), 0, c->stream, reinterpret_cast<uint32_t*>(M.bad), nsys + 1);
    for (int l = 0; l < nl; ++l)
        if (M.lv[l].m <= 7)
            hipLaunchKernelGGL(k_mg_diag<7>, dim3(grid_for(M.lv[l].N, kMgT, kMgBlocks), nsys), dim3(kMgT), 0, c->stream,
                               lv_args(M.lv[l]), M.lv[l].dinv, M.gmax, nl, l);
        else
            hipLaunchKernelGGL(k_mg_diag<13>, dim3(grid_for(M.lv[l].N, kMgT, kMgBlocks), nsys), dim3(kMgT), 0, c->stream,
                               lv_args(M.lv[l]), M.lv[l].dinv, M.gmax, nl, l);
    // finest level, coarse levels; M_delta's (strongly varying diffusivity)
    // take larger weights, still below 2 / g so that the cycle stays SPD
    hipLaunchKernelGGL(k_mg_weights, dim3(1), dim3(kMgT), 0, c->stream, M.gmax, nsys, nl,
                       op == Op::Prior ? 7.0 / 4.0 : 8.0 / 5.0, op == Op::Prior ? 39.0 / 20.0 : 19.0 / 10.0, M.w, M.bad);
    dense_spd_inverse(M, c->stream);
    QPAT_HIP(c, hipGetLastError());
    int bad_h[3] = {0, 0, 0};
    QPAT_HIP(c, hipMemcpyAsync(bad_h, M.bad, (nsys + 1) * sizeof(int), hipMemcpyDeviceToHost, c->stream));
    QPAT_HIP(c, hipStreamSynchronize(c->stream));
    const char* what = op == Op::K ? "K" : "M_delta";
    if (bad_h[nsys]) return fail(c, QPAT_ERR_ARG, "multigrid: non-positive diagonal in %s", what);
    for (int sys = 0; sys < nsys; ++sys)
        if (bad_h[sys]) return fail(c, QPAT_ERR_ARG, "multigrid: coarsest %s is not positive definite", what);
    if (op == Op::Prior) QPAT_TRY(region_setup(c, M));
    if (M.lv[0].Uf && op == Op::Prior) M.lv[0].kind = 3;
    if (M.lv[0].Uf32 && op == Op::Prior) M.lv[0].vkind = 5;   // the V-cycle's sweeps and residuals on FP32 rows
    for (int l = 1; op == Op::Prior && l < nl; ++l) {
        if (M.lv[l].Uf) M.lv[l].kind = 4;
        if (M.lv[l].Uf32) M.lv[l].vkind = 6;   // the V-cycle's sweeps and residuals on FP32 rows
    }
    M.current = true;
    return QPAT_OK;
}

namespace {
// columns col ... of a vector [N][ld], its right-hand sides
template <int B>
struct ColAt {
    const double* x;
    int64_t ld;
    __device__ __forceinline__ TB<B> operator()(int32_t i) const { return vld<TB<B>>(x + i * ld); }
};
template <int B>
__global__ __launch_bounds__(kMgT) void k_mg_apply(LvArgs L, const double* __restrict__ in, int ld,
                                                   double* __restrict__ out, double scale) {
    using T = TB<B>;
    const int v = threadIdx.x % Pk<B>::BV * Pk<B>::V;
    walk<Pk<B>::BV>(L.nx, L.ny, L.nz, [&](int32_t ix, int32_t iy, int32_t iz, int32_t i, int32_t) {
        vst<T>(out + (int64_t)i * B + v, scale * apply<1, B>(L, L.U, ColAt<B>{in + v, ld}, ix, iy, iz, i));
    });
}
}  // namespace

// out [N][B] = scale U in, U a Kuhn stencil form [N][8] of the lattice, in
// [N][ld] (columns col ... col + B - 1; both multiples of B), with the
// LDS-tiled kernel of the K hierarchy's finest level, below 8 right-hand sides
// with the walk kernels' rows. done = false: not available for B.
template <int B>
static qpat_status apply_B(qpat_ctx* c, const double* U, const double* in, int ld, int col, double* out,
                           double scale, bool* done) {
    *done = false;
    MgState* M = state_of(c, Op::K);
    if (!M || !mg_ready(c, Op::K)) return QPAT_OK;
    if constexpr (B < 8) {
        if (M->lv[0].kind != 1) return QPAT_OK;
        LvArgs L = lv_args(M->lv[0]);
        L.U = U;
        hipLaunchKernelGGL(k_mg_apply<B>, sgrid<B>(c->N), dim3(kMgT), 0, c->stream, L, in + col, ld, out, scale);
        QPAT_HIP(c, hipGetLastError());
        *done = true;
    } else {
        QPAT_TRY(tile_setup<B>(c, *M));
        const TileGeo& t = M->tiles[B];
        if (!t.on) return QPAT_OK;
        const MgLevel& L = M->lv[0];
        if ((int64_t)L.nx * L.ny * ld * (int64_t)sizeof(double) >= (int64_t(1) << 31)) return QPAT_OK;
        TileArgs g{};
        g.nx = L.nx;
        g.ny = L.ny;
        g.nz = L.nz;
        g.tiles_x = t.tiles_x;
        g.tiles_y = t.tiles_y;
        g.zc = t.zc;
        g.items = t.items;
        g.ld = ld;
        g.col = col;
        g.scale = scale;
        g.U = U;
        g.in = in;
        g.out = out;
        hipLaunchKernelGGL((k_mg_tile<kTApply, B>), dim3(t.blocks), dim3(MgTile<B>::T), MgTile<B>::LDS, c->stream, g);
        QPAT_HIP(c, hipGetLastError());
        *done = true;
    }
    return QPAT_OK;
}

qpat_status mg_tile_schedule(const qpat_ctx* c, int B, int32_t out[8]) {
    const MgState* M = state_of(const_cast<qpat_ctx*>(c), Op::K);
    if (!M) return QPAT_ERR_STATE;
    const auto it = M->tiles.find(B);
    if (it == M->tiles.end() || !it->second.ready) return QPAT_ERR_STATE;
    const TileGeo& t = it->second;
    out[0] = t.on ? 1 : 0;
    out[1] = t.on ? t.zc : 0;
    out[2] = t.on ? t.zc_model : 0;
    out[3] = t.on ? t.ps_zc : 0;
    out[4] = t.on ? t.ps_zc_model : 0;
    out[5] = out[3];   // one form for both precisions
    out[6] = out[4];
    out[7] = t.tuned ? 1 : 0;
    return QPAT_OK;
}

// whether mg_stencil_apply has the form for fewer than 8 right-hand sides
bool mg_stencil_ready(qpat_ctx* c) { return mg_ready(c, Op::K) && state_of(c, Op::K)->lv[0].kind == 1; }

qpat_status mg_stencil_apply(qpat_ctx* c, int B, const double* U, const double* in, int ld, int col, double* out,
                             double scale, bool* done) {
    switch (B) {
        case 1: return apply_B<1>(c, U, in, ld, col, out, scale, done);
        case 2: return apply_B<2>(c, U, in, ld, col, out, scale, done);
        case 4: return apply_B<4>(c, U, in, ld, col, out, scale, done);
        case 8: return apply_B<8>(c, U, in, ld, col, out, scale, done);
        case 16: return apply_B<16>(c, U, in, ld, col, out, scale, done);
        default: *done = false; return QPAT_OK;
    }
}

// A x = b with the multigrid-preconditioned PCG: b in c->b64 ([nsys][N][B],
// overwritten by its deflated form), x in c->x64 (has_x0: it holds the
// start); for M_delta c->scal[sys].mean receives mean(b)/delta.
qpat_status mg_solve(qpat_ctx* c, Op op, int B, SolveStats* st, bool has_x0) {
    if (B > state_of(c, op)->bmax) return fail(c, QPAT_ERR_ARG, "multigrid: block of %d right-hand sides", B);
    switch (B) {
        case 1: return solve_B<1>(c, op, st, has_x0);
        case 2: return solve_B<2>(c, op, st, has_x0);
        case 4: return solve_B<4>(c, op, st, has_x0);
        case 8: return solve_B<8>(c, op, st, has_x0);
        case 16: return solve_B<16>(c, op, st, has_x0);
        default: return fail(c, QPAT_ERR_ARG, "multigrid: block size %d not supported", B);
    }
}

}  // namespace qpat
