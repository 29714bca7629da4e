// Grid-tiled ILU(0) sweeps for 7-point stencils in natural order.
//
// The solves of eq. (3) on an nx x ny x nz grid: cell (i, j, k) of the
// forward sweep needs (i-1, j, k), (i, j-1, k) and (i, j, k-1); the
// backward sweep the +1 neighbours.  The level of a cell is i + j + k
// (hyperplanes), as in the generic level schedule, but here the grid's
// (j, k) plane is cut into TJ x TK tiles of x-lines and one 64-lane
// wavefront owns a tile, one lane per line.  At step t lane (jj, kk)
// processes i = t - jj - kk, so
//   * (i-1) is the lane's own result of the previous step (a register),
//   * (j-1) and (k-1) are the results of lanes jj-1 and kk-1 of the
//     previous step (a ring in LDS; the factorization moves them across
//     lanes),
//   * only lanes on the tile's low faces need values of neighbouring
//     tiles, which those tiles publish into small per-step face buffers.
// A dependency chain therefore crosses memory only when it crosses a tile
// face: NJ + NK hops per sweep instead of nx + ny + nz levels.  Tiles are
// handed to workgroups in the order of J + K from an atomic counter, so a
// tile's producers are always running already (no deadlock).
//
// Layouts (all step-major per tile in 64-lane planes, so every wavefront
// access of the sweeps is one contiguous row):
//   factors  the 3 bs^2 values of a cell's forward blocks (0: k-1, 1: j-1,
//            2: i-1) at step t of tile T are step T S + t of Lt, in the
//            pieces of StepPlanes; backward blocks (0: i+1, 1: j+1, 2: k+1)
//            likewise in Ut, indexed by the backward step, diagonal-block
//            inverses in Dt;
//   result   yt: the forward result of the cell of lane l at forward step t,
//            read by the backward sweep at its step S - 1 - t;
//   faces    a record of FaceRec per step of a tile: the TK j-face cells
//            (lane kk), then the TJ k-face cells (lane jj), each part padded
//            to whole 16-byte pieces.
// Missing neighbours, idle lanes and steps outside the line hold zero
// factors and zero right-hand sides.  Lanes and steps of a tile that have no
// cell so compute exact zeros, and a real cell multiplies a zero block only by
// one of these or by a halo of zeros: the sweeps need no per-lane predication.
// (A value that is not finite makes NaNs of them, but only where the cells
// beside them depend on that value too.)  Lanes past TJ TK read parts of the
// result ring that nothing wrote, and no lane of the tile reads theirs.
#include <algorithm>
#include <type_traits>

#include "device.hpp"
#include "internal.hpp"

namespace kry {

constexpr int NLOAD = 2;       // DMA loader wavefronts per workgroup
constexpr int GWG = 64 * 8;    // wavefronts of a sweep workgroup (roles below)
constexpr int NFACE = 40;      // >= TJ + TK for every tiling used

// The N values of T that each of the 64 lanes holds in one step, as pieces of
// up to 16 bytes per lane (piece by piece: 64 lanes of W consecutive values),
// so that a lane reads them from LDS in 16-byte instructions: these run at
// 128 bytes a clock against 64 for two 8-byte planes at once (14 KB: 112
// against 228 clocks).  BF16 values are padded to whole 8-byte pieces.
template <typename T, int N>
struct StepPlanes {
    static constexpr int V = 16 / (int)sizeof(T);
    static constexpr int NP = sizeof(T) == 2 ? (N + 3) / 4 * 4 : N;
    static constexpr int SIZE = NP * 64;                    // values per step
    static constexpr int BYTES = SIZE * (int)sizeof(T);
    static_assert(BYTES % 256 == 0, "whole DMA pieces");
    // width of the piece that starts at value b: V while that many are left,
    // then the binary parts of the rest, largest first
    static __host__ __device__ constexpr int width(int b) {
        const int left = NP - b;
        return left >= V ? V : left >= 4 ? 4 : left >= 2 ? 2 : 1;
    }
    // place of value e of a lane within the step (no loops: folds for a
    // constant e)
    static __host__ __device__ constexpr int at(int e, int lane) {
        int b = e / V * V;
        if (width(b) < V) {
            if (e >= b + width(b)) b += width(b);
            if (e >= b + width(b)) b += width(b);
        }
        return b * 64 + lane * width(b) + (e - b);
    }
    template <typename TC, int B = 0>
    static __device__ __forceinline__ void read(const char *p, int lane, TC *v);
};

// values of one step's face record: the j-face part, then the k-face part
template <typename TC, int BS>
struct FaceRec {
    static constexpr int V = 16 / (int)sizeof(TC);
    static __host__ __device__ constexpr int part(int cells) { return (cells * BS + V - 1) / V * V; }
    static __host__ __device__ constexpr int size(int TJ, int TK) { return part(TK) + part(TJ); }
};

// a cell of zeros: the right-hand side of lanes and steps with no cell
static __device__ __align__(16) const double zero_cell[4] = {0.0, 0.0, 0.0, 0.0};

// ---------------------------------------------------------------------------
// setup
// ---------------------------------------------------------------------------
template <int BS>
__global__ void k_grid_pack(GridTiles G, const int *__restrict__ rowptr,
                            const int *__restrict__ col, const int *__restrict__ diag,
                            const double *__restrict__ lu, const double *__restrict__ uinv,
                            double *__restrict__ Lt, double *__restrict__ Ut,
                            double *__restrict__ Dt) {
    constexpr int B2 = BS * BS;
    const int64_t g = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    const int lane = static_cast<int>(g & 63);
    const int64_t rest = g >> 6;
    const int t = static_cast<int>(rest % G.S);
    const int T = static_cast<int>(rest / G.S);
    if (T >= G.ntiles) return;
    const int JK = G.order[T];
    const int jj = lane % G.TJ, kk = lane / G.TJ;
    const int j = (JK & 0xffff) * G.TJ + jj, k = (JK >> 16) * G.TK + kk;
    const bool lane_ok = lane < G.TJ * G.TK && j < G.ny && k < G.nz;
    const int64_t sJ = G.nx, sK = (int64_t)G.nx * G.ny;
    const int64_t step = (int64_t)T * G.S + t;
    using PF = StepPlanes<double, 3 * B2>;
    using PD = StepPlanes<double, B2>;
    double *lf = Lt + step * PF::SIZE;
    double *ub = Ut + step * PF::SIZE;
    double *db = Dt + step * PD::SIZE;
    for (int e = 0; e < 3 * B2; e++) {
        lf[PF::at(e, lane)] = 0.0;
        ub[PF::at(e, lane)] = 0.0;
    }
    for (int e = 0; e < B2; e++) db[PD::at(e, lane)] = 0.0;
    // forward cell of this step
    const int i = t - jj - kk;
    if (lane_ok && i >= 0 && i < G.nx) {
        const int64_t c = i + sJ * j + sK * k;
        for (int p = rowptr[c]; p < diag[c]; p++) {
            const int64_t cc = col[p];
            const int b = cc == c - sK ? 0 : (cc == c - sJ ? 1 : 2);
            for (int e = 0; e < B2; e++) lf[PF::at(b * B2 + e, lane)] = lu[(int64_t)p * B2 + e];
        }
    }
    // backward cell of this step
    const int ib = G.nx - 1 - (t - (G.TJ - 1 - jj) - (G.TK - 1 - kk));
    if (lane_ok && ib >= 0 && ib < G.nx) {
        const int64_t c = ib + sJ * j + sK * k;
        for (int p = diag[c] + 1; p < rowptr[c + 1]; p++) {
            const int64_t cc = col[p];
            const int b = cc == c + 1 ? 0 : (cc == c + sJ ? 1 : 2);
            for (int e = 0; e < B2; e++) ub[PF::at(b * B2 + e, lane)] = lu[(int64_t)p * B2 + e];
        }
        for (int e = 0; e < B2; e++) db[PD::at(e, lane)] = uinv[c * B2 + e];
    }
}

// FP64 planes of `steps` steps rounded to FP32 or BF16 planes
template <typename T, int N>
__global__ __launch_bounds__(256) void k_grid_round(int64_t steps, const double *__restrict__ x,
                                                    T *__restrict__ y) {
    using PS = StepPlanes<double, N>;
    using PD = StepPlanes<T, N>;
    const int lane = threadIdx.x & 63;
    for (int64_t s = blockIdx.x * 4 + (threadIdx.x >> 6); s < steps; s += (int64_t)gridDim.x * 4) {
        const double *xs = x + s * PS::SIZE;
        T *ys = y + s * PD::SIZE;
#pragma unroll
        for (int e = 0; e < PD::NP; e++) {
            const float f = e < N ? static_cast<float>(xs[PS::at(e, lane)]) : 0.0f;
            if constexpr (sizeof(T) == 2) ys[PD::at(e, lane)] = f32_to_bf16_rne(f);
            else ys[PD::at(e, lane)] = f;
        }
    }
}
template <typename T>
static void launch_round(hipStream_t s, int bs, bool diag, int64_t steps, const double *x, T *y) {
    const dim3 g(2048), b(256);
    if (bs == 1 && diag) hipLaunchKernelGGL((k_grid_round<T, 1>), g, b, 0, s, steps, x, y);
    else if (bs == 1) hipLaunchKernelGGL((k_grid_round<T, 3>), g, b, 0, s, steps, x, y);
    else if (diag) hipLaunchKernelGGL((k_grid_round<T, 9>), g, b, 0, s, steps, x, y);
    else hipLaunchKernelGGL((k_grid_round<T, 27>), g, b, 0, s, steps, x, y);
}

template <typename T>
__global__ void k_grid_fill_sentinel(int64_t n, T *__restrict__ y) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        y[i] = sentinel_value<T>();
}

// ---------------------------------------------------------------------------
// grid-tiled numeric factorization (nx >= 3 and ny >= 3)
// ---------------------------------------------------------------------------
// For a 7-point stencil in natural order with nx, ny >= 3, ILU(0) changes
// only the diagonal blocks: no product L_ik U_kj of the elimination lands on
// an off-diagonal entry of row i, so
//   D_c = A_cc - sum over the lower neighbours n of (A_cn D_n^-1) A_nc,
// with the neighbours taken in column order (k-1, j-1, i-1) as the
// row-wise elimination takes them.  The kernel walks the forward
// hyperplanes like the forward sweep (one wavefront per tile, one lane per
// x-line), takes D_n^-1 of i-1 from the lane's previous step, of j-1 and
// k-1 from neighbouring lanes or from the face entries published by the
// upstream tiles, and writes the packed sweep layout directly:
// Lt = A_cn D_n^-1, Dt = D_c^-1 (Ut, the upper blocks of A, needs no order:
// grid_upper_body).
//
// Bound by the chain of steps: what a step waits for counts, and the one
// wavefront's own loads (a row's blocks lie apart, so each load instruction
// takes 64 requests).  The blocks of step t + 1 are loaded while step t's
// stores drain and the next faces are polled, their places follow from the
// stencil (row_start), and both upstream tiles are polled at once; Ut is left
// to a launch of its own.  Measured at 64x64x64, 3x3 blocks: 1485 -> 1028 us
// (5.4 us a step) and 31 us for Ut; with Ut here 1251 us.  Waiting for rowptr,
// then for the blocks, then for one face after the other took 7.8 us a step.

// where row (0, j, k) of a full 7-point stencil in natural order starts: seven
// entries per row before it, less those that the grid's faces cut off
__device__ __forceinline__ int row_start(int nx, int ny, int nz, int j, int k) {
    const int64_t line = j + (int64_t)ny * k, plane = (int64_t)nx * ny, c = nx * line;
    const int64_t cut = 2 * line                                     // i = 0, i = nx - 1
                        + (int64_t)nx * (k + (j > 0))                // j = 0
                        + (int64_t)nx * k                            // j = ny - 1
                        + (k > 0 ? plane : c)                        // k = 0
                        + (k == nz - 1 ? c - plane * (nz - 1) : 0);  // k = nz - 1
    return static_cast<int>(7 * c - cut);
}

template <int BS>
__device__ __forceinline__ void load_block(const double *__restrict__ val, int64_t p, double (&x)[BS * BS]) {
#pragma unroll
    for (int e = 0; e < BS * BS; e++) x[e] = val[p * (BS * BS) + e];
}

template <int BS>
__device__ __forceinline__ void grid_factor_body(const GridTiles &G, const double *__restrict__ val,
                                                 double *__restrict__ Lt, double *__restrict__ Dt,
                                                 double *faces, int *ctr, int *err) {
    constexpr int B2 = BS * BS;
    using PF = StepPlanes<double, 3 * B2>;
    using PD = StepPlanes<double, B2>;
    const int lane = threadIdx.x;
    const int TJ = G.TJ, TK = G.TK, NF = G.NF, nx = G.nx, ny = G.ny, nz = G.nz, S = G.S;
    const int jj = lane % TJ, kk = lane / TJ;
    const int fj = jj == TJ - 1 && kk < TK ? kk : -1;       // published face entries
    const int fk = kk == TK - 1 ? TK + jj : -1;
    for (;;) {
        int t0 = 0;
        if (lane == 0) t0 = atomicAdd(ctr, 1);
        const int T = __shfl(t0, 0, 64);
        if (T >= G.ntiles) break;
        const int JK = G.order[T];
        const int J = JK & 0xffff, K = JK >> 16;
        const int j = J * TJ + jj, k = K * TK + kk;
        const bool lane_ok = lane < TJ * TK && j < ny && k < nz;
        // face cells of step 0 of the upstream tiles
        const bool from_j = jj == 0 && J > 0 && lane_ok, from_k = kk == 0 && K > 0 && lane_ok;
        const int64_t srcj = from_j ? ((int64_t)G.tidx[(J - 1) * G.NK + K] * S + (TJ - 1)) * NF + kk : -1;
        const int64_t srck = from_k ? ((int64_t)G.tidx[J * G.NK + K - 1] * S + (TK - 1)) * NF + TK + jj : -1;
        double *frow = faces + (int64_t)T * S * NF * B2;
        // blocks of the step's cell: lower (k-1, j-1, i-1), diagonal, and the
        // blocks A_nc of its lower neighbours
        double al[3][B2], ad[B2], an[3][B2];
        // starts of the rows of the next cell to load and of its lower
        // neighbours (k-1, j-1, i-1); rowlen: entries of a row but i-1, i+1
        const bool up_j = j < ny - 1, up_k = k < nz - 1;
        int pc = 0, pk = 0, pj = 0, pi = 0;
        if (lane_ok) {
            pc = row_start(nx, ny, nz, j, k);
            if (k > 0) pk = row_start(nx, ny, nz, j, k - 1);
            if (j > 0) pj = row_start(nx, ny, nz, j - 1, k);
        }
        const int rowlen = 1 + (j > 0) + up_j + (k > 0) + up_k;
        const int rowlen_k = 1 + (j > 0) + up_j + (k > 1) + 1, rowlen_j = 1 + (j > 1) + 1 + (k > 0) + up_k;
        auto load_cell = [&](int t) {
            const int i = t - jj - kk;
            if (!lane_ok || i < 0 || i >= nx) return;
            const int lo_i = i > 0, up_i = i < nx - 1;
            int64_t p = pc;
            // A_nc sits in row n after n's lower blocks, its diagonal and
            // the upper neighbours of n that precede this cell
            if (k > 0) {
                load_block<BS>(val, p++, al[0]);
                load_block<BS>(val, pk + (k > 1) + (j > 0) + lo_i + 1 + up_i + up_j, an[0]);
            }
            if (j > 0) {
                load_block<BS>(val, p++, al[1]);
                load_block<BS>(val, pj + (k > 0) + (j > 1) + lo_i + 1 + up_i, an[1]);
            }
            if (i > 0) {
                load_block<BS>(val, p++, al[2]);
                load_block<BS>(val, pi + (k > 0) + (j > 0) + (i > 1) + 1, an[2]);
            }
            load_block<BS>(val, p, ad);
            pi = pc;
            pc += rowlen + lo_i + up_i;
            pk += rowlen_k + lo_i + up_i;
            pj += rowlen_j + lo_i + up_i;
        };
        load_cell(0);
        double dp[B2];
#pragma unroll
        for (int e = 0; e < B2; e++) dp[e] = 0.0;
        for (int t = 0; t < S; t++) {
            const int i = t - jj - kk;
            const bool valid = lane_ok && i >= 0 && i < nx;
            // D^-1 of the lower neighbours: (k-1, j-1, i-1)
            double dn[3][B2];
#pragma unroll
            for (int e = 0; e < B2; e++) {
                dn[0][e] = __shfl_up(dp[e], TJ, 64);
                dn[1][e] = __shfl_up(dp[e], 1, 64);
                dn[2][e] = dp[e];
            }
            if (valid && (from_j || from_k)) {
                const int64_t cells[2] = {from_k ? srck + (int64_t)t * NF : -1, from_j ? srcj + (int64_t)t * NF : -1};
                double f[2][B2];
                wait_cells<double, B2, 2>(faces, cells, f, err);
#pragma unroll
                for (int e = 0; e < B2; e++) {
                    if (from_k) dn[0][e] = f[0][e];
                    if (from_j) dn[1][e] = f[1][e];
                }
            }
            double L[3][B2], R[B2];
#pragma unroll
            for (int e = 0; e < B2; e++) {
                R[e] = 0.0;
#pragma unroll
                for (int b = 0; b < 3; b++) L[b][e] = 0.0;
            }
            if (valid) {
                const bool has[3] = {k > 0, j > 0, i > 0};
                // D = A_cc minus L A_nc in column order, L = A_cn D_n^-1
                double D[B2];
#pragma unroll
                for (int e = 0; e < B2; e++) D[e] = ad[e];
#pragma unroll
                for (int b = 0; b < 3; b++) {
                    if (!has[b]) continue;
#pragma unroll
                    for (int r = 0; r < BS; r++)
#pragma unroll
                        for (int cc = 0; cc < BS; cc++) {
                            double sacc = 0.0;
#pragma unroll
                            for (int m = 0; m < BS; m++) sacc += al[b][r * BS + m] * dn[b][m * BS + cc];
                            L[b][r * BS + cc] = sacc;
                        }
#pragma unroll
                    for (int r = 0; r < BS; r++)
#pragma unroll
                        for (int cc = 0; cc < BS; cc++) {
                            double sacc = 0.0;
#pragma unroll
                            for (int m = 0; m < BS; m++) sacc += L[b][r * BS + m] * an[b][m * BS + cc];
                            D[r * BS + cc] -= sacc;
                        }
                }
                if (!dev_block_inverse<BS>(D, R)) {
                    __hip_atomic_store(err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
                    for (int e = 0; e < B2; e++) R[e] = 0.0;
                }
            }
            if (fj >= 0)
#pragma unroll
                for (int e = 0; e < B2; e++) publish<double>(frow + ((int64_t)t * NF + fj) * B2 + e, R[e]);
            if (fk >= 0)
#pragma unroll
                for (int e = 0; e < B2; e++) publish<double>(frow + ((int64_t)t * NF + fk) * B2 + e, R[e]);
            // forward blocks of this step (zeros for idle lanes and steps)
            // and the inverse, at the backward step
            double *lf = Lt + ((int64_t)T * S + t) * PF::SIZE;
#pragma unroll
            for (int b = 0; b < 3; b++)
#pragma unroll
                for (int e = 0; e < B2; e++) lf[PF::at(b * B2 + e, lane)] = L[b][e];
            if (valid) {
                const int tb = (nx - 1 - i) + (TJ - 1 - jj) + (TK - 1 - kk);
                double *db = Dt + ((int64_t)T * S + tb) * PD::SIZE;
#pragma unroll
                for (int e = 0; e < B2; e++) db[PD::at(e, lane)] = R[e];
            }
            if (t + 1 < S) load_cell(t + 1);
#pragma unroll
            for (int e = 0; e < B2; e++) dp[e] = R[e];
        }
    }
}

// Ut = the upper blocks of A: one wavefront per tile and backward step, four
// steps to a workgroup of the grid's nwg
template <int BS>
__device__ __forceinline__ void grid_upper_body(const GridTiles &G, const double *__restrict__ val,
                                                double *__restrict__ Ut, int wg, int nwg) {
    constexpr int B2 = BS * BS;
    using PF = StepPlanes<double, 3 * B2>;
    const int lane = threadIdx.x & 63, jj = lane % G.TJ, kk = lane / G.TJ;
    const int64_t steps = (int64_t)G.ntiles * G.S;
    for (int64_t u = wg * (int64_t)4 + (threadIdx.x >> 6); u < steps; u += (int64_t)nwg * 4) {
        const int JK = G.order[u / G.S], t = (int)(u % G.S);
        const int j = (JK & 0xffff) * G.TJ + jj, k = (JK >> 16) * G.TK + kk;
        const int i = G.nx - 1 - (t - (G.TJ - 1 - jj) - (G.TK - 1 - kk));
        if (lane >= G.TJ * G.TK || j >= G.ny || k >= G.nz || i < 0 || i >= G.nx) continue;
        const bool up_j = j < G.ny - 1, up_k = k < G.nz - 1;
        const int low = (j > 0) + (k > 0);
        // the row's start, then its lower blocks and its diagonal
        int64_t p = row_start(G.nx, G.ny, G.nz, j, k) + (int64_t)i * (1 + low + up_j + up_k) + (i > 0 ? 2 * i - 1 : 0);
        p += low + (i > 0) + 1;
        double *ub = Ut + u * PF::SIZE;
        const bool has[3] = {i < G.nx - 1, up_j, up_k};
#pragma unroll
        for (int b = 0; b < 3; b++)
            if (has[b]) {
                double x[B2];
                load_block<BS>(val, p++, x);
#pragma unroll
                for (int e = 0; e < B2; e++) ub[PF::at(b * B2 + e, lane)] = x[e];
            }
    }
}

template <int BS>
__global__ __launch_bounds__(256) void k_grid_upper(GridTiles G, const double *__restrict__ val,
                                                    double *__restrict__ Ut) {
    grid_upper_body<BS>(G, val, Ut, blockIdx.x, gridDim.x);
}

template <int BS>
__global__ __launch_bounds__(64) void k_grid_factor(GridTiles G, const double *__restrict__ val,
                                                    double *__restrict__ Lt, double *__restrict__ Dt,
                                                    double *faces, int *ctr, int *err) {
    grid_factor_body<BS>(G, val, Lt, Dt, faces, ctr, err);
}

// A pointer read from a descriptor, as an offset from `origin`, a kernel
// argument that is null: derived from a kernel argument, its accesses are
// global instructions; those of a pointer read from memory are flat ones,
// which also wait on the LDS counter.
template <typename T>
__device__ __forceinline__ T *as_global(char *origin, T *p) {
    return reinterpret_cast<T *>(origin + reinterpret_cast<uintptr_t>(p));
}
__device__ __forceinline__ void globalize(char *origin, GridTiles &G) {
    G.order = as_global(origin, const_cast<int *>(G.order));
    G.tidx = as_global(origin, const_cast<int *>(G.tidx));
    G.qtiles = as_global(origin, const_cast<int *>(G.qtiles));
    G.qjk = as_global(origin, const_cast<int *>(G.qjk));
    G.qoff = as_global(origin, const_cast<int *>(G.qoff));
}

// the factorizations of several independent grids in one launch: grid g
// owns the workgroups [wg0, next wg0)
template <int BS>
__global__ __launch_bounds__(64) void k_grid_factor_multi(const FactorMulti *__restrict__ d,
                                                          int ngrid, int *err, char *origin) {
    int g = 0;
    while (g + 1 < ngrid && (int)blockIdx.x >= d[g + 1].wg0) g++;
    FactorMulti D = d[g];
    globalize(origin, D.G);
    grid_factor_body<BS>(D.G, as_global(origin, const_cast<double *>(D.val)), as_global(origin, D.lt),
                         as_global(origin, D.dt), as_global(origin, D.faces), as_global(origin, D.ctr), err);
}

template <int BS>
__global__ __launch_bounds__(256) void k_grid_upper_multi(const FactorMulti *__restrict__ d, int ngrid,
                                                          char *origin) {
    int g = 0;
    while (g + 1 < ngrid && (int)blockIdx.x >= d[g + 1].wg0) g++;
    FactorMulti D = d[g];
    globalize(origin, D.G);
    grid_upper_body<BS>(D.G, as_global(origin, const_cast<double *>(D.val)), as_global(origin, D.ut),
                        blockIdx.x - D.wg0, (g + 1 < ngrid ? d[g + 1].wg0 : (int)gridDim.x) - D.wg0);
}

// tiling of the (j, k) plane and the tile order (J + K diagonals)
static int grid_tiling(const MAT_ *A, IluFactor &F) {
    GridTiles &G = F.G;
    G.nx = A->gnx;
    G.ny = A->gny;
    G.nz = A->gnz;
    G.TJ = std::min(8, G.ny);
    G.TK = std::min(std::min(64 / G.TJ, G.nz), NFACE - G.TJ);
    G.NF = G.TJ + G.TK;
    G.NJ = (G.ny + G.TJ - 1) / G.TJ;
    G.NK = (G.nz + G.TK - 1) / G.TK;
    G.ntiles = G.NJ * G.NK;
    G.S = G.nx + G.TJ + G.TK - 2;
    if (G.NJ > 0xffff || G.NK > 0x7fff) return set_error(KRY_ERR_UNSUPPORTED, "grid too large for tiling");
    std::vector<int> ord, tid(G.ntiles);
    ord.reserve(G.ntiles);
    for (int d = 0; d <= G.NJ + G.NK - 2; d++)
        for (int J = 0; J < G.NJ; J++) {
            const int K = d - J;
            if (K >= 0 && K < G.NK) {
                tid[J * G.NK + K] = static_cast<int>(ord.size());
                ord.push_back(J | (K << 16));
            }
        }
    // queues of tile columns: tiles sharing J (the k-face neighbours) stay
    // on one XCD and exchange faces through its L2
    G.NQ = GRID_QUEUES;
    std::vector<int> qt, qo(G.NQ + 1, 0);
    qt.reserve(G.ntiles);
    for (int q = 0; q < G.NQ; q++) {
        qo[q] = static_cast<int>(qt.size());
        for (int T = 0; T < G.ntiles; T++)
            if (((ord[T] & 0xffff) + F.qrot) % G.NQ == q) qt.push_back(T);
    }
    qo[G.NQ] = static_cast<int>(qt.size());
    G.qmax = 0;
    for (int q = 0; q < G.NQ; q++) G.qmax = std::max(G.qmax, qo[q + 1] - qo[q]);
    KRY_TRY(F.order.alloc(G.ntiles));
    KRY_TRY(F.tidx.alloc(G.ntiles));
    KRY_TRY(F.qtiles.alloc(2 * (size_t)G.ntiles));
    KRY_TRY(F.qoff.alloc(G.NQ + 1));
    KRY_HIP(hipMemcpy(F.order.p, ord.data(), sizeof(int) * G.ntiles, hipMemcpyHostToDevice));
    KRY_HIP(hipMemcpy(F.tidx.p, tid.data(), sizeof(int) * G.ntiles, hipMemcpyHostToDevice));
    for (int e = 0; e < G.ntiles; e++) qt.push_back(ord[qt[e]]);
    KRY_HIP(hipMemcpy(F.qtiles.p, qt.data(), sizeof(int) * 2 * G.ntiles, hipMemcpyHostToDevice));
    KRY_HIP(hipMemcpy(F.qoff.p, qo.data(), sizeof(int) * (G.NQ + 1), hipMemcpyHostToDevice));
    G.order = F.order.p;
    G.tidx = F.tidx.p;
    G.qtiles = F.qtiles.p;
    G.qjk = F.qtiles.p + G.ntiles;
    G.qoff = F.qoff.p;
    const int b2 = A->bs * A->bs;
    const int64_t steps = (int64_t)G.ntiles * G.S;
    KRY_TRY(F.lt64.alloc(steps * 3 * b2 * 64));
    KRY_TRY(F.ut64.alloc(steps * 3 * b2 * 64));
    KRY_TRY(F.dt64.alloc(steps * b2 * 64));
    return KRY_OK;
}

// reduced-precision copies of the FP64 planes, result and face buffers
static int grid_finish(hipStream_t s, const MAT_ *A, IluFactor &F) {
    const GridTiles &G = F.G;
    const int bs = A->bs, b2 = bs * bs;
    const int64_t steps = (int64_t)G.ntiles * G.S;
    const int64_t nlu = steps * 3 * b2 * 64, nd = steps * b2 * 64;
    const int64_t nyt = steps * bs * 64;
    const bool f64 = F.prec == KRY_PREC_F64;
    const int64_t nf = steps * (f64 ? (bs == 1 ? FaceRec<double, 1>::size(G.TJ, G.TK)
                                               : FaceRec<double, 3>::size(G.TJ, G.TK))
                                    : (bs == 1 ? FaceRec<float, 1>::size(G.TJ, G.TK)
                                               : FaceRec<float, 3>::size(G.TJ, G.TK)));
    const dim3 blk(256);
    if (F.prec != KRY_PREC_F64) {
        KRY_TRY(F.dt32.alloc(nd));
        launch_round(s, bs, true, steps, F.dt64.p, F.dt32.p);
        if (F.prec == KRY_PREC_F32) {
            KRY_TRY(F.lt32.alloc(nlu));
            KRY_TRY(F.ut32.alloc(nlu));
            launch_round(s, bs, false, steps, F.lt64.p, F.lt32.p);
            launch_round(s, bs, false, steps, F.ut64.p, F.ut32.p);
        } else {
            const int64_t n16 = steps * (bs == 1 ? StepPlanes<uint16_t, 3>::SIZE
                                                 : StepPlanes<uint16_t, 27>::SIZE);
            KRY_TRY(F.lt16.alloc(n16));
            KRY_TRY(F.ut16.alloc(n16));
            launch_round(s, bs, false, steps, F.lt64.p, F.lt16.p);
            launch_round(s, bs, false, steps, F.ut64.p, F.ut16.p);
        }
        KRY_HIP(hipGetLastError());
        KRY_HIP(hipStreamSynchronize(s));
        F.lt64.release();
        F.ut64.release();
        F.dt64.release();
        // result and face buffers in FP32; faces start out unwritten
        KRY_TRY(F.yt32.alloc(nyt));
        KRY_TRY(F.ff32.alloc(nf));
        KRY_TRY(F.fb32.alloc(nf));
        hipLaunchKernelGGL(k_grid_fill_sentinel<float>, dim3(1024), blk, 0, s, nf, F.ff32.p);
        hipLaunchKernelGGL(k_grid_fill_sentinel<float>, dim3(1024), blk, 0, s, nf, F.fb32.p);
    } else {
        KRY_TRY(F.yt64.alloc(nyt));
        KRY_TRY(F.ff64.alloc(nf));
        KRY_TRY(F.fb64.alloc(nf));
        hipLaunchKernelGGL(k_grid_fill_sentinel<double>, dim3(1024), blk, 0, s, nf, F.ff64.p);
        hipLaunchKernelGGL(k_grid_fill_sentinel<double>, dim3(1024), blk, 0, s, nf, F.fb64.p);
    }
    KRY_HIP(hipGetLastError());
    F.grid = true;
    return KRY_OK;
}

int ilu_grid_setup(hipStream_t s, const MAT_ *A, const double *lu, const double *uinv,
                   IluFactor &F) {
    KRY_TRY(grid_tiling(A, F));
    const GridTiles &G = F.G;
    const int64_t steps = (int64_t)G.ntiles * G.S;
    const dim3 g((steps * 64 + 255) / 256), blk(256);
    if (A->bs == 1)
        hipLaunchKernelGGL(k_grid_pack<1>, g, blk, 0, s, G, A->rowptr.p, A->col.p, A->diag.p, lu,
                           uinv, F.lt64.p, F.ut64.p, F.dt64.p);
    else
        hipLaunchKernelGGL(k_grid_pack<3>, g, blk, 0, s, G, A->rowptr.p, A->col.p, A->diag.p, lu,
                           uinv, F.lt64.p, F.ut64.p, F.dt64.p);
    KRY_HIP(hipGetLastError());
    return grid_finish(s, A, F);
}

// Allocate a grid factor's tiling, planes, work buffers and tile counters
// for a later factor launch (FP64 only): F is complete once a factor launch
// on `faces` (sentinel-filled, steps * NF * bs^2) and `fctr` (zero) ran.
int grid_factor_prepare(hipStream_t s, const MAT_ *A, IluFactor &F, DBuf<double> &faces,
                        DBuf<int> &fctr) {
    if (!ilu_grid_can_factor(A)) return set_error(KRY_ERR_ARG, "grid factorization needs nx, ny >= 3");
    F.bs = A->bs;
    F.nb = A->nb;
    F.prec = KRY_PREC_F64;
    F.nlev_f = F.nlev_b = A->gnx + A->gny + A->gnz - 2;
    KRY_TRY(grid_tiling(A, F));
    const GridTiles &G = F.G;
    const int64_t steps = (int64_t)G.ntiles * G.S;
    KRY_TRY(faces.alloc(steps * G.NF * A->bs * A->bs));
    KRY_TRY(fctr.alloc(1));
    KRY_TRY(F.ctr.alloc(2 * GRID_QUEUES));
    KRY_HIP(hipMemsetAsync(F.ctr.p, 0, 2 * GRID_QUEUES * sizeof(int), s));
    return grid_finish(s, A, F);
}

// re-arm the work buffers of a prepared factor before a factor launch
int grid_factor_rearm(hipStream_t s, IluFactor &F, DBuf<double> &faces, DBuf<int> &fctr) {
    KRY_HIP(hipMemsetAsync(F.ut64.p, 0, F.ut64.bytes(), s));
    KRY_HIP(hipMemsetAsync(F.dt64.p, 0, F.dt64.bytes(), s));
    hipLaunchKernelGGL(k_grid_fill_sentinel<double>, dim3(1024), dim3(256), 0, s,
                       (int64_t)faces.n, faces.p);
    KRY_HIP(hipMemsetAsync(fctr.p, 0, sizeof(int), s));
    KRY_HIP(hipGetLastError());
    return KRY_OK;
}

int grid_factor_desc(const MAT_ *A, const IluFactor &F, DBuf<double> &faces, DBuf<int> &fctr,
                     int wg0, FactorMulti &d, int *wgs) {
    d.G = F.G;
    d.val = A->val.p;
    d.lt = F.lt64.p;
    d.ut = F.ut64.p;
    d.dt = F.dt64.p;
    d.faces = faces.p;
    d.ctr = fctr.p;
    d.wg0 = wg0;
    *wgs = std::min(F.G.ntiles, 1024);
    return KRY_OK;
}

int grid_factor_multi(hipStream_t s, int bs, const FactorMulti *d_desc, int ngrid, int total_wgs,
                      int *err) {
    TimedScope t("ras_grid_factor", s);
    char *const origin = nullptr;
    if (bs == 1) {
        hipLaunchKernelGGL(k_grid_factor_multi<1>, dim3(total_wgs), dim3(64), 0, s, d_desc, ngrid, err, origin);
        hipLaunchKernelGGL(k_grid_upper_multi<1>, dim3(total_wgs), dim3(256), 0, s, d_desc, ngrid, origin);
    } else {
        hipLaunchKernelGGL(k_grid_factor_multi<3>, dim3(total_wgs), dim3(64), 0, s, d_desc, ngrid, err, origin);
        hipLaunchKernelGGL(k_grid_upper_multi<3>, dim3(total_wgs), dim3(256), 0, s, d_desc, ngrid, origin);
    }
    KRY_HIP(hipGetLastError());
    return KRY_OK;
}

bool ilu_grid_can_factor(const MAT_ *A) {
    return A->gnx >= 3 && A->gny >= 3 && A->gnz >= 1 && (A->bs == 1 || A->bs == 3);
}

int ilu_grid_factor_setup(hipStream_t s, const MAT_ *A, const double *d_val, IluFactor &F,
                          int *d_err) {
    if (!ilu_grid_can_factor(A)) return set_error(KRY_ERR_ARG, "grid factorization needs nx, ny >= 3");
    KRY_TRY(grid_tiling(A, F));
    const GridTiles &G = F.G;
    const int b2 = A->bs * A->bs;
    const int64_t steps = (int64_t)G.ntiles * G.S;
    // backward planes are written only where a cell exists
    KRY_HIP(hipMemsetAsync(F.ut64.p, 0, F.ut64.bytes(), s));
    KRY_HIP(hipMemsetAsync(F.dt64.p, 0, F.dt64.bytes(), s));
    DBuf<double> faces;
    DBuf<int> ctr;
    const int64_t nf = steps * G.NF * b2;
    KRY_TRY(faces.alloc(nf));
    KRY_TRY(ctr.alloc(1));
    hipLaunchKernelGGL(k_grid_fill_sentinel<double>, dim3(1024), dim3(256), 0, s, nf, faces.p);
    KRY_HIP(hipMemsetAsync(ctr.p, 0, sizeof(int), s));
    const int wgs = std::min(G.ntiles, 1024);
    {
        TimedScope t("ilu_grid_factor", s);
        const dim3 gu((unsigned)std::min<int64_t>((steps + 3) / 4, 4096));
        if (A->bs == 1) {
            hipLaunchKernelGGL(k_grid_factor<1>, dim3(wgs), dim3(64), 0, s, G, d_val, F.lt64.p, F.dt64.p,
                               faces.p, ctr.p, d_err);
            hipLaunchKernelGGL(k_grid_upper<1>, gu, dim3(256), 0, s, G, d_val, F.ut64.p);
        } else {
            hipLaunchKernelGGL(k_grid_factor<3>, dim3(wgs), dim3(64), 0, s, G, d_val, F.lt64.p, F.dt64.p,
                               faces.p, ctr.p, d_err);
            hipLaunchKernelGGL(k_grid_upper<3>, gu, dim3(256), 0, s, G, d_val, F.ut64.p);
        }
    }
    KRY_HIP(hipGetLastError());
    // the face buffer and counter are freed on return
    KRY_HIP(hipStreamSynchronize(s));
    return grid_finish(s, A, F);
}

// ---------------------------------------------------------------------------
// sweeps: one workgroup per tile, wavefront-specialised
//   wave 0            compute: consumes one hyperplane step at a time from
//                     LDS and leaves its result in LDS; it touches no global
//                     memory and waits for nothing but its operands
//   waves 1, 7        boundary: poll the face buffers of the two upstream
//                     tiles and stage the values in LDS, steps in turn
//   waves 2, 3        loaders: copy each step's factor planes (and the
//                     forward's right-hand side, the backward's diagonal
//                     inverses and forward result) straight from global
//                     memory into an LDS ring with the gfx950 global-to-LDS
//                     DMA loads, several steps in flight per wavefront and
//                     no register staging; when a tile is done they re-arm
//                     the other sweep's face slots of that tile
//   wave 4            only passes the tile barriers: wavefronts go to the
//                     four SIMDs in turn, and the compute wavefront keeps
//                     its SIMD to itself
//   wave 5            publisher: takes each step's result from LDS and
//                     publishes the face cells; in the forward sweep it
//                     also stores the tile-step rows the backward sweep reads
//   wave 6            forward: copies the right-hand side into its LDS ring;
//                     backward: writer, takes the results of a few steps at
//                     a time from LDS and stores them to the caller's vector
//                     in natural order, with its epilogue
//
// Result ring.  Slot t of YRing holds what step t reads: the tile's results
// of step t - 1 in the interior of a (TK + 1) x (TJ + 1) array of cells, and
// in its first row and column the neighbouring tiles' face values for step
// t, put there by the boundary wavefront.  A lane finds its j- and
// k-neighbours at fixed places of the slot whether they belong to the tile
// or not, so the exchange is two LDS writes and four reads a step with no
// selects, and the same slots feed the publisher and the writer.
//
// What bounds a step: the compute wavefront issues about one instruction
// every four cycles, so the step's length is its instruction count plus the
// LDS round trip of the neighbours' results.
//
// Ring slots carry the step's stamp (a running step count of the
// workgroup), so no slot is ever reset.  LDS operations of one wavefront
// execute in order, so a progress word written after the reads (or writes)
// it stands for needs no wait in between.
// ---------------------------------------------------------------------------
// ring slots for steps of SB bytes in ROOM bytes of LDS (2 to 8)
template <int SB, int ROOM>
constexpr int ring_slots() {
    return (ROOM / SB) > 8 ? 8 : (ROOM / SB) < 2 ? 2 : (ROOM / SB);
}

typedef __attribute__((address_space(3))) void lds_void_t;

// global-to-LDS DMA of a contiguous block of BYTES (a multiple of 256) by
// one wavefront: whole 1 KiB pieces as 16 bytes per lane, then 256-byte
// pieces as 4 bytes per lane.  Lane l of a piece at offset o copies
// src + o + w l to dst + o + w l (w its width; the LDS address of a lane is
// the wave-uniform base plus w l).  Every instruction runs on the whole
// wavefront: the LDS base of an instruction must be wave-uniform, so none
// sits under a lane-dependent branch.  NT: non-temporal loads, for factors
// that stream through once per sweep (a full-chip read of 2 GB runs at 7.3
// TB/s with them, 5.9 without); the scalar factors of CPR's pressure stage,
// swept several times in a row and a ninth of the size, are better left in
// the caches (64^3, FP64: 68 us a sweep against 76 with non-temporal loads).
constexpr int dma_count(int bytes) { return bytes / 1024 + (bytes % 1024) / 256; }
template <int BYTES, bool NT>
__device__ __forceinline__ void dma_block(const void *src, char *dst, int lane) {
    static_assert(BYTES % 256 == 0, "256-byte pieces");
    const char *g = static_cast<const char *>(src);
    constexpr int N16 = BYTES / 1024, N4 = (BYTES % 1024) / 256;
#pragma unroll
    for (int q = 0; q < N16; q++)
        __builtin_amdgcn_global_load_lds(g + q * 1024 + lane * 16, (lds_void_t *)(dst + q * 1024),
                                         16, 0, NT ? 2 : 0);
#pragma unroll
    for (int q = 0; q < N4; q++) {
        const int o = N16 * 1024 + q * 256;
        __builtin_amdgcn_global_load_lds(g + o + lane * 4, (lds_void_t *)(dst + o), 4, 0, NT ? 2 : 0);
    }
}
// W bytes per lane (4 or 12) from each lane's own address into dst + S l,
// S = 4 for dwords and 16 for three-dword pieces (the DMA keeps a 16-byte
// stride per lane for those)
template <int W>
__device__ __forceinline__ void dma_piece(const void *src, char *dst) {
    static_assert(W == 4 || W == 12, "dword or three-dword pieces");
    if constexpr (W == 4)
        __builtin_amdgcn_global_load_lds(src, (lds_void_t *)(dst), 4, 0, 0);
    else
        __builtin_amdgcn_global_load_lds(src, (lds_void_t *)(dst), 12, 0, 0);
}
// wait until at most N vector memory instructions of this wavefront are
// outstanding (they complete in order, so every older one has landed)
template <int N>
__device__ __forceinline__ void wait_vm() {
    static_assert(N >= 0 && N < 64, "vmcnt range");
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}

// value types of the ring: factor storage TF read as the compute type TC
template <typename TC, typename TF>
__device__ __forceinline__ TC cvt(TF v) { return static_cast<TC>(v); }
template <>
__device__ __forceinline__ float cvt<float, uint16_t>(uint16_t v) { return bf16_to_f32(v); }

template <typename T, int N>
template <typename TC, int B>
__device__ __forceinline__ void StepPlanes<T, N>::read(const char *p, int lane, TC *v) {
    if constexpr (B < NP) {
        constexpr int W = width(B);
        const T *q = reinterpret_cast<const T *>(p) + B * 64 + lane * W;
        if constexpr (W == 1) {
            v[B] = cvt<TC, T>(*q);
        } else {
            typedef T vec_t __attribute__((ext_vector_type(W)));
            const vec_t u = *reinterpret_cast<const vec_t *>(q);
#pragma unroll
            for (int i = 0; i < W; i++)
                if (B + i < N) v[B + i] = cvt<TC, T>(u[i]);
        }
        read<TC, B + W>(p, lane, v);
    }
}

// The right-hand side of the forward sweep: a ring of RS_STEPS steps in LDS,
// filled RS_CH steps at a time by a wavefront of its own.  At a step the 64
// lanes read 64 cells of 64 lines far apart in memory; taking RS_CH steps at
// once lets one DMA instruction copy runs of RS_CH consecutive cells of a few
// lines instead of one cell of each line (FP64 blocks: 8 lines of 96 bytes;
// the gather of single cells cost as many memory requests as the factor
// planes, 12% of the sweep at 64^3 and 9% at 256 x 256 x 128).
// A cell is UH units of UB bytes in LDS: 3 doubles two 12-byte pieces (the
// DMA keeps 16 bytes per lane for those), 3 floats one; a double of BS = 1
// two dwords side by side, a float one dword.  Block q of a chunk (one DMA
// instruction, UPI units) holds the lines q LPB .. q LPB + LPB - 1, UL units
// of each in turn (neighbouring lanes copy neighbouring memory; with a
// line's units spread over the block no requests merge and the ring fills
// too slowly).  A line's units are permuted by XOR with `twist`, which puts
// the units that a wavefront reads together (one of every line) on distinct
// banks.  Cells outside the line are copied from a cell of zeros.
constexpr int RS_CH = 4, RS_STEPS = 16;
template <typename TIN, int BS>
struct RhsRing {
    static constexpr int CB = BS * (int)sizeof(TIN);        // bytes of a cell
    static constexpr int UH = CB == 24 ? 2 : 1;
    static constexpr int UB = CB % 12 == 0 ? 16 : CB;       // bytes of a unit in LDS
    static constexpr int LPU = UB == 8 ? 2 : 1;             // DMA lanes per unit
    static constexpr int UPI = 64 / LPU;
    static constexpr int LPB = UPI / (RS_CH * UH);
    static constexpr int UL = RS_CH * UH;                   // units of a line
    static constexpr int NI = 64 / LPB;                     // DMA instructions per chunk
    static constexpr int IB = UPI * UB, CHB = NI * IB, BYTES = (RS_STEPS / RS_CH) * CHB;
    static __device__ __forceinline__ int twist(int q, int r) {   // line r of block q
        return (UB == 16 ? (UL == 8 ? r : r >> 2) : q) & (UL - 1);
    }
    static __device__ __forceinline__ int unit(int lane, int s, int h) {
        const int q = lane / LPB, r = lane % LPB;
        return q * IB + (r * UL + ((s * UH + h) ^ twist(q, r))) * UB;
    }
    // the lane's cell of step t, s = t % RS_CH
    template <typename TC>
    static __device__ __forceinline__ void read(const char *ring, int t, int s, int lane, TC *v) {
        const char *c = ring + ((t / RS_CH) & (RS_STEPS / RS_CH - 1)) * CHB;
        if constexpr (CB == 24) {   // the fourth dword of a piece is never written
            const uint4 a = *reinterpret_cast<const uint4 *>(c + unit(lane, s, 0));
            const uint4 b = *reinterpret_cast<const uint4 *>(c + unit(lane, s, 1));
            v[0] = static_cast<TC>(join(a.x, a.y));
            v[1] = static_cast<TC>(join(a.z, b.x));
            v[2] = static_cast<TC>(join(b.y, b.z));
        } else if constexpr (CB == 12) {
            const uint4 a = *reinterpret_cast<const uint4 *>(c + unit(lane, s, 0));
            v[0] = static_cast<TC>(__uint_as_float(a.x));
            v[1] = static_cast<TC>(__uint_as_float(a.y));
            v[2] = static_cast<TC>(__uint_as_float(a.z));
        } else {
            v[0] = static_cast<TC>(*reinterpret_cast<const TIN *>(c + unit(lane, s, 0)));
        }
    }
    static __device__ __forceinline__ double join(uint32_t lo, uint32_t hi) {
        return __longlong_as_double(static_cast<long long>((static_cast<uint64_t>(hi) << 32) | lo));
    }
};

// LDS flag access from a wavefront with DMA loads in flight.  The
// compiler treats any LDS access as possibly aliasing the DMA's LDS writes
// and would drain every outstanding DMA first; these two touch only the
// flag word, so they are written as single LDS instructions (the read waits
// for its own result inside the same statement).
__device__ __forceinline__ int lds_flag_get(const int *p) {
    const unsigned a = (unsigned)(size_t)((const __attribute__((address_space(3))) int *)p);
    int v;
    asm volatile("ds_read_b32 %0, %1\n\ts_waitcnt lgkmcnt(0)" : "=v"(v) : "v"(a) : "memory");
    return v;
}
__device__ __forceinline__ void lds_flag_put(int *p, int v) {
    const unsigned a = (unsigned)(size_t)((__attribute__((address_space(3))) int *)p);
    asm volatile("ds_write_b32 %0, %1\n\ts_waitcnt lgkmcnt(0)" : : "v"(a), "v"(v) : "memory");
}

// Progress word of a role: every lane writes the value to its own word, so
// the store needs no exec mask and meets no bank conflict; readers take
// word 0.
struct Progress {
    int w[64];
};
__device__ __forceinline__ void progress_put(Progress &p, int lane, int v) {
    const unsigned a = (unsigned)(size_t)((__attribute__((address_space(3))) int *)(p.w + lane));
    asm volatile("ds_write_b32 %0, %1" : : "v"(a), "v"(v) : "memory");
}
__device__ __forceinline__ int progress_get(const Progress &p) {
    return __builtin_amdgcn_readfirstlane(lds_get(const_cast<int *>(p.w)));
}
// wait until the progress word reaches v (it is kept by a wavefront of this
// workgroup that waits only on earlier steps)
__device__ __forceinline__ void progress_wait(const Progress &p, int v, int &seen, int *err) {
#pragma clang loop unroll(disable)
    for (uint32_t it = 0; seen < v; ++it) {
        seen = progress_get(p);
        if (it > 4 * SPIN_LIMIT) {
            __hip_atomic_store(err, ERR_STALL_FLAG, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            break;
        }
    }
    asm volatile("" : : : "memory");
}

// The result ring (see the head of this section): DY slots of CELLS cells.
// A cell's BS values are one 16-byte piece and, for three doubles, an
// 8-byte piece in a second plane, so a cell moves in one or two LDS
// instructions.  CELLS >= (TK + 1)(TJ + 1) for every tiling, idle lanes
// included (at most 99), and makes the slot strides (408 and 204 words) hit
// distinct banks when a wavefront reads a few consecutive slots at once.
template <typename TC, int BS>
struct YRing {
    static constexpr int DY = BS == 1 ? 32 : 16;
    static constexpr int CELLS = 102;
    static constexpr int WA = BS == 3 ? 16 : (int)sizeof(TC);
    static constexpr int WB = BS == 3 && sizeof(TC) == 8 ? 8 : 0;
    static constexpr int BYTES = DY * CELLS * (WA + WB);
    static __device__ __forceinline__ int slot(int t) { return t & (DY - 1); }
    // byte offset of value r of a cell in slot 0, and the slots' stride
    static __device__ __forceinline__ void place(int cell, int r, int &off, int &stride) {
        const bool second = WB != 0 && r == 2;
        off = second ? DY * CELLS * WA + cell * WB : cell * WA + r * (int)sizeof(TC);
        stride = second ? CELLS * WB : CELLS * WA;
    }
    static __device__ __forceinline__ void load(const char *ring, int s, int cell, TC (&v)[BS]) {
        const char *p = ring + s * (CELLS * WA) + cell * WA;
        if constexpr (BS == 1) {
            v[0] = *reinterpret_cast<const TC *>(p);
        } else if constexpr (sizeof(TC) == 8) {
            const double2 a = *reinterpret_cast<const double2 *>(p);
            v[0] = a.x;
            v[1] = a.y;
            v[2] = *reinterpret_cast<const double *>(ring + DY * CELLS * WA + s * (CELLS * WB) + cell * WB);
        } else {
            const float4 a = *reinterpret_cast<const float4 *>(p);
            v[0] = a.x;
            v[1] = a.y;
            v[2] = a.z;
        }
    }
    static __device__ __forceinline__ void store(char *ring, int s, int cell, const TC (&v)[BS]) {
        char *p = ring + s * (CELLS * WA) + cell * WA;
        if constexpr (BS == 1) {
            *reinterpret_cast<TC *>(p) = v[0];
        } else if constexpr (sizeof(TC) == 8) {
            *reinterpret_cast<double2 *>(p) = make_double2(v[0], v[1]);
            *reinterpret_cast<double *>(ring + DY * CELLS * WA + s * (CELLS * WB) + cell * WB) = v[2];
        } else {
            *reinterpret_cast<float4 *>(p) = make_float4(v[0], v[1], v[2], 0.0f);
        }
    }
};

// Stamps of a step slot: .x = boundary staged for step t (slot t), .y =
// planes loaded for step t + 1 (slot t), one 8-byte word so the compute
// wavefront checks both with one read and one compare.
union StepFlag {
    int h[2];
    unsigned long long u;
};
__device__ __forceinline__ unsigned long long step_flag_get(const StepFlag &f) {
    return __hip_atomic_load(const_cast<unsigned long long *>(&f.u), __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_WORKGROUP);
}
// wait for both stamps; pre = the flag read ahead during the previous step
__device__ __forceinline__ void step_wait(unsigned long long pre, const StepFlag &f, int st, int *err) {
    const unsigned long long want =
        (static_cast<unsigned long long>(static_cast<unsigned>(st + 1)) << 32) | static_cast<unsigned>(st);
    if (__builtin_amdgcn_ballot_w64(pre != want) != 0) {
#pragma clang loop unroll(disable)
        for (uint32_t it = 0; __builtin_amdgcn_ballot_w64(step_flag_get(f) != want) != 0; ++it)
            if (it > 4 * SPIN_LIMIT) {
                __hip_atomic_store(err, ERR_STALL_FLAG, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                break;
            }
    }
    asm volatile("" : : : "memory");
}

// Loader loop of one tile: steps t = w, w + NLOAD, ... of S; issue(t) starts
// the DMA of step t into ring slot t % D (P instructions); at most K steps of
// this wavefront in flight; a step is stamped once its DMA landed.  Slot
// t % D is free once the compute wavefront has finished step t - D (its
// planes are read during the step before, those of step 0 before step 0).
// The wait counts assume no other vector memory operation of the wavefront
// is outstanding when the loop starts.
// A step is stamped only when `rhs_p` (where given) shows its right-hand side
// staged too.
template <int D, int P, int K, int DY, typename F>
__device__ __forceinline__ void loader_loop(int w, int S, int base, const Progress &done_p,
                                            const Progress *rhs_p, StepFlag (&fl)[DY], int lane,
                                            int *err, F &&issue) {
    // the wave's vector memory counter holds at most 63 outstanding
    // instructions: every DMA of the K steps in flight must fit in it
    static_assert(K >= 1 && K <= 4 && K * P <= 63, "in-flight DMA within the vmcnt range");
    static_assert(D < DY, "the stamps of the steps in the ring are distinct slots");
    int next = w, done = w, rhs = base;
    uint32_t idle = 0;
    wait_vm<0>();
    while (done < S) {
        while (next < S && next - done < K * NLOAD &&
               (next < D || __builtin_amdgcn_readfirstlane(lds_flag_get(done_p.w)) >=
                                base + (next - D > 1 ? next - D : 1))) {
            issue(next);
            next += NLOAD;
        }
        const int inflight = (next - done) / NLOAD;
        if (inflight == 0) {   // the ring is full: wait for the compute wavefront
            if (++idle > 4 * SPIN_LIMIT) {
                __hip_atomic_store(err, ERR_STALL_FLAG, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                break;
            }
            __builtin_amdgcn_s_sleep(1);
            continue;
        }
        idle = 0;
        // the oldest step's DMA has landed once at most (inflight - 1) * P
        // newer instructions are outstanding
        if constexpr (K >= 4) { if (inflight == 4) wait_vm<(K >= 4 ? 3 * P : 0)>(); }
        if constexpr (K >= 3) { if (inflight == 3) wait_vm<(K >= 3 ? 2 * P : 0)>(); }
        if constexpr (K >= 2) { if (inflight == 2) wait_vm<(K >= 2 ? P : 0)>(); }
        if (inflight == 1) wait_vm<0>();
        if (rhs_p)
#pragma clang loop unroll(disable)
            for (uint32_t it = 0; rhs <= base + done; ++it) {
                rhs = __builtin_amdgcn_readfirstlane(lds_flag_get(rhs_p->w));
                if (it > 4 * SPIN_LIMIT) {
                    __hip_atomic_store(err, ERR_STALL_FLAG, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    break;
                }
            }
        if (lane == 0) lds_flag_put(&fl[(done + DY - 1) & (DY - 1)].h[1], base + done);
        done += NLOAD;
    }
    // the last step has no next planes to wait for: stamp them all the same
    // (step S belongs to wavefront S % NLOAD)
    if (S % NLOAD == w && lane == 0) lds_flag_put(&fl[(S + DY - 1) & (DY - 1)].h[1], base + S);
}

// acc -= B y for block b of the planes in v
template <int BS, typename TC, int NV>
__device__ __forceinline__ void block_sub(TC (&acc)[BS], const TC (&v)[NV], int b, const TC (&y)[BS]) {
#pragma unroll
    for (int r = 0; r < BS; r++)
#pragma unroll
        for (int c = 0; c < BS; c++) acc[r] -= v[b * BS * BS + r * BS + c] * y[c];
}

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
// 16 bytes that see other workgroups' published values (device scope), the
// load waited for in the same statement.
//   The values in them validate themselves one by one, so each has to arrive
// whole: no 8-byte half of a piece may be seen half written.  This is taken
// from the hardware: a lane's piece is aligned to 16 bytes (records are padded
// to whole pieces), so it lies within one cache line and is stored and read by
// one request each.  The programming model promises it for atomic accesses of
// up to 8 bytes alone.
__device__ __forceinline__ u32x4 load_published(const void *a) {
    u32x4 r;
    asm volatile("global_load_dwordx4 %0, %1, off sc1\n\t"
                 "s_waitcnt vmcnt(0)"
                 : "=&v"(r)
                 : "v"(a)
                 : "memory");
    return r;
}
// Lane l's 16 bytes of a record of `bytes` bytes (the same record in every
// lane), device scope.  A buffer store: lanes past the record are dropped by
// its bounds, and the compiler sees it.  It has to, because a vector
// instruction may overwrite the data registers of a 16-byte store only two
// wait states after it.  (As inline assembly with its own wait states: CPR in
// FP32 at 125x97x61 1160 us an application, this way 1150.)
__device__ __forceinline__ void store_published(void *rec, int bytes, int lane, u32x4 v) {
    constexpr int SC1 = 16, RAW = 0x20000;
    __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(rec, 0, bytes, RAW);
    __builtin_amdgcn_raw_buffer_store_b128(v, r, lane * 16, 0, SC1);
}

// What the publisher's lane u holds of a step's face record: 16 bytes of it
// (lanes past the record hold none), gathered from the result ring's cells.
// One store instruction publishes both faces, whole lines at a time: stores
// of single values by the lanes that own the cells touched every line three
// times while the neighbours were polling it.
template <typename TC, int BS, bool REV>
struct FacePublisher {
    using U = typename Bits<TC>::U;
    using YR = YRing<TC, BS>;
    using FR = FaceRec<TC, BS>;
    int off[FR::V], stride[FR::V];
    __device__ __forceinline__ FacePublisher(int TJ, int TK, int lane) {
        const int PJ = FR::part(TK);
        const bool mine = lane * FR::V < FR::size(TJ, TK);
        const bool isj = lane * FR::V < PJ;
        const int e0 = isj ? lane * FR::V : lane * FR::V - PJ;
#pragma unroll
        for (int i = 0; i < FR::V; i++) {
            const int c = (e0 + i) / BS, r = e0 + i - c * BS;
            int cell = YR::CELLS - 1;   // padding: any value will do
            if (mine && isj && c < TK) cell = (REV ? TK - c : c + 1) * (TJ + 1) + TJ;
            if (mine && !isj && c < TJ) cell = TK * (TJ + 1) + (REV ? TJ - c : c + 1);
            YR::place(cell, r, off[i], stride[i]);
        }
    }
    // this lane's piece of the results in ring slot s
    __device__ __forceinline__ u32x4 gather(const char *ring, int s) const {
        U w[FR::V];
#pragma unroll
        for (int i = 0; i < FR::V; i++) w[i] = *reinterpret_cast<const U *>(ring + off[i] + s * stride[i]);
#pragma unroll
        for (int i = 0; i < FR::V; i++)
            if (w[i] == Bits<TC>::sentinel) w[i] = Bits<TC>::qnan;
        u32x4 v;
        __builtin_memcpy(&v, w, 16);
        return v;
    }
};

// Boundary role, on two wavefronts (`part` 0 and 1).  A step's halo is a
// record part of the j-upstream tile and one of the k-upstream tile, read as
// 16-byte pieces, one per lane: n lanes hold a step, a wavefront GL = 64 / n
// steps (FP64 blocks on 8 x 8 tiles: 24 lanes, 2 steps), and the wavefronts
// take GL steps in turn.  The values validate themselves (sentinel =
// unwritten); a group of n lanes whose pieces are all written, and whose ring
// slot has been taken, stages its step and moves on.
//   A round is one memory round trip (0.6 us) and under 100 instructions, so
// a halo arrives one trip after its publication, and the wavefronts' rounds
// overlap.  A tile runs at its producers' pace and keeps whatever it once
// fell behind, so the rounds must keep up with the compute wavefront from the
// first step on: one wavefront with twice the loads and more bookkeeping
// took 1.35 us for four steps, and 4 us a tile hop.  Two steps a round also
// for the smaller records of FP32 and of BS = 1: with five or eight the
// missing ones are asked for too often (64^3 FP32 forward 86 against 77 us,
// BS = 1 66 against 56).
// `prog` (and `prog2` where it is given) show that slot t's results of step
// t - DY - 1 have been taken from the ring, which also means that the
// compute wavefront is past step t - DY.
template <typename TC, int BS, bool REV>
__device__ __forceinline__ void boundary_role(const GridTiles &G, int JK, int base, int lane, int part,
                                              const TC *faces, char *yring,
                                              StepFlag (&fl)[YRing<TC, BS>::DY], const Progress &prog,
                                              const Progress *prog2, int *err) {
    using U = typename Bits<TC>::U;
    using YR = YRing<TC, BS>;
    using FR = FaceRec<TC, BS>;
    constexpr int V = FR::V;
    const int TJ = G.TJ, TK = G.TK, S = G.S;
    const int PJ = FR::part(TK), FV = FR::size(TJ, TK);
    const int n = FV / V;                                   // lanes per step, at most 51
    const int GL = min(64 / n, 2);                 // steps per round
    const int g = lane / n, u = lane - g * n;
    const bool lane_ok = g < GL;
    const bool isj = u * V < PJ;
    const int e0 = isj ? u * V : u * V - PJ;                // first value within the part
    const int J = (JK & 0xffff) + (isj ? (REV ? 1 : -1) : 0);
    const int K = (JK >> 16) + (isj ? 0 : (REV ? 1 : -1));
    const int sh = isj ? TJ - 1 : TK - 1;                   // producer step - this tile's step
    const bool have = lane_ok && J >= 0 && J < G.NJ && K >= 0 && K < G.NK;
    // where the lane's values go in a ring slot: value i at off[i] + slot
    // stride[i]; padding goes to a cell that nobody reads
    int off[V], stride[V];
    bool real[V];
#pragma unroll
    for (int i = 0; i < V; i++) {
        const int e = e0 + i, c = e / BS, r = e - c * BS;
        real[i] = c < (isj ? TK : TJ);
        const int cell = !real[i] ? YR::CELLS - 1
                         : isj    ? (REV ? TK - c : c + 1) * (TJ + 1)
                                  : (REV ? TJ - c : c + 1);
        YR::place(cell, r, off[i], stride[i]);
    }
    const uint64_t gmask = lane_ok ? ((1ull << n) - 1ull) << (g * n) : ~0ull;
    // this lane's next step; steps from `lim` on have no producer step (their
    // halo is zero)
    int ts = lane_ok ? part * GL + g : S;
    int lim = have ? S - sh : 0;
    const TC *sp = have ? faces + ((int64_t)G.tidx[J * G.NK + K] * S + sh + ts) * FV + u * V : faces;
    const int64_t hop = have ? (int64_t)2 * GL * FV : 0;
    U fill = 0;
    bool failed = false;
    uint32_t idle = 0;
    while (__ballot(ts < S) != 0) {
        const int taken = min(progress_get(prog), prog2 ? progress_get(*prog2) : INT32_MAX);
        const bool act = ts < S;
        U w[V];
#pragma unroll
        for (int i = 0; i < V; i++) w[i] = fill;
        if (act && ts < lim) {
            const u32x4 raw = load_published(sp);
            __builtin_memcpy(w, &raw, 16);
        }
        bool ready = act && taken >= base + ts - YR::DY + 1;
#pragma unroll
        for (int i = 0; i < V; i++) ready = ready && !(real[i] && w[i] == Bits<TC>::sentinel);
        const bool go = (__ballot(ready) & gmask) == gmask;
        if (go) {
            const int s = YR::slot(ts);
#pragma unroll
            for (int i = 0; i < V; i++)
                *reinterpret_cast<U *>(yring + off[i] + s * stride[i]) = w[i];
            // LDS operations execute in order: the stamp follows the values
            asm volatile("" : : : "memory");
            if (u == 0) {
                const unsigned a = (unsigned)(size_t)((__attribute__((address_space(3))) int *)&fl[s].h[0]);
                asm volatile("ds_write_b32 %0, %1" : : "v"(a), "v"(base + ts) : "memory");
            }
            ts += 2 * GL;
            sp += hop;
        }
        if (__ballot(go) != 0) {
            idle = 0;
            continue;
        }
        if ((++idle & 63u) == 0u && !failed) {
            const int e = __hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (e != 0 || idle > SPIN_LIMIT) {
                if (e == 0 && lane == 0)
                    __hip_atomic_store(err, ERR_STALL_FLAG, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                failed = true;   // stage NaNs from now on so the compute wave drains
                fill = Bits<TC>::qnan;
                lim = 0;
            }
        }
        __builtin_amdgcn_s_sleep(1);
    }
}

// The next tile of this workgroup (same value in every wavefront).  Each
// role runs its own tile loop, so every wavefront passes the two barriers
// once per tile and once more at the end.
// next tile of this workgroup's queue (b % NQ), first to last or, for the
// backward sweep, last to first; -1 when the queue is empty.  Within a
// queue the tiles come in dependency order and every queue is served by at
// least one workgroup, so every taken tile's producers are running.
struct Tile {
    int T, JK;   // tile, J | K << 16
};
__device__ __forceinline__ Tile next_tile(const GridTiles &G, int *ctr, Tile *tile, bool rev,
                                          int blk) {
    __syncthreads();
    if (threadIdx.x == 0) {
        const int q = blk % G.NQ;
        const int i = atomicAdd(ctr + q, 1);
        const int q0 = G.qoff[q], len = G.qoff[q + 1] - q0;
        const int e = q0 + (rev ? len - 1 - i : i);
        *tile = i < len ? Tile{G.qtiles[e], G.qjk[e]} : Tile{-1, 0};
    }
    __syncthreads();
    return *tile;
}

// forward sweep of one grid; blk = this workgroup's index within the grid's
// workgroups (a multiple of GRID_QUEUES of them)
// b is read at cell (i, j, k) of the grid as b[(i + j vsJ + k vsK) BS + r]:
// vsJ = nx, vsK = nx ny for a whole grid, the caller's strides for a box of
// a larger grid
template <int BS, typename TF, typename TC, typename TIN>
__device__ __forceinline__ void grid_fwd_body(const GridTiles &G, const TF *__restrict__ Lt,
                                              const TIN *__restrict__ b, TC *yt, TC *ff, TC *fb,
                                              int *ctr, int *other_ctr, int *err, int blk,
                                              int64_t vsJ, int64_t vsK) {
    constexpr int NM = 3 * BS * BS, NV = NM + BS;
    using PL = StepPlanes<TF, NM>;
    using RR = RhsRing<TIN, BS>;
    using YR = YRing<TC, BS>;
    using FR = FaceRec<TC, BS>;
    constexpr int DY = YR::DY;
    constexpr int SB = PL::BYTES;
    constexpr int D = ring_slots<SB, 120000 - RR::BYTES>();
    constexpr int P = dma_count(SB);                           // DMA instructions per step
    constexpr int KM = (D / NLOAD) < (63 / P) ? (D / NLOAD) : (63 / P), K = KM < 4 ? KM : 4;
    __shared__ __attribute__((aligned(16))) char ringb[D * SB];
    __shared__ __attribute__((aligned(16))) char yring[YR::BYTES];
    __shared__ __attribute__((aligned(16))) char rring[RR::BYTES];
    __shared__ StepFlag fl[DY];
    // steps computed, taken by the publisher, with a staged right-hand side
    __shared__ Progress done_p, pub_p, rhs_p;
    __shared__ Tile tile;
    // wave-uniform role index (an SGPR), so the roles are real branches
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (blk == 0 && (int)threadIdx.x < G.NQ) other_ctr[threadIdx.x] = 0;
    if (threadIdx.x < DY) fl[threadIdx.x].h[0] = fl[threadIdx.x].h[1] = -1;
    if (threadIdx.x < 64)
        done_p.w[threadIdx.x] = pub_p.w[threadIdx.x] = rhs_p.w[threadIdx.x] = 0;
    const int TJ = G.TJ, TK = G.TK, nx = G.nx, S = G.S;
    const int jj = lane % TJ, kk = lane / TJ;
    const int own = (kk + 1) * (TJ + 1) + jj + 1;   // this lane's cell of a ring slot
    if (wave == 0) {
        // ---- compute ----
        // planes and right-hand side of step t, s = t % RS_CH
        auto read_step = [&](const char *sl, int t, int s, TC (&v)[NV]) {
            PL::template read<TC>(sl, lane, v);
            RR::template read<TC>(rring, t, s, lane, v + NM);
        };
        for (int base = 0;; base += S + 1) {
            const Tile tl = next_tile(G, ctr, &tile, false, blk);
            const int T = tl.T;
            if (T < 0) break;
            TC yp[BS];
#pragma unroll
            for (int r = 0; r < BS; r++) yp[r] = TC(0);
            YR::store(yring, 0, own, yp);   // no results before step 0
            progress_put(done_p, lane, base);
            unsigned long long pre = ~0ull;   // flag of the next step, read one step early
            int slot = D > 1 ? SB : 0;        // byte offset of step t + 1's planes
            // step t computes with the planes in vc and reads the planes of
            // step t + 1 into vn; the two arrays swap roles every step.
            // s1 = (t + 1) % RS_CH (the steps are unrolled by RS_CH)
            auto step = [&](int t, int s1, const TC (&vc)[NV], TC (&vn)[NV]) {
                const int st = base + t;
                step_wait(pre, fl[YR::slot(t)], st, err);
                TC yj[BS], yk[BS];
                YR::load(yring, YR::slot(t), own - (TJ + 1), yk);
                YR::load(yring, YR::slot(t), own - 1, yj);
                read_step(ringb + slot, t + 1, s1, vn);
                slot = slot == (D - 1) * SB ? 0 : slot + SB;
                pre = step_flag_get(fl[YR::slot(t + 1)]);
                TC acc[BS];
#pragma unroll
                for (int r = 0; r < BS; r++) acc[r] = vc[NM + r];
                block_sub<BS>(acc, vc, 0, yk);
                block_sub<BS>(acc, vc, 1, yj);
                block_sub<BS>(acc, vc, 2, yp);
#pragma unroll
                for (int r = 0; r < BS; r++) yp[r] = acc[r];
                YR::store(yring, YR::slot(t + 1), own, yp);
                progress_put(done_p, lane, st + 1);
            };
            TC va[NV], vb[NV];
            lds_wait_eq(&fl[DY - 1].h[1], base, err);
            read_step(ringb, 0, 0, va);
            static_assert(RS_CH == 4, "the step loop is unrolled by RS_CH");
            int t = 0;
            for (; t + 3 < S; t += 4) {
                step(t, 1, va, vb);
                step(t + 1, 2, vb, va);
                step(t + 2, 3, va, vb);
                step(t + 3, 0, vb, va);
            }
            if (t < S) step(t, 1, va, vb);
            if (t + 1 < S) step(t + 1, 2, vb, va);
            if (t + 2 < S) step(t + 2, 3, va, vb);
        }
    } else if (wave == 1 || wave == 7) {
        // ---- boundary: faces of tiles (J-1, K) and (J, K-1) ----
        for (int base = 0;; base += S + 1) {
            const Tile tl = next_tile(G, ctr, &tile, false, blk);
            const int T = tl.T;
            if (T < 0) break;
            boundary_role<TC, BS, false>(G, tl.JK, base, lane, wave == 1 ? 0 : 1, ff, yring, fl, pub_p, nullptr, err);
        }
    } else if (wave < 2 + NLOAD) {
        // ---- loaders: DMA of steps w, w + NLOAD, ... ----
        const int w = wave - 2;
        for (int base = 0;; base += S + 1) {
            const Tile tl = next_tile(G, ctr, &tile, false, blk);
            const int T = tl.T;
            if (T < 0) break;
            const TF *lb = Lt + (int64_t)T * S * PL::SIZE;
            auto issue = [&](int t) {
                dma_block<SB, BS == 3>(lb + (int64_t)t * PL::SIZE, ringb + (t % D) * SB, lane);
            };
            loader_loop<D, P, K>(w, S, base, done_p, &rhs_p, fl, lane, err, issue);
            // the backward sweep's face slots of this tile start unwritten
            const int64_t nf = (int64_t)S * FR::size(TJ, TK);
            TC *fr = fb + (int64_t)T * nf;
            for (int64_t e = w * 64 + lane; e < nf; e += NLOAD * 64) fr[e] = sentinel_value<TC>();
        }
    } else if (wave == 5) {
        // ---- publisher: high faces feed tiles J+1, K+1 ----
        const int FV = FR::size(TJ, TK);
        const FacePublisher<TC, BS, false> fp(TJ, TK, lane);
        for (int base = 0;; base += S + 1) {
            // in scalar registers, as the records' place is
            const int T = __builtin_amdgcn_readfirstlane(next_tile(G, ctr, &tile, false, blk).T);
            if (T < 0) break;
            using PY = StepPlanes<TC, BS>;
            TC *yrow = yt + (int64_t)T * S * PY::SIZE;
            TC *frow = ff + (int64_t)T * S * FV;
            int seen = base;
            for (int t = 0; t < S; t++, frow += FV) {
                progress_wait(done_p, base + t + 1, seen, err);
                const u32x4 rec = fp.gather(yring, YR::slot(t + 1));
                TC y[BS];
                YR::load(yring, YR::slot(t + 1), own, y);
                progress_put(pub_p, lane, base + t + 1);
                store_published(frow, FV * (int)sizeof(TC), lane, rec);
#pragma unroll
                for (int r = 0; r < BS; r++) yrow[(int64_t)t * PY::SIZE + PY::at(r, lane)] = y[r];
            }
        }
    } else if (wave == 6) {
        // ---- right-hand side: runs of RS_CH cells of every line ----
        for (int base = 0;; base += S + 1) {
            const Tile tl = next_tile(G, ctr, &tile, false, blk);
            const int T = tl.T;
            if (T < 0) break;
            const int JK = tl.JK;
            // this lane's cell of instruction q: line l, step s of the chunk
            const TIN *src[RR::NI];
            int x[RR::NI];
            const int un = lane / RR::LPU;
            const int rTJ = 65536 / TJ + 1;   // l / TJ = (l rTJ) >> 16 for l < 64, TJ <= 8
#pragma unroll
            for (int q = 0; q < RR::NI; q++) {
                const int r = un / RR::UL, sh = (un % RR::UL) ^ RR::twist(q, r);
                const int l = q * RR::LPB + r;
                const int lkk = (l * rTJ) >> 16, ljj = l - lkk * TJ;
                const int j = (JK & 0xffff) * TJ + ljj, k = (JK >> 16) * TK + lkk;
                const bool ok = l < TJ * TK && j < G.ny && k < G.nz;
                x[q] = ok ? sh / RR::UH - ljj - lkk : INT32_MIN / 2;   // x of the chunk at step 0
                // 12-byte halves of a cell, or the dwords of a double
                const int part = RR::UH == 2 ? (sh % RR::UH) * 12 : (lane % RR::LPU) * 4;
                src[q] = reinterpret_cast<const TIN *>(
                    reinterpret_cast<const char *>(b + ((ok ? vsJ * j + vsK * k : 0) + x[q]) * BS) + part);
            }
            // chunk c overwrites the steps RS_STEPS before its own; up to
            // NCH chunks in flight
            constexpr int NCH = RS_STEPS / RS_CH;
            static_assert(NCH == 4 && NCH * RR::NI <= 63, "in-flight DMA within the vmcnt range");
            const int nchunk = (S + RS_CH - 1) / RS_CH;
            int next = 0, done = 0;
            uint32_t idle = 0;
            wait_vm<0>();
            while (done < nchunk) {
                while (next < nchunk && next - done < NCH &&
                       (next < NCH || __builtin_amdgcn_readfirstlane(lds_flag_get(done_p.w)) >=
                                          base + (next - NCH + 1) * RS_CH)) {
                    char *dst = rring + (next & (NCH - 1)) * RR::CHB;
                    const int t0 = next * RS_CH;
#pragma unroll
                    for (int q = 0; q < RR::NI; q++) {
                        const int xi = x[q] + t0;
                        const bool ok = xi >= 0 && xi < nx;
                        dma_piece<RR::UB == 16 ? 12 : 4>(
                            ok ? static_cast<const void *>(src[q] + (int64_t)t0 * BS)
                               : static_cast<const void *>(zero_cell),
                            dst + q * RR::IB);
                    }
                    next++;
                }
                const int inflight = next - done;
                if (inflight == 0) {
                    if (++idle > 4 * SPIN_LIMIT) {
                        __hip_atomic_store(err, ERR_STALL_FLAG, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        break;
                    }
                    __builtin_amdgcn_s_sleep(1);
                    continue;
                }
                idle = 0;
                if (inflight == 4) wait_vm<3 * RR::NI>();
                if (inflight == 3) wait_vm<2 * RR::NI>();
                if (inflight == 2) wait_vm<RR::NI>();
                if (inflight == 1) wait_vm<0>();
                done++;
                progress_put(rhs_p, lane, base + min(done * RS_CH, S));
            }
        }
    } else {
        while (next_tile(G, ctr, &tile, false, blk).T >= 0) {
        }
    }
}

// cells of a grid written by the backward sweep: those with i in [i0, i1),
// j in [j0, j1), k in [k0, k1), at (i + j vsJ + k vsK) BS of the output (all
// of a whole grid's; a subdomain's owned cells under RAS)
struct OutBox {
    int i0, i1, j0, j1, k0, k1;
    int64_t vsJ, vsK;
};

// Writer role of the backward sweep.  It takes CK steps of a tile at a time
// from the result ring, a lane one cell of a group of 64 / CK lines, so that
// a store covers runs of CK consecutive cells of each line (96 bytes for
// three doubles): the run of the next CK steps completes the cache lines in
// the XCD's L2.  The epilogues of ilu_apply: ADD 0 xo = x; 1 add_out =
// add_in + x; 2 add_out = (add_in[cell], 0, 0) + x.  Their operands are
// loaded before the wait for the steps, off everyone's critical path.
template <int BS, typename TC, typename TO, int ADD, typename TAI, typename TAO>
__device__ __forceinline__ void writer_role(const GridTiles &G, int JK, int base, int lane,
                                            const char *yring, const Progress &done_p, Progress &wr_p,
                                            const OutBox &box, TO *__restrict__ xo,
                                            const TAI *__restrict__ add_in,
                                            TAO *__restrict__ add_out, int *err) {
    using YR = YRing<TC, BS>;
    constexpr int CK = YR::DY / 4, LPI = 64 / CK, NA = ADD == 1 ? BS : 1;
    const int TJ = G.TJ, TK = G.TK, S = G.S;
    const int j0 = (JK & 0xffff) * TJ, k0 = (JK >> 16) * TK;
    const int rTJ = 65536 / TJ + 1;   // l / TJ = (l rTJ) >> 16 for l < 64, TJ <= 8
    int seen = base;
    for (int c0 = 0; c0 < S; c0 += CK) {
        const int tau = c0 + lane % CK;
        int64_t off[CK];
        int cell[CK];
        TAI ain[ADD ? CK : 1][NA];
#pragma unroll
        for (int g = 0; g < CK; g++) {
            const int l = g * LPI + lane / CK;
            const int kk = (l * rTJ) >> 16, jj = l - kk * TJ;
            const int i = S - 1 - tau - jj - kk, j = j0 + jj, k = k0 + kk;
            const bool ok = tau < S && l < TJ * TK && i >= box.i0 && i < box.i1 && j >= box.j0 &&
                            j < box.j1 && k >= box.k0 && k < box.k1;
            off[g] = ok ? i + box.vsJ * j + box.vsK * k : -1;
            cell[g] = ((kk < TK ? TK - 1 - kk : kk) + 1) * (TJ + 1) + TJ - jj;
            if (ADD)
#pragma unroll
                for (int r = 0; r < NA; r++) ain[g][r] = ok ? add_in[off[g] * NA + r] : TAI(0);
        }
        const int upto = base + (c0 + CK < S ? c0 + CK : S);
        progress_wait(done_p, upto, seen, err);
#pragma unroll
        for (int g = 0; g < CK; g++) {
            TC v[BS];
            YR::load(yring, YR::slot(tau + 1), cell[g], v);
            if (off[g] < 0) continue;
#pragma unroll
            for (int r = 0; r < BS; r++) {
                if (ADD == 0) xo[off[g] * BS + r] = static_cast<TO>(v[r]);
                if (ADD == 1)
                    add_out[off[g] * BS + r] = static_cast<TAO>(ain[g][r]) + static_cast<TAO>(v[r]);
                if (ADD == 2) {
                    const TC base0 = (r == 0) ? static_cast<TC>(ain[g][0]) : TC(0);
                    add_out[off[g] * BS + r] = static_cast<TAO>(base0 + v[r]);
                }
            }
        }
        asm volatile("" : : : "memory");
        progress_put(wr_p, lane, upto);
    }
}

template <int BS, typename TF, typename TD, typename TC, typename TO, int ADD, typename TAI,
          typename TAO>
__device__ __forceinline__ void grid_bwd_body(const GridTiles &G, const TF *__restrict__ Ut,
                                              const TD *__restrict__ Dt, const TC *yt, TC *fb, TC *ff,
                                              int *ctr, int *other_ctr, int *err, int blk,
                                              const OutBox &box, TO *__restrict__ xo,
                                              const TAI *__restrict__ add_in,
                                              TAO *__restrict__ add_out) {
    constexpr int B2 = BS * BS, NM = 3 * B2, NV = NM + B2 + BS;
    // ring step: the factor planes, the diagonal inverses, the forward result
    using PL = StepPlanes<TF, NM>;
    using PD = StepPlanes<TD, B2>;
    using PY = StepPlanes<TC, BS>;
    using YR = YRing<TC, BS>;
    using FR = FaceRec<TC, BS>;
    constexpr int DY = YR::DY;
    constexpr int PB = PL::BYTES, DBY = PD::BYTES, YB = PY::BYTES;
    constexpr int SB = PB + DBY + YB;
    constexpr int D = ring_slots<SB, 120000>();
    constexpr int P = dma_count(PB) + dma_count(DBY) + dma_count(YB);
    constexpr int KM = (D / NLOAD) < (63 / P) ? (D / NLOAD) : (63 / P), K = KM < 4 ? KM : 4;
    __shared__ __attribute__((aligned(16))) char ringb[D * SB];
    __shared__ __attribute__((aligned(16))) char yring[YR::BYTES];
    __shared__ StepFlag fl[DY];
    __shared__ Progress done_p, pub_p, wr_p;   // computed, published, written
    __shared__ Tile tile;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (blk == 0 && (int)threadIdx.x < G.NQ) other_ctr[threadIdx.x] = 0;
    if (threadIdx.x < DY) fl[threadIdx.x].h[0] = fl[threadIdx.x].h[1] = -1;
    if (threadIdx.x < 64) done_p.w[threadIdx.x] = pub_p.w[threadIdx.x] = wr_p.w[threadIdx.x] = 0;
    const int TJ = G.TJ, TK = G.TK, S = G.S;
    const int jj = lane % TJ, kk = lane / TJ;
    // the ring slots hold the tile mirrored in j and k, so the +1 neighbours
    // sit where the forward sweep has its -1 neighbours
    const int own = ((kk < TK ? TK - 1 - kk : kk) + 1) * (TJ + 1) + TJ - jj;
    if (wave == 0) {
        // ---- compute ----
        auto read_step = [&](const char *sl, TC (&v)[NV]) {
            PL::template read<TC>(sl, lane, v);
            PD::template read<TC>(sl + PB, lane, v + NM);
            PY::template read<TC>(sl + PB + DBY, lane, v + NM + B2);
        };
        for (int base = 0;; base += S + 1) {
            const int T = next_tile(G, ctr, &tile, true, blk).T;   // reverse tile order
            if (T < 0) break;
            TC xp[BS];
#pragma unroll
            for (int r = 0; r < BS; r++) xp[r] = TC(0);
            YR::store(yring, 0, own, xp);
            progress_put(done_p, lane, base);
            unsigned long long pre = ~0ull;
            int slot = D > 1 ? SB : 0;
            auto step = [&](int t, const TC (&vc)[NV], TC (&vn)[NV]) {
                const int st = base + t;
                step_wait(pre, fl[YR::slot(t)], st, err);
                TC xj[BS], xk[BS];
                YR::load(yring, YR::slot(t), own - 1, xj);
                YR::load(yring, YR::slot(t), own - (TJ + 1), xk);
                read_step(ringb + slot, vn);
                slot = slot == (D - 1) * SB ? 0 : slot + SB;
                pre = step_flag_get(fl[YR::slot(t + 1)]);
                TC acc[BS];
#pragma unroll
                for (int r = 0; r < BS; r++) acc[r] = vc[NM + B2 + r];
                block_sub<BS>(acc, vc, 0, xp);
                block_sub<BS>(acc, vc, 1, xj);
                block_sub<BS>(acc, vc, 2, xk);
                // neighbours consume the value as the caller's output type
#pragma unroll
                for (int r = 0; r < BS; r++) {
                    TC sum = TC(0);
#pragma unroll
                    for (int q = 0; q < BS; q++) sum += vc[NM + r * BS + q] * acc[q];
                    xp[r] = static_cast<TC>(static_cast<TO>(sum));
                }
                YR::store(yring, YR::slot(t + 1), own, xp);
                progress_put(done_p, lane, st + 1);
            };
            TC va[NV], vb[NV];
            lds_wait_eq(&fl[DY - 1].h[1], base, err);
            read_step(ringb, va);
            int t = 0;
            for (; t + 1 < S; t += 2) {
                step(t, va, vb);
                step(t + 1, vb, va);
            }
            if (t < S) step(t, va, vb);
        }
    } else if (wave == 1 || wave == 7) {
        // ---- boundary: faces of tiles (J+1, K) and (J, K+1) ----
        for (int base = 0;; base += S + 1) {
            const Tile tl = next_tile(G, ctr, &tile, true, blk);
            const int T = tl.T;
            if (T < 0) break;
            boundary_role<TC, BS, true>(G, tl.JK, base, lane, wave == 1 ? 0 : 1, fb, yring, fl, pub_p, &wr_p, err);
        }
    } else if (wave < 2 + NLOAD) {
        // ---- loaders: DMA of U blocks, diagonal inverses, forward result ----
        const int w = wave - 2;
        for (int base = 0;; base += S + 1) {
            const Tile tl = next_tile(G, ctr, &tile, true, blk);
            const int T = tl.T;
            if (T < 0) break;
            const TF *ub = Ut + (int64_t)T * S * PL::SIZE;
            const TD *db = Dt + (int64_t)T * S * PD::SIZE;
            const TC *yb = yt + (int64_t)T * S * PY::SIZE;
            auto issue = [&](int t) {
                char *sl = ringb + (t % D) * SB;
                dma_block<PB, BS == 3>(ub + (int64_t)t * PL::SIZE, sl, lane);
                dma_block<DBY, BS == 3>(db + (int64_t)t * PD::SIZE, sl + PB, lane);
                // the forward result of the same cells: forward step S - 1 - t
                dma_block<YB, BS == 3>(yb + (int64_t)(S - 1 - t) * PY::SIZE, sl + PB + DBY, lane);
            };
            loader_loop<D, P, K>(w, S, base, done_p, nullptr, fl, lane, err, issue);
            // the forward sweep's face slots of this tile start unwritten
            const int64_t nf = (int64_t)S * FR::size(TJ, TK);
            TC *fr = ff + (int64_t)T * nf;
            for (int64_t e = w * 64 + lane; e < nf; e += NLOAD * 64) fr[e] = sentinel_value<TC>();
        }
    } else if (wave == 5) {
        // ---- publisher: low faces feed tiles J-1, K-1 ----
        const int FV = FR::size(TJ, TK);
        const FacePublisher<TC, BS, true> fp(TJ, TK, lane);
        for (int base = 0;; base += S + 1) {
            // in scalar registers, as the records' place is
            const int T = __builtin_amdgcn_readfirstlane(next_tile(G, ctr, &tile, true, blk).T);
            if (T < 0) break;
            TC *frow = fb + (int64_t)T * S * FV;
            int seen = base;
            for (int t = 0; t < S; t++, frow += FV) {
                progress_wait(done_p, base + t + 1, seen, err);
                const u32x4 rec = fp.gather(yring, YR::slot(t + 1));
                progress_put(pub_p, lane, base + t + 1);
                store_published(frow, FV * (int)sizeof(TC), lane, rec);
            }
        }
    } else if (wave == 6) {
        // ---- writer ----
        for (int base = 0;; base += S + 1) {
            const Tile tl = next_tile(G, ctr, &tile, true, blk);
            const int T = tl.T;
            if (T < 0) break;
            writer_role<BS, TC, TO, ADD, TAI, TAO>(G, tl.JK, base, lane, yring, done_p, wr_p, box, xo,
                                                   add_in, add_out, err);
        }
    } else {
        while (next_tile(G, ctr, &tile, true, blk).T >= 0) {
        }
    }
}

template <int BS, typename TF, typename TC, typename TIN>
__global__ __launch_bounds__(GWG) void k_grid_fwd(GridTiles G, const TF *__restrict__ Lt,
                                                  const TIN *__restrict__ b, TC *yt, TC *ff,
                                                  TC *fb, int *ctr, int *other_ctr, int *err) {
    grid_fwd_body<BS, TF, TC, TIN>(G, Lt, b, yt, ff, fb, ctr, other_ctr, err, blockIdx.x, G.nx,
                                   (int64_t)G.nx * G.ny);
}

template <int BS, typename TF, typename TD, typename TC, typename TO, int ADD, typename TAI,
          typename TAO>
__global__ __launch_bounds__(GWG) void k_grid_bwd(GridTiles G, const TF *__restrict__ Ut,
                                                  const TD *__restrict__ Dt, const TC *yt, TC *fb,
                                                  TC *ff, int *ctr, int *other_ctr, int *err,
                                                  TO *__restrict__ xo, const TAI *__restrict__ add_in,
                                                  TAO *__restrict__ add_out) {
    const OutBox box{0, G.nx, 0, G.ny, 0, G.nz, G.nx, (int64_t)G.nx * G.ny};
    grid_bwd_body<BS, TF, TD, TC, TO, ADD, TAI, TAO>(G, Ut, Dt, yt, fb, ff, ctr, other_ctr, err,
                                                     blockIdx.x, box, xo, add_in, add_out);
}

// ---------------------------------------------------------------------------
// several independent grids in one launch (the subdomains of RAS): grid g
// owns the workgroups [wg0, wg0 + wgs) of each kernel (multiples of
// GRID_QUEUES, so a workgroup's queue, and XCD, keep their mapping)
// ---------------------------------------------------------------------------
__device__ __forceinline__ int find_grid(const GridMulti *__restrict__ d, int ngrid, int blk) {
    int g = 0;
    while (g + 1 < ngrid && blk >= d[g + 1].wg0) g++;
    return g;
}

template <int BS>
__global__ __launch_bounds__(GWG) void k_grid_fwd_multi(const GridMulti *__restrict__ d, int ngrid,
                                                        const double *__restrict__ v, int *err,
                                                        char *origin) {
    const int g = find_grid(d, ngrid, blockIdx.x);
    GridMulti D = d[g];
    globalize(origin, D.G);
    grid_fwd_body<BS, double, double, double>(
        D.G, as_global(origin, D.lt), v + D.boff, as_global(origin, D.yt), as_global(origin, D.ff), as_global(origin, D.fb),
        as_global(origin, D.ctr), as_global(origin, D.ctr) + D.G.NQ, err, blockIdx.x - D.wg0, D.vsJ, D.vsK);
}

template <int BS>
__global__ __launch_bounds__(GWG) void k_grid_bwd_multi(const GridMulti *__restrict__ d, int ngrid,
                                                        double *__restrict__ z, int *err,
                                                        char *origin) {
    const int g = find_grid(d, ngrid, blockIdx.x);
    GridMulti D = d[g];
    globalize(origin, D.G);
    const OutBox box{D.oi0, D.oi1, D.oj0, D.oj1, D.ok0, D.ok1, D.vsJ, D.vsK};
    grid_bwd_body<BS, double, double, double, double, 0, double, double>(
        D.G, as_global(origin, D.ut), as_global(origin, D.dt), as_global(origin, D.yt), as_global(origin, D.fb), as_global(origin, D.ff),
        as_global(origin, D.ctr) + D.G.NQ, as_global(origin, D.ctr), err, blockIdx.x - D.wg0, box, z + D.boff,
        nullptr, nullptr);
}

int grid_multi_launch_size(const IluFactor &F, int *wgs) {
    if (!F.grid) return set_error(KRY_ERR_ARG, "grid_multi: not a grid-tiled factor");
    *wgs = F.G.NQ * std::max(1, std::min(F.G.qmax, 512 / F.G.NQ));
    return KRY_OK;
}

int grid_multi_desc(const IluFactor &F, int64_t boff, int64_t vsJ, int64_t vsK, const int own[6],
                    int wg0, GridMulti &d) {
    if (!F.grid || F.prec != KRY_PREC_F64)
        return set_error(KRY_ERR_ARG, "grid_multi: needs an FP64 grid-tiled factor");
    d.G = F.G;
    d.lt = F.lt64.p;
    d.ut = F.ut64.p;
    d.dt = F.dt64.p;
    d.yt = F.yt64.p;
    d.ff = F.ff64.p;
    d.fb = F.fb64.p;
    d.ctr = F.ctr.p;
    d.boff = boff;
    d.vsJ = vsJ;
    d.vsK = vsK;
    d.oi0 = own[0];
    d.oi1 = own[1];
    d.oj0 = own[2];
    d.oj1 = own[3];
    d.ok0 = own[4];
    d.ok1 = own[5];
    d.wg0 = wg0;
    return KRY_OK;
}

int grid_multi_apply(hipStream_t s, int bs, const GridMulti *d_desc, int ngrid, int total_wgs,
                     const double *v, double *z, int *err) {
    {
        TimedScope t("ras_ilu_fwd", s);
        if (bs == 1)
            hipLaunchKernelGGL(k_grid_fwd_multi<1>, dim3(total_wgs), dim3(GWG), 0, s, d_desc, ngrid, v, err,
                               static_cast<char *>(nullptr));
        else
            hipLaunchKernelGGL(k_grid_fwd_multi<3>, dim3(total_wgs), dim3(GWG), 0, s, d_desc, ngrid, v, err,
                               static_cast<char *>(nullptr));
    }
    {
        TimedScope t("ras_ilu_bwd", s);
        if (bs == 1)
            hipLaunchKernelGGL(k_grid_bwd_multi<1>, dim3(total_wgs), dim3(GWG), 0, s, d_desc, ngrid, z, err,
                               static_cast<char *>(nullptr));
        else
            hipLaunchKernelGGL(k_grid_bwd_multi<3>, dim3(total_wgs), dim3(GWG), 0, s, d_desc, ngrid, z, err,
                               static_cast<char *>(nullptr));
    }
    KRY_HIP(hipGetLastError());
    return KRY_OK;
}

// ---------------------------------------------------------------------------
// dispatch (same type combinations as the level-scheduled sweeps)
// ---------------------------------------------------------------------------
template <int BS, typename TF, typename TD, typename TC, typename TIN, typename TO, int ADD,
          typename TAI, typename TAO>
static int grid_pair(hipStream_t s, IluFactor &F, const TF *lt, const TF *ut, const TD *dt,
                     TC *yt, TC *ff, TC *fb, const TIN *b, TO *xo, const TAI *add_in,
                     TAO *add_out, int *err) {
    // one workgroup per tile in flight (LDS-bound, 256 CUs): NQ workgroups
    // per queue position, so every queue has a workgroup per tile up to
    // the cap, and always at least one
    const int wgs = F.G.NQ * std::max(1, std::min(F.G.qmax, 512 / F.G.NQ));
    {
        TimedScope t(F.timer_fwd ? F.timer_fwd : sweep_timer_name(true, BS, sizeof(TF), ADD), s);
        hipLaunchKernelGGL((k_grid_fwd<BS, TF, TC, TIN>), dim3(wgs), dim3(GWG), 0, s, F.G, lt, b,
                           yt, ff, fb, F.ctr.p, F.ctr.p + F.G.NQ, err);
    }
    {
        TimedScope t(F.timer_bwd ? F.timer_bwd : sweep_timer_name(false, BS, sizeof(TF), ADD), s);
        hipLaunchKernelGGL((k_grid_bwd<BS, TF, TD, TC, TO, ADD, TAI, TAO>), dim3(wgs), dim3(GWG), 0,
                           s, F.G, ut, dt, yt, fb, ff, F.ctr.p + F.G.NQ, F.ctr.p, err, xo, add_in,
                           add_out);
    }
    KRY_HIP(hipGetLastError());
    return KRY_OK;
}

template <int BS, typename TIN, typename TO>
static int grid_typed(hipStream_t s, IluFactor &F, const TIN *b, TO *xo, int add_mode,
                      const void *add_in, void *add_out, int *err) {
    if (F.prec == KRY_PREC_F64) {
        using TC = double;
        TC *yt = F.yt64.p, *ff = F.ff64.p, *fb = F.fb64.p;
        if (add_mode == 0)
            return grid_pair<BS, double, double, TC, TIN, TO, 0, double, double>(
                s, F, F.lt64.p, F.ut64.p, F.dt64.p, yt, ff, fb, b, xo, nullptr, nullptr, err);
        if (add_mode == 1)
            return grid_pair<BS, double, double, TC, TIN, TO, 1, TO, TO>(
                s, F, F.lt64.p, F.ut64.p, F.dt64.p, yt, ff, fb, b, xo, (const TO *)add_in,
                (TO *)add_out, err);
        return grid_pair<BS, double, double, TC, TIN, TO, 2, TC, double>(
            s, F, F.lt64.p, F.ut64.p, F.dt64.p, yt, ff, fb, b, xo, (const TC *)add_in,
            (double *)add_out, err);
    }
    using TC = float;
    TC *yt = F.yt32.p, *ff = F.ff32.p, *fb = F.fb32.p;
    if (F.prec == KRY_PREC_F32) {
        if (add_mode == 0)
            return grid_pair<BS, float, float, TC, TIN, TO, 0, float, float>(
                s, F, F.lt32.p, F.ut32.p, F.dt32.p, yt, ff, fb, b, xo, nullptr, nullptr, err);
        if (add_mode == 1)
            return grid_pair<BS, float, float, TC, TIN, TO, 1, TO, TO>(
                s, F, F.lt32.p, F.ut32.p, F.dt32.p, yt, ff, fb, b, xo, (const TO *)add_in,
                (TO *)add_out, err);
        return grid_pair<BS, float, float, TC, TIN, TO, 2, TC, double>(
            s, F, F.lt32.p, F.ut32.p, F.dt32.p, yt, ff, fb, b, xo, (const TC *)add_in,
            (double *)add_out, err);
    }
    if (add_mode == 0)
        return grid_pair<BS, uint16_t, float, TC, TIN, TO, 0, float, float>(
            s, F, F.lt16.p, F.ut16.p, F.dt32.p, yt, ff, fb, b, xo, nullptr, nullptr, err);
    if (add_mode == 1)
        return grid_pair<BS, uint16_t, float, TC, TIN, TO, 1, TO, TO>(
            s, F, F.lt16.p, F.ut16.p, F.dt32.p, yt, ff, fb, b, xo, (const TO *)add_in,
            (TO *)add_out, err);
    return grid_pair<BS, uint16_t, float, TC, TIN, TO, 2, TC, double>(
        s, F, F.lt16.p, F.ut16.p, F.dt32.p, yt, ff, fb, b, xo, (const TC *)add_in,
        (double *)add_out, err);
}

template <int BS>
static int grid_bs(hipStream_t s, IluFactor &F, const void *b, int in_type, void *xscr,
                   int out_type, int add_mode, const void *add_in, void *add_out, int *err) {
    if (in_type == 0 && out_type == 0)
        return grid_typed<BS>(s, F, (const double *)b, (double *)xscr, add_mode, add_in, add_out, err);
    if (in_type == 0 && out_type == 1)
        return grid_typed<BS>(s, F, (const double *)b, (float *)xscr, add_mode, add_in, add_out, err);
    if (in_type == 1 && out_type == 0)
        return grid_typed<BS>(s, F, (const float *)b, (double *)xscr, add_mode, add_in, add_out, err);
    return grid_typed<BS>(s, F, (const float *)b, (float *)xscr, add_mode, add_in, add_out, err);
}

int ilu_grid_apply(hipStream_t s, IluFactor &F, const void *b, int in_type, void *xscr,
                   int out_type, int add_mode, const void *add_in, void *add_out, int *d_err) {
    if (F.bs == 1) return grid_bs<1>(s, F, b, in_type, xscr, out_type, add_mode, add_in, add_out, d_err);
    return grid_bs<3>(s, F, b, in_type, xscr, out_type, add_mode, add_in, add_out, d_err);
}

}  // namespace kry
