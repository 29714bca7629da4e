// ILU(0) and block ILU(0) preconditioner: the incomplete factorization
// named in Section 1 (point-wise and block-wise) and the two triangular
// solves of eq. (3), which Section 4.1 notes are row-by-row serial.
//
// gfx950 design
//  * Level scheduling: row i of L y = b depends on the rows k < i of its
//    pattern; its level is one more than the deepest of them (rows with no
//    dependency are level 0).  Backward levels are built the same way from
//    the upper pattern.  For a 7-point stencil in natural order these are
//    the hyperplanes i + j + k = const.
//  * Factorization: one launch per forward level, one thread per row,
//    row-oriented elimination restricted to the pattern (IKJ); the inverse
//    of each diagonal block is formed once (Gaussian elimination with
//    partial pivoting) and reused by every later row and by the solve.
//  * Layout: rows are permuted by level and each level is padded to whole
//    64-row slices, so a wavefront always holds rows of one level, which
//    are mutually independent; for the row blocks rows are permuted by level
//    inside blocks of 256 only.  Values sit in entry-major planes (sliced
//    ELLPACK), so the factor streams from HBM in full cache lines.
//  * Sweeps: one launch per sweep.  Rows with few dependencies are swept by
//    blocks of consecutive rows (see there).  For wider ones wavefronts take
//    slices in level order from an atomic counter; a row waits only for the
//    rows it reads.  Each output value is published with a relaxed
//    agent-scope store into a slot pre-filled with a reserved NaN payload,
//    and consumers poll the slot itself -- no flags, no fences, no grid
//    barriers.  What a slice (a block) reads lies in earlier slices (blocks),
//    which were handed to wavefronts that are already running, so the sweep
//    cannot deadlock; a bounded spin turns any broken schedule into an error
//    instead of a hang.
#include <algorithm>
#include <cmath>
#include <cstdlib>

#include "device.hpp"
#include "internal.hpp"

namespace kry {

// ---------------------------------------------------------------------------
// host: level sets and level-ordered slices
// ---------------------------------------------------------------------------
struct LevelSlices {
    std::vector<int> perm;        // nslices * 64, -1 = padding lane
    std::vector<int> off;         // nslices + 1 slot offsets
    std::vector<int> lev_slice;   // nlev + 1: first slice of each level
    std::vector<int> slice_of;    // row -> slice
    int nslices = 0, nlev = 0, maxw = 0;
};

// lev: level of each row; ndep(row) number of dependencies (slot count)
template <typename F>
static void build_slices(int nb, const std::vector<int> &lev, int nlev, F ndep,
                         LevelSlices &L) {
    std::vector<int> cnt(nlev + 1, 0);
    for (int i = 0; i < nb; i++) cnt[lev[i] + 1]++;
    for (int l = 0; l < nlev; l++) cnt[l + 1] += cnt[l];
    std::vector<int> order(nb);
    {
        std::vector<int> pos(cnt.begin(), cnt.end() - 1);
        for (int i = 0; i < nb; i++) order[pos[lev[i]]++] = i;   // stable by row index
    }
    L.nlev = nlev;
    L.lev_slice.assign(nlev + 1, 0);
    int ns = 0;
    for (int l = 0; l < nlev; l++) {
        L.lev_slice[l] = ns;
        ns += (cnt[l + 1] - cnt[l] + 63) / 64;
    }
    L.lev_slice[nlev] = ns;
    L.nslices = ns;
    L.perm.assign((size_t)ns * 64, -1);
    L.off.assign(ns + 1, 0);
    L.slice_of.assign(nb, -1);
    L.maxw = 0;
    for (int l = 0; l < nlev; l++) {
        const int r0 = cnt[l], m = cnt[l + 1] - cnt[l];
        for (int q = 0; q < m; q++) {
            const int sl = L.lev_slice[l] + q / 64;
            L.perm[(size_t)sl * 64 + q % 64] = order[r0 + q];
            L.slice_of[order[r0 + q]] = sl;
        }
    }
    for (int s = 0; s < ns; s++) {
        int w = 0;
        for (int q = 0; q < 64; q++) {
            const int r = L.perm[(size_t)s * 64 + q];
            if (r >= 0) w = std::max(w, ndep(r));
        }
        L.off[s + 1] = L.off[s] + w;
        L.maxw = std::max(L.maxw, w);
    }
}

// every dependency of a row must live in an earlier slice
template <typename F>
static bool schedule_is_acyclic(int nb, const LevelSlices &L, F for_deps) {
    for (int i = 0; i < nb; i++) {
        const int si = L.slice_of[i];
        bool ok = si >= 0;
        for_deps(i, [&](int k) { ok = ok && L.slice_of[k] >= 0 && L.slice_of[k] < si; });
        if (!ok) return false;
    }
    return true;
}

// ---------------------------------------------------------------------------
// blocks of consecutive rows
// ---------------------------------------------------------------------------
constexpr int RB_ROWS = 256;             // rows of a block, one lane each
constexpr int RB_SLICES = RB_ROWS / 64;  // its compute wavefronts
constexpr int RB_IMPORT = 4;             // its importing wavefronts
constexpr int RB_THREADS = RB_ROWS + 64 * RB_IMPORT;
constexpr int RB_WIDE = 6;               // most dependencies of a row
constexpr int RB_TABLE = 2048;           // hash table of a block's outside rows
static_assert(RB_TABLE > RB_ROWS * RB_WIDE, "the table never fills");

// Blocks in the order in which they are started: ascending rows for the
// lower pattern, descending for the upper one, so that a block reads only
// blocks started before it.  Rows of a block are put to lanes by level, then
// by number.  A dependency inside the block is LDS cell `lane`, one outside
// of it cell RB_ROWS + n, n counting the block's distinct outside rows by
// first use (lane by lane).
//   One workgroup per block and direction (y: 0 lower, 1 upper), a thread a
// row.  WRITE = false: the rows of the lanes, each slice's width into off and
// each block's number of outside rows into woff.  WRITE = true, off and woff
// being offsets now: the cells and the vector elements to import.
//   Made here and not by the host, where it took longer than the
// factorization at every assembly.  Red-black order, 3x3 blocks: an assembly
// of 262 144 rows 13.4 -> 4.0 ms, of 1 572 864 rows 83 -> 17 ms (the level
// schedule: 5.0 and 29 ms).
template <bool WRITE>
__global__ __launch_bounds__(RB_ROWS) void k_row_blocks(int nb, int bs, const int *__restrict__ rowptr,
                                                        const int *__restrict__ col,
                                                        const int *__restrict__ diag,
                                                        const int *__restrict__ lev_l,
                                                        const int *__restrict__ lev_u, RowBlocks lower,
                                                        RowBlocks upper) {
    __shared__ __attribute__((aligned(16))) int lev[RB_ROWS];
    __shared__ int lane_of[RB_ROWS], uses[RB_ROWS], width[RB_SLICES], sums[RB_SLICES];
    __shared__ int key[RB_TABLE], first[RB_TABLE];   // a row, its first use (later its number)
    const bool up = blockIdx.y != 0;
    const RowBlocks P = up ? upper : lower;
    const int blk = blockIdx.x, t = threadIdx.x;
    const int r1 = up ? nb - blk * RB_ROWS : min(nb, (blk + 1) * RB_ROWS);
    const int r0 = up ? max(0, r1 - RB_ROWS) : blk * RB_ROWS;
    // the thread's row: the block's t-th, in the second pass lane t's
    const int i = WRITE ? P.perm[(int64_t)blk * RB_ROWS + t] : r0 + t < r1 ? r0 + t : -1;
    const bool live = i >= 0;
    int p0 = 0, n = 0, k[RB_WIDE];
    if (live) {
        p0 = up ? diag[i] + 1 : rowptr[i];
        n = (up ? rowptr[i + 1] : diag[i]) - p0;
    }
#pragma unroll
    for (int d = 0; d < RB_WIDE; d++) k[d] = d < n ? col[p0 + d] : -1;
    if (!WRITE) lev[t] = live ? (up ? lev_u : lev_l)[i] : INT_MAX;
    if (t < RB_SLICES) width[t] = 0;
    for (int e = t; e < RB_TABLE; e += RB_ROWS) {
        key[e] = -1;
        first[e] = INT_MAX;
    }
    __syncthreads();
    int lane = t;   // rows that there are not come last
    if (!WRITE && live) {
        const int4 *l4 = reinterpret_cast<const int4 *>(lev);
        const int own = lev[t];
        lane = 0;
#pragma unroll 4
        for (int q = 0; q < RB_ROWS / 4; q++) {
            const int4 l = l4[q];
            lane += (l.x < own + (4 * q < t)) + (l.y < own + (4 * q + 1 < t)) + (l.z < own + (4 * q + 2 < t)) +
                    (l.w < own + (4 * q + 3 < t));
        }
    }
    if (live) lane_of[i - r0] = lane;
    // the outside rows into the table, with the least use of each
    int at[RB_WIDE];
#pragma unroll
    for (int d = 0; d < RB_WIDE; d++) {
        at[d] = -1;
        if (d >= n || (k[d] >= r0 && k[d] < r1)) continue;
        int h = static_cast<int>(static_cast<uint32_t>(k[d]) * 2654435761u >> 21);
        static_assert(RB_TABLE == 1 << (32 - 21), "the hash has the table's range");
        for (int old; (old = atomicCAS(&key[h], -1, k[d])) != -1 && old != k[d];) h = (h + 1) & (RB_TABLE - 1);
        atomicMin(&first[h], lane * RB_WIDE + d);
        at[d] = h;
    }
    if (live) atomicMax(&width[lane >> 6], n);
    __syncthreads();
    // a row that an earlier use has counted has its number from there
    unsigned firsts = 0;
#pragma unroll
    for (int d = 0; d < RB_WIDE; d++)
        if (at[d] >= 0 && first[at[d]] == lane * RB_WIDE + d) firsts |= 1u << d;
    uses[lane] = __popc(firsts);
    __syncthreads();
    // the uses of the lanes before each lane
    const int own = uses[t], wave = t >> 6;
    int sum = own;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int v = __shfl_up(sum, o);
        if ((t & 63) >= o) sum += v;
    }
    if ((t & 63) == 63) sums[wave] = sum;
    __syncthreads();
    for (int w = 0; w < wave; w++) sum += sums[w];
    if (!WRITE) {
        P.perm[(int64_t)blk * RB_ROWS + lane] = live ? i : -1;
        if (t < RB_SLICES) P.off[blk * RB_SLICES + t] = width[t];
        if (t == RB_ROWS - 1) P.woff[blk] = sum;
        return;
    }
    uses[t] = sum - own;
    __syncthreads();
    int num = uses[lane];
    int *words = P.words + P.woff[blk];
#pragma unroll
    for (int d = 0; d < RB_WIDE; d++)
        if (firsts >> d & 1u) {
            for (int r = 0; r < bs; r++) words[num * bs + r] = k[d] * bs + r;
            first[at[d]] = num++;
        }
    __syncthreads();
    const int s = blk * RB_SLICES + (lane >> 6), o0 = P.off[s], w = P.off[s + 1] - o0;
#pragma unroll
    for (int d = 0; d < RB_WIDE; d++)
        if (d < w)
            P.cell[(int64_t)(o0 + d) * 64 + (lane & 63)] =
                d >= n ? -1 : at[d] >= 0 ? RB_ROWS + first[at[d]] : lane_of[k[d] - r0];
}

// counts to offsets: h[0..n) exclusively summed (times unit), h[n] the total;
// the largest count
static int counts_to_offsets(int *h, int n, int unit) {
    int sum = 0, most = 0;
    for (int e = 0; e < n; e++) {
        const int c = h[e];
        h[e] = sum;
        sum += c * unit;
        most = std::max(most, c);
    }
    h[n] = sum;
    return most;
}

// ---------------------------------------------------------------------------
// numeric factorization of the rows of one level (block inverse:
// dev_block_inverse, device.hpp)
// ---------------------------------------------------------------------------
template <int BS>
__global__ __launch_bounds__(256) void k_ilu_factor_level(
    int first_lane, int nlanes, const int *__restrict__ perm, const int *__restrict__ rowptr,
    const int *__restrict__ col, const int *__restrict__ diag, double *__restrict__ lu,
    double *__restrict__ uinv, int *err) {
    constexpr int B2 = BS * BS;
    const int g = blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= nlanes) return;
    const int i = perm[first_lane + g];
    if (i < 0) return;
    const int p0 = rowptr[i], p1 = rowptr[i + 1], di = diag[i];
    for (int p = p0; p < di; p++) {
        const int k = col[p];
        double L[B2];
        const double *a = lu + (int64_t)p * B2;
        const double *ui = uinv + (int64_t)k * B2;
#pragma unroll
        for (int r = 0; r < BS; r++)
#pragma unroll
            for (int c = 0; c < BS; c++) {
                double s = 0.0;
#pragma unroll
                for (int q = 0; q < BS; q++) s += a[r * BS + q] * ui[q * BS + c];
                L[r * BS + c] = s;
            }
#pragma unroll
        for (int e = 0; e < B2; e++) lu[(int64_t)p * B2 + e] = L[e];
        // a_ij -= L_ik U_kj for j > k in row k with (i, j) in the pattern
        int sidx = p + 1;
        const int q1 = rowptr[k + 1];
        for (int q = diag[k] + 1; q < q1; q++) {
            const int j = col[q];
            while (sidx < p1 && col[sidx] < j) sidx++;
            if (sidx < p1 && col[sidx] == j) {
                const double *u = lu + (int64_t)q * B2;
                double *t = lu + (int64_t)sidx * B2;
#pragma unroll
                for (int r = 0; r < BS; r++)
#pragma unroll
                    for (int c = 0; c < BS; c++) {
                        double s = 0.0;
#pragma unroll
                        for (int m = 0; m < BS; m++) s += L[r * BS + m] * u[m * BS + c];
                        t[r * BS + c] -= s;
                    }
            }
        }
    }
    double D[B2], R[B2];
#pragma unroll
    for (int e = 0; e < B2; e++) D[e] = lu[(int64_t)di * B2 + e];
    if (!dev_block_inverse<BS>(D, R)) {
        __hip_atomic_store(err, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
        for (int e = 0; e < B2; e++) R[e] = 0.0;
    }
#pragma unroll
    for (int e = 0; e < B2; e++) uinv[(int64_t)i * B2 + e] = R[e];
}

// ---------------------------------------------------------------------------
// packing into level-ordered slices
// ---------------------------------------------------------------------------
// one sweep's slices: rows and slot offsets, where columns and values go
struct PackTarget {
    int nslices;
    const int *perm, *off;
    int *col;
    double *val;
};

// L (blockIdx.y = 0) and U with the inverses of its diagonal blocks
template <int BS>
__global__ void k_ilu_pack(PackTarget lower, PackTarget upper, const int *__restrict__ rowptr,
                           const int *__restrict__ diag, const int *__restrict__ col,
                           const double *__restrict__ lu, const double *__restrict__ uinv,
                           double *__restrict__ dinv) {
    constexpr int B2 = BS * BS;
    const bool up = blockIdx.y != 0;
    const PackTarget P = up ? upper : lower;
    const int g = blockIdx.x * blockDim.x + threadIdx.x;
    const int s = g >> 6, lane = g & 63;
    if (s >= P.nslices) return;
    const int row = P.perm[g];
    const int o0 = P.off[s], w = P.off[s + 1] - o0;
    int p0 = 0, len = 0;
    if (row >= 0) {
        p0 = up ? diag[row] + 1 : rowptr[row];
        len = up ? rowptr[row + 1] - p0 : diag[row] - p0;
    }
    for (int t = 0; t < w; t++) {
        const int64_t slot = o0 + t;
        const bool have = t < len;
        P.col[slot * 64 + lane] = have ? col[p0 + t] : -1;
#pragma unroll
        for (int e = 0; e < B2; e++)
            P.val[(slot * B2 + e) * 64 + lane] = have ? lu[(int64_t)(p0 + t) * B2 + e] : 0.0;
    }
    if (up) {
#pragma unroll
        for (int e = 0; e < B2; e++)
            dinv[((int64_t)s * B2 + e) * 64 + lane] = row >= 0 ? uinv[(int64_t)row * B2 + e] : 0.0;
    }
}

__global__ void k_round_f32(int64_t n, const double *__restrict__ x, float *__restrict__ y) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        y[i] = static_cast<float>(x[i]);
}

__global__ void k_round_bf16(int64_t n, const double *__restrict__ x, uint16_t *__restrict__ y) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        y[i] = f32_to_bf16_rne(static_cast<float>(x[i]));
}

// y unwritten, the counters zero
template <typename T>
__global__ void k_sweep_start(int64_t n, T *y, int *ctr) {
    if (blockIdx.x == 0 && threadIdx.x < 2 * GRID_QUEUES) ctr[threadIdx.x] = 0;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * blockDim.x)
        y[i] = sentinel_value<T>();
}

// ---------------------------------------------------------------------------
// sync-free sweeps
// ---------------------------------------------------------------------------
constexpr int CHUNK = 4;   // dependency slots loaded ahead of the waits

template <typename TC, typename TF>
__device__ __forceinline__ TC ldf(const TF *p) { return static_cast<TC>(*p); }
template <>
__device__ __forceinline__ float ldf<float, uint16_t>(const uint16_t *p) { return bf16_to_f32(*p); }

__device__ __forceinline__ int next_slice(int *ctr) {
    int s = 0;
    if ((threadIdx.x & 63) == 0) s = atomicAdd(ctr, 1);
    return __shfl(s, 0, 64);
}

// forward: y_i = b_i - sum_{k<i} L_ik y_k; also marks xo (the backward
// output) as unwritten.
template <int BS, typename TF, typename TC, typename TIN, typename TO>
__global__ __launch_bounds__(256) void k_ilu_fwd(
    int nslices, const int *__restrict__ perm, const int *__restrict__ off,
    const int *__restrict__ col, const TF *__restrict__ val, const TIN *__restrict__ b,
    TC *y, TO *xo, int *ctr, int *other_ctr, int *err) {
    constexpr int B2 = BS * BS;
    const int lane = threadIdx.x & 63;
    if (blockIdx.x == 0 && threadIdx.x == 0) *other_ctr = 0;
    for (;;) {
        const int s = next_slice(ctr);
        if (s >= nslices) break;
        const int row = perm[(int64_t)s * 64 + lane];
        if (row >= 0) {
            TC acc[BS];
#pragma unroll
            for (int r = 0; r < BS; r++) acc[r] = static_cast<TC>(b[(int64_t)row * BS + r]);
            const int o0 = off[s], o1 = off[s + 1];
            for (int t0 = o0; t0 < o1; t0 += CHUNK) {
                int cc[CHUNK];
                TC lv[CHUNK][B2];
#pragma unroll
                for (int q = 0; q < CHUNK; q++) {
                    const int t = t0 + q;
                    cc[q] = t < o1 ? col[(int64_t)t * 64 + lane] : -1;
#pragma unroll
                    for (int e = 0; e < B2; e++)
                        lv[q][e] = cc[q] >= 0 ? ldf<TC, TF>(val + ((int64_t)t * B2 + e) * 64 + lane)
                                              : TC(0);
                }
#pragma unroll
                for (int q = 0; q < CHUNK; q++) {
                    if (cc[q] >= 0) {
                        TC yc[BS];
                        wait_values<TC, BS>(y + (int64_t)cc[q] * BS, yc, err);
#pragma unroll
                        for (int r = 0; r < BS; r++)
#pragma unroll
                            for (int k = 0; k < BS; k++) acc[r] -= lv[q][r * BS + k] * yc[k];
                    }
                }
            }
#pragma unroll
            for (int r = 0; r < BS; r++) publish<TC>(y + (int64_t)row * BS + r, acc[r]);
#pragma unroll
            for (int r = 0; r < BS; r++) xo[(int64_t)row * BS + r] = sentinel_value<TO>();
        }
    }
}

// backward: x_i = U_ii^-1 (y_i - sum_{j>i} U_ij x_j); resets y for the next
// forward sweep.  ADD = 1: add_out = add_in + x; ADD = 2: add_out =
// (add_in[i], 0, 0) + x (pressure injection).
template <int BS, typename TF, typename TD, typename TC, typename TO, int ADD, typename TAI,
          typename TAO>
__global__ __launch_bounds__(256) void k_ilu_bwd(
    int nslices, const int *__restrict__ perm, const int *__restrict__ off,
    const int *__restrict__ col, const TF *__restrict__ val, const TD *__restrict__ dinv, TC *y,
    TO *xo, const TAI *__restrict__ add_in, TAO *__restrict__ add_out, int *ctr, int *other_ctr,
    int *err) {
    constexpr int B2 = BS * BS;
    const int lane = threadIdx.x & 63;
    if (blockIdx.x == 0 && threadIdx.x == 0) *other_ctr = 0;
    for (;;) {
        const int s = next_slice(ctr);
        if (s >= nslices) break;
        const int row = perm[(int64_t)s * 64 + lane];
        if (row >= 0) {
            TC acc[BS];
#pragma unroll
            for (int r = 0; r < BS; r++) {
                acc[r] = y[(int64_t)row * BS + r];
                y[(int64_t)row * BS + r] = sentinel_value<TC>();
            }
            TC dv[B2];
#pragma unroll
            for (int e = 0; e < B2; e++)
                dv[e] = static_cast<TC>(dinv[((int64_t)s * B2 + e) * 64 + lane]);
            const int o0 = off[s], o1 = off[s + 1];
            for (int t0 = o0; t0 < o1; t0 += CHUNK) {
                int cc[CHUNK];
                TC uv[CHUNK][B2];
#pragma unroll
                for (int q = 0; q < CHUNK; q++) {
                    const int t = t0 + q;
                    cc[q] = t < o1 ? col[(int64_t)t * 64 + lane] : -1;
#pragma unroll
                    for (int e = 0; e < B2; e++)
                        uv[q][e] = cc[q] >= 0 ? ldf<TC, TF>(val + ((int64_t)t * B2 + e) * 64 + lane)
                                              : TC(0);
                }
#pragma unroll
                for (int q = 0; q < CHUNK; q++) {
                    if (cc[q] >= 0) {
                        TO xr[BS];
                        wait_values<TO, BS>(xo + (int64_t)cc[q] * BS, xr, err);
#pragma unroll
                        for (int r = 0; r < BS; r++)
#pragma unroll
                            for (int k = 0; k < BS; k++)
                                acc[r] -= uv[q][r * BS + k] * static_cast<TC>(xr[k]);
                    }
                }
            }
            TC res[BS];
#pragma unroll
            for (int r = 0; r < BS; r++) {
                TC t = TC(0);
#pragma unroll
                for (int k = 0; k < BS; k++) t += dv[r * BS + k] * acc[k];
                res[r] = t;
            }
#pragma unroll
            for (int r = 0; r < BS; r++) {
                publish<TO>(xo + (int64_t)row * BS + r, static_cast<TO>(res[r]));
                if (ADD == 1)
                    add_out[(int64_t)row * BS + r] =
                        static_cast<TAO>(add_in[(int64_t)row * BS + r]) + static_cast<TAO>(res[r]);
                if (ADD == 2) {
                    TC base = (r == 0) ? static_cast<TC>(add_in[row]) : TC(0);
                    add_out[(int64_t)row * BS + r] = static_cast<TAO>(base + res[r]);
                }
            }
        }
    }
}

// ---------------------------------------------------------------------------
// sweeps over row blocks
//
// What bounds a level-by-level sweep is the chain of levels: a result has to
// reach the next level's wavefront through memory, about 1 us there and a
// poll back, and a row's dependencies one after another.  Here a workgroup
// owns RB_ROWS consecutive rows, which most dependencies of a matrix in a
// natural order stay inside of, and hands their results on through LDS: a
// level inside a block costs one turn of the loop below (an LDS read and the
// products) and only a step from block to block goes through memory.
//
// Each lane owns one row, with its factor entries in registers from the
// start, and looks for its dependencies on its own, so that lanes of a
// wavefront may depend on each other.  RB_IMPORT wavefronts fetch what the
// block reads of others into LDS: one vector element per lane, polled where
// its owner publishes it, in level order; only the first of them polls
// before the block's first import has arrived.
//
// Measured, 3x3 blocks in FP64: 0.3 us a level inside a block, 1-1.5 us from
// block to block; 60x52x41 cells with 12 % inactive (112 600 rows, 151
// levels) 535 -> 125 us a sweep.  Blocks of 128 rows are 15 % slower, of 512
// no faster; neither are 2 to 8 importing wavefronts or other poll intervals.
// ---------------------------------------------------------------------------
template <typename T>
__device__ __forceinline__ void lds_poke(T *p, T v) {
    using U = typename Bits<T>::U;
    __hip_atomic_store(reinterpret_cast<U *>(p), Bits<T>::to(v), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_WORKGROUP);
}

// true when the wait has to end: another wavefront raised the error flag or
// this one has waited for SPIN_LIMIT rounds
__device__ __forceinline__ bool spin_over(uint32_t it, int *err) {
    if ((it & 63u) != 63u) return false;
    const int e = __hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (e == 0 && it > SPIN_LIMIT)
        __hip_atomic_store(err, ERR_STALL_FLAG, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return e != 0 || it > SPIN_LIMIT;
}

__device__ __forceinline__ void wait_vector_memory() { __builtin_amdgcn_s_waitcnt(0x0f70); }  // vmcnt(0)

// 0 for the values that sentinel_like names
template <typename T>
__device__ __forceinline__ uint32_t sentinel_distance(T v) {
    using U = typename Bits<T>::U;
    constexpr int SH = static_cast<int>(sizeof(U)) * 8 - 32;
    return static_cast<uint32_t>(Bits<T>::to(v) >> SH) ^ static_cast<uint32_t>(Bits<T>::sentinel >> SH);
}

// wavefront `iw` of the importing ones: element n of the list goes to
// imp[n]; lanes advance on their own, each through a list of its own in LDS
template <typename T>
__device__ __forceinline__ void import_words(int iw, const int *__restrict__ list, int n, const T *src,
                                             T *imp, int *todo, int *started, int *err) {
    using U = typename Bits<T>::U;
    constexpr int STEP = RB_IMPORT * 64;
    const int lane = threadIdx.x & 63;
    if (iw * 64 >= n) return;
    int at = iw * 64 + lane;
    for (int m = at; m < n; m += STEP) todo[m] = list[m];
    wait_vector_memory();
    if (iw > 0)
        for (uint32_t it = 0; lds_get(started) == 0; ++it) {
            if (spin_over(it, err)) return;
            __builtin_amdgcn_s_sleep(4);
        }
    bool told = iw > 0;
    for (uint32_t it = 0; __any(at < n); ++it) {
        bool got = false;
        if (at < n) {
            const U u = __hip_atomic_load(reinterpret_cast<const U *>(src + todo[at]), __ATOMIC_RELAXED,
                                          __HIP_MEMORY_SCOPE_AGENT);
            if (!sentinel_like(Bits<T>::from(u))) {
                lds_poke(imp + at, Bits<T>::from(u));
                got = true;
                at += STEP;
            }
        }
        if (__any(got)) {
            it = 0;
            if (!told && lane == 0) lds_put(started, 1);
            told = true;
        } else if (spin_over(it, err)) {
            return;
        }
    }
}

// Waits until the lane's dependencies (LDS cells idx[0..W)) are all there,
// takes them off acc with the factor blocks f in slot order and calls
// done(acc) once; lanes go on their own, the wavefront leaves together.
// A value is there when its high word is not the sentinel's.
template <int BS, int W, typename T, typename TC, typename F>
__device__ __forceinline__ void take_deps(bool live, const int (&idx)[W], const TC (&f)[W][BS * BS],
                                          TC (&acc)[BS], const T *cells, int *err, F done) {
    // nothing is loaded in the loop: without this wait the compiler's own
    // ones in the loop would wait for its stores as well, 1 us each time
    wait_vector_memory();
    for (uint32_t it = 0;; ++it) {
        bool ready = live;
        if (live) {
            T v[W][BS];
            asm volatile("" ::: "memory");   // read them anew
#pragma unroll
            for (int q = 0; q < W; q++)
#pragma unroll
                for (int r = 0; r < BS; r++) v[q][r] = cells[idx[q] * BS + r];
            uint32_t low = 0xffffffffu;
#pragma unroll
            for (int q = 0; q < W; q++)
#pragma unroll
                for (int r = 0; r < BS; r++) low = min(low, sentinel_distance(v[q][r]));
            ready = low != 0;
            if (ready) {
#pragma unroll
                for (int q = 0; q < W; q++)
#pragma unroll
                    for (int r = 0; r < BS; r++)
#pragma unroll
                        for (int k = 0; k < BS; k++) acc[r] -= f[q][r * BS + k] * static_cast<TC>(v[q][k]);
                done(acc);
                live = false;
            }
        }
        if (!__any(live)) return;
        if (__any(ready)) {
            it = 0;
        } else {
            if (spin_over(it, err)) break;
            __builtin_amdgcn_s_sleep(1);
        }
    }
    if (live) {
#pragma unroll
        for (int r = 0; r < BS; r++) acc[r] = Bits<TC>::from(Bits<TC>::qnan);
        done(acc);
    }
}

// the block this workgroup takes; its LDS cells are all unwritten but for
// the last, which stands for the dependencies that a row does not have
template <int BS, typename T>
__device__ __forceinline__ int start_block(int *ctr, T *cells, int ncells, int *sh) {
    if (threadIdx.x == 0) {
        sh[0] = atomicAdd(ctr, 1);
        sh[1] = 0;
    }
    for (int c = threadIdx.x; c < ncells * BS; c += RB_THREADS)
        cells[c] = c < (ncells - 1) * BS ? sentinel_value<T>() : T(0);
    __syncthreads();
    return sh[0];
}

template <int BS, int W, typename TF, typename TC>
__device__ __forceinline__ void load_deps(int s, const int *__restrict__ off, const int *__restrict__ cell,
                                          const TF *__restrict__ val, int none, int (&idx)[W],
                                          TC (&f)[W][BS * BS]) {
    const int lane = threadIdx.x & 63;
    const int o0 = off[s], w = off[s + 1] - o0;
#pragma unroll
    for (int q = 0; q < W; q++) {
        const int c = q < w ? cell[(int64_t)(o0 + q) * 64 + lane] : -1;
        idx[q] = c >= 0 ? c : none;
#pragma unroll
        for (int e = 0; e < BS * BS; e++)
            f[q][e] = q < w ? ldf<TC, TF>(val + ((int64_t)(o0 + q) * BS * BS + e) * 64 + lane) : TC(0);
    }
}

// k_ilu_fwd over row blocks
template <int BS, int W, typename TF, typename TC, typename TIN, typename TO>
__global__ __launch_bounds__(RB_THREADS) void k_ilu_fwd_rows(
    int ncells, const int *__restrict__ perm, const int *__restrict__ off,
    const int *__restrict__ cell, const int *__restrict__ woff, const int *__restrict__ words,
    const TF *__restrict__ val, const TIN *__restrict__ b, TC *y, TO *xo, int *ctr, int *other_ctr,
    int *err) {
    extern __shared__ __align__(16) char smem[];
    __shared__ int sh[2];
    TC *cells = reinterpret_cast<TC *>(smem);
    if (blockIdx.x == 0 && threadIdx.x == 0) *other_ctr = 0;
    const int blk = start_block<BS>(ctr, cells, ncells, sh);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (wave >= RB_SLICES) {
        import_words<TC>(wave - RB_SLICES, words + woff[blk], woff[blk + 1] - woff[blk], y,
                         cells + RB_ROWS * BS, reinterpret_cast<int *>(cells + ncells * BS), sh + 1, err);
        return;
    }
    const int row = perm[(int64_t)blk * RB_ROWS + threadIdx.x];
    int idx[W];
    TC f[W][BS * BS], acc[BS];
    load_deps<BS, W, TF, TC>(blk * RB_SLICES + wave, off, cell, val, ncells - 1, idx, f);
#pragma unroll
    for (int r = 0; r < BS; r++) {
        acc[r] = row >= 0 ? static_cast<TC>(b[(int64_t)row * BS + r]) : TC(0);
        if (row >= 0) xo[(int64_t)row * BS + r] = sentinel_value<TO>();
    }
    take_deps<BS, W, TC, TC>(row >= 0, idx, f, acc, cells, err, [&](const TC (&a)[BS]) {
        TC v[BS];
        unsentinel<TC, BS>(a, v);
#pragma unroll
        for (int r = 0; r < BS; r++) lds_poke(cells + threadIdx.x * BS + r, v[r]);
        publish_checked<TC, BS>(y + (int64_t)row * BS, v);
    });
}

// k_ilu_bwd over row blocks
template <int BS, int W, typename TF, typename TD, typename TC, typename TO, int ADD, typename TAI,
          typename TAO>
__global__ __launch_bounds__(RB_THREADS) void k_ilu_bwd_rows(
    int ncells, const int *__restrict__ perm, const int *__restrict__ off,
    const int *__restrict__ cell, const int *__restrict__ woff, const int *__restrict__ words,
    const TF *__restrict__ val, const TD *__restrict__ dinv, TC *y, TO *xo,
    const TAI *__restrict__ add_in, TAO *__restrict__ add_out, int *ctr, int *other_ctr, int *err) {
    extern __shared__ __align__(16) char smem[];
    __shared__ int sh[2];
    TO *cells = reinterpret_cast<TO *>(smem);
    if (blockIdx.x == 0 && threadIdx.x == 0) *other_ctr = 0;
    const int blk = start_block<BS>(ctr, cells, ncells, sh);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (wave >= RB_SLICES) {
        import_words<TO>(wave - RB_SLICES, words + woff[blk], woff[blk + 1] - woff[blk], xo,
                         cells + RB_ROWS * BS, reinterpret_cast<int *>(cells + ncells * BS), sh + 1, err);
        return;
    }
    const int row = perm[(int64_t)blk * RB_ROWS + threadIdx.x];
    const int s = blk * RB_SLICES + wave, lane = threadIdx.x & 63;
    int idx[W];
    TC f[W][BS * BS], acc[BS], dv[BS * BS];
    load_deps<BS, W, TF, TC>(s, off, cell, val, ncells - 1, idx, f);
#pragma unroll
    for (int e = 0; e < BS * BS; e++)
        dv[e] = static_cast<TC>(dinv[((int64_t)s * BS * BS + e) * 64 + lane]);
#pragma unroll
    for (int r = 0; r < BS; r++) {
        acc[r] = row >= 0 ? y[(int64_t)row * BS + r] : TC(0);
        if (row >= 0) y[(int64_t)row * BS + r] = sentinel_value<TC>();
    }
    take_deps<BS, W, TO, TC>(row >= 0, idx, f, acc, cells, err, [&](const TC (&a)[BS]) {
        TC res[BS];
        TO x[BS], v[BS];
#pragma unroll
        for (int r = 0; r < BS; r++) {
            TC t = TC(0);
#pragma unroll
            for (int k = 0; k < BS; k++) t += dv[r * BS + k] * a[k];
            res[r] = t;
            x[r] = static_cast<TO>(t);
        }
        unsentinel<TO, BS>(x, v);
#pragma unroll
        for (int r = 0; r < BS; r++) lds_poke(cells + threadIdx.x * BS + r, v[r]);
        publish_checked<TO, BS>(xo + (int64_t)row * BS, v);
#pragma unroll
        for (int r = 0; r < BS; r++) {
            if (ADD == 1)
                add_out[(int64_t)row * BS + r] =
                    static_cast<TAO>(add_in[(int64_t)row * BS + r]) + static_cast<TAO>(res[r]);
            if (ADD == 2) {
                TC base = (r == 0) ? static_cast<TC>(add_in[row]) : TC(0);
                add_out[(int64_t)row * BS + r] = static_cast<TAO>(base + res[r]);
            }
        }
    });
}

// ---------------------------------------------------------------------------
// setup
// ---------------------------------------------------------------------------
static int sweep_waves_cap() {
    static int cap = -1;
    if (cap < 0) {
        const char *e = getenv("KRY_SWEEP_WAVES");
        cap = e ? std::max(4, atoi(e)) : 1024;
    }
    return cap;
}

static int upload_layout(hipStream_t s, const LevelSlices &L, Sell &S, int bs) {
    S.bs = bs;
    S.nslices = L.nslices;
    S.maxw = L.maxw;
    S.h_off = L.off;
    S.nslots = L.off[L.nslices];
    KRY_TRY(S.off.alloc(L.nslices + 1));
    KRY_TRY(S.perm.alloc((size_t)L.nslices * 64));
    KRY_TRY(S.col.alloc(std::max<int64_t>(1, S.nslots) * 64));
    KRY_TRY(S.val.alloc(std::max<int64_t>(1, S.nslots) * 64 * bs * bs));
    KRY_HIP(hipMemcpyAsync(S.off.p, L.off.data(), sizeof(int) * (L.nslices + 1),
                           hipMemcpyHostToDevice, s));
    KRY_HIP(hipMemcpyAsync(S.perm.p, L.perm.data(), sizeof(int) * L.perm.size(),
                           hipMemcpyHostToDevice, s));
    return KRY_OK;
}

// The row blocks of both sweeps up to their offsets, and the storage that
// these measure out: F.plan holds [off, woff] of the lower and of the upper
// blocks and the rows of their lanes, F.lists cells and words.  lev: the
// rows' forward and backward levels; h: the offsets, for as long as the
// stream may read them.
static int plan_row_blocks(hipStream_t s, const MAT_ *A, const int *lev, std::vector<int> &h, IluFactor &F) {
    const int nb = A->nb, bs = A->bs;
    const int nblk = (nb + RB_ROWS - 1) / RB_ROWS, ns = nblk * RB_SLICES, nh = ns + nblk + 2;
    KRY_TRY(F.plan.alloc(2 * ((size_t)nh + (size_t)nblk * RB_ROWS)));
    RowBlocks *const blocks[2] = {&F.Lrows, &F.Urows};
    for (int q = 0; q < 2; q++) {
        blocks[q]->off = F.plan.p + (size_t)q * nh;
        blocks[q]->woff = blocks[q]->off + ns + 1;
        blocks[q]->perm = F.plan.p + 2 * (size_t)nh + (size_t)q * nblk * RB_ROWS;
    }
    hipLaunchKernelGGL(k_row_blocks<false>, dim3(nblk, 2), dim3(RB_ROWS), 0, s, nb, bs, A->rowptr.p,
                       A->col.p, A->diag.p, lev, lev + nb, F.Lrows, F.Urows);
    KRY_HIP(hipGetLastError());
    h.resize(2 * (size_t)nh);
    KRY_HIP(hipMemcpyAsync(h.data(), F.plan.p, sizeof(int) * h.size(), hipMemcpyDeviceToHost, s));
    KRY_HIP(hipStreamSynchronize(s));
    int64_t cells[2], nlists = 0;
    Sell *const sell[2] = {&F.L, &F.U};
    for (int q = 0; q < 2; q++) {
        int *off = h.data() + (size_t)q * nh, *woff = off + ns + 1;
        Sell &S = *sell[q];
        S.bs = bs;
        S.nslices = ns;
        S.maxw = counts_to_offsets(off, ns, 1);
        S.nslots = off[ns];
        blocks[q]->imports = counts_to_offsets(woff, nblk, bs);
        blocks[q]->ncells = RB_ROWS + blocks[q]->imports + 1;
        cells[q] = std::max<int64_t>(1, S.nslots) * 64;
        nlists += cells[q] + std::max(1, woff[nblk]);
        KRY_TRY(S.val.alloc(cells[q] * bs * bs));
    }
    KRY_TRY(F.lists.alloc(nlists));
    F.Lrows.cell = F.lists.p;
    F.Urows.cell = F.Lrows.cell + cells[0];
    F.Lrows.words = F.Urows.cell + cells[1];
    F.Urows.words = F.Lrows.words + std::max(1, h[ns + 1 + nblk]);
    KRY_HIP(hipMemcpyAsync(F.plan.p, h.data(), sizeof(int) * h.size(), hipMemcpyHostToDevice, s));
    return KRY_OK;
}

int ilu_setup(hipStream_t s, const MAT_ *A, const double *d_val, IluFactor &F, int prec,
              int *d_err, int layout) {
    const int nb = A->nb, bs = A->bs, b2 = bs * bs;
    const std::vector<int> &rp = A->h_rowptr, &ci = A->h_col, &dg = A->h_diag;
    F.bs = bs;
    F.nb = nb;
    F.prec = prec;
    if (layout == KRY_SWEEP_GRID && A->gnx == 0)
        return set_error(KRY_ERR_ARG, "grid sweep layout requested for a matrix that is not a 7-point grid stencil");
    const bool use_grid = layout == KRY_SWEEP_GRID || (layout == KRY_SWEEP_AUTO && A->gnx > 0);
    if (use_grid && ilu_grid_can_factor(A)) {
        // no level analysis: the grid-tiled factorization writes the sweep
        // layout directly
        F.nlev_f = F.nlev_b = A->gnx + A->gny + A->gnz - 2;
        KRY_TRY(ilu_grid_factor_setup(s, A, d_val, F, d_err));
        KRY_TRY(F.ctr.alloc(2 * GRID_QUEUES));
        KRY_HIP(hipMemsetAsync(F.ctr.p, 0, 2 * GRID_QUEUES * sizeof(int), s));
        KRY_HIP(hipStreamSynchronize(s));
        return KRY_OK;
    }
    // level sets
    std::vector<int> levf(nb, 0), levb(nb, 0);
    int nlf = 0, nlb = 0;
    for (int i = 0; i < nb; i++) {
        int l = 0;
        for (int p = rp[i]; p < dg[i]; p++) l = std::max(l, levf[ci[p]] + 1);
        levf[i] = l;
        nlf = std::max(nlf, l + 1);
    }
    for (int i = nb - 1; i >= 0; i--) {
        int l = 0;
        for (int p = dg[i] + 1; p < rp[i + 1]; p++) l = std::max(l, levb[ci[p]] + 1);
        levb[i] = l;
        nlb = std::max(nlb, l + 1);
    }
    F.nlev_f = nlf;
    F.nlev_b = nlb;
    // Rows with at most RB_WIDE dependencies (every stencil of the reservoir
    // systems, with holes and a few extra connections) are swept by row
    // blocks.  An application, level by level -> row blocks (3x3 blocks, FP64):
    // 60x52x41 with 12 % of the cells inactive 1090 -> 285 us.  Locality is not
    // asked for, since orders that put most dependencies in other blocks gain
    // too, if less: the same in random order 254 -> 100 us, 128x128x96 in
    // random order 855 -> 773 us, red-black 647 -> 500 us, six distant
    // dependencies a row (200 000 rows) 2395 -> 1050 us.  The lanes hold the
    // entries in registers: six 3x3 blocks in FP64 take 188 of the 256 that a
    // workgroup of eight wavefronts can have.  Wider rows are swept level by
    // level, and a single one sends the whole matrix there.
    int wide = 0;
    for (int i = 0; i < nb; i++) wide = std::max(wide, std::max(dg[i] - rp[i], rp[i + 1] - dg[i] - 1));
    F.rows = !use_grid && wide <= RB_WIDE;
    LevelSlices LF, LB;
    build_slices(nb, levf, nlf, [&](int r) { return dg[r] - rp[r]; }, LF);
    if (!use_grid && !F.rows) {
        build_slices(nb, levb, nlb, [&](int r) { return rp[r + 1] - dg[r] - 1; }, LB);
        const bool ok = schedule_is_acyclic(nb, LF, [&](int i, auto f) {
                            for (int p = rp[i]; p < dg[i]; p++) f(ci[p]);
                        }) &&
                        schedule_is_acyclic(nb, LB, [&](int i, auto f) {
                            for (int p = dg[i] + 1; p < rp[i + 1]; p++) f(ci[p]);
                        });
        if (!ok) return set_error(KRY_ERR_ARG, "ILU: inconsistent level schedule");
        KRY_TRY(upload_layout(s, LF, F.L, bs));
        KRY_TRY(upload_layout(s, LB, F.U, bs));
    }
    // the levels' rows, which the factorization walks, and (row blocks) the
    // rows' levels, in one copy
    DBuf<int> levels;
    std::vector<int> &up = LF.perm, offsets;
    const size_t np = up.size();
    const int *level_perm = F.L.perm.p;
    if (use_grid || F.rows) {
        if (F.rows) {
            up.insert(up.end(), levf.begin(), levf.end());
            up.insert(up.end(), levb.begin(), levb.end());
        }
        KRY_TRY(levels.alloc(up.size()));
        level_perm = levels.p;
        KRY_HIP(hipMemcpyAsync(levels.p, up.data(), sizeof(int) * up.size(), hipMemcpyHostToDevice, s));
        if (F.rows) KRY_TRY(plan_row_blocks(s, A, levels.p + np, offsets, F));
    }

    // numeric factorization on a working copy of the values
    DBuf<double> lu, uinv;
    KRY_TRY(lu.alloc((size_t)A->nnzb * b2));
    KRY_TRY(uinv.alloc((size_t)nb * b2));
    KRY_HIP(hipMemcpyAsync(lu.p, d_val, sizeof(double) * A->nnzb * b2, hipMemcpyDeviceToDevice, s));
    for (int l = 0; l < nlf; l++) {
        const int first = LF.lev_slice[l] * 64;
        const int nl = (LF.lev_slice[l + 1] - LF.lev_slice[l]) * 64;
        dim3 g((nl + 255) / 256);
        if (bs == 1)
            hipLaunchKernelGGL(k_ilu_factor_level<1>, g, dim3(256), 0, s, first, nl, level_perm,
                               A->rowptr.p, A->col.p, A->diag.p, lu.p, uinv.p, d_err);
        else
            hipLaunchKernelGGL(k_ilu_factor_level<3>, g, dim3(256), 0, s, first, nl, level_perm,
                               A->rowptr.p, A->col.p, A->diag.p, lu.p, uinv.p, d_err);
    }
    KRY_HIP(hipGetLastError());

    if (use_grid) {
        KRY_TRY(ilu_grid_setup(s, A, lu.p, uinv.p, F));
    } else {
    // pack L and U (+ diagonal inverses) in level order
    KRY_TRY(F.dinv.alloc((size_t)F.U.nslices * 64 * b2));
    {
        const PackTarget lo = F.rows ? PackTarget{F.L.nslices, F.Lrows.perm, F.Lrows.off, F.Lrows.cell, F.L.val.p}
                                     : PackTarget{F.L.nslices, F.L.perm.p, F.L.off.p, F.L.col.p, F.L.val.p};
        const PackTarget hi = F.rows ? PackTarget{F.U.nslices, F.Urows.perm, F.Urows.off, F.Urows.cell, F.U.val.p}
                                     : PackTarget{F.U.nslices, F.U.perm.p, F.U.off.p, F.U.col.p, F.U.val.p};
        const dim3 g((std::max(F.L.nslices, F.U.nslices) * 64 + 255) / 256, 2);
        hipLaunchKernelGGL(bs == 1 ? k_ilu_pack<1> : k_ilu_pack<3>, g, dim3(256), 0, s, lo, hi, A->rowptr.p,
                           A->diag.p, A->col.p, lu.p, uinv.p, F.dinv.p);
        if (F.rows)   // cells in the place of the packed columns
            hipLaunchKernelGGL(k_row_blocks<true>, dim3(F.L.nslices / RB_SLICES, 2), dim3(RB_ROWS), 0, s, nb,
                               bs, A->rowptr.p, A->col.p, A->diag.p, levels.p + np,
                               levels.p + np + nb, F.Lrows, F.Urows);
        KRY_HIP(hipGetLastError());
    }
    // reduced-precision copies: off-diagonal blocks to FP32 or BF16,
    // diagonal inverses to FP32
    if (prec != KRY_PREC_F64) {
        const int64_t nl = std::max<int64_t>(1, F.L.nslots) * 64 * b2;
        const int64_t nu = std::max<int64_t>(1, F.U.nslots) * 64 * b2;
        const int64_t nd = (int64_t)F.U.nslices * 64 * b2;
        KRY_TRY(F.dinvf.alloc(nd));
        hipLaunchKernelGGL(k_round_f32, dim3(1024), dim3(256), 0, s, nd, F.dinv.p, F.dinvf.p);
        if (prec == KRY_PREC_F32) {
            KRY_TRY(F.L.valf.alloc(nl));
            KRY_TRY(F.U.valf.alloc(nu));
            hipLaunchKernelGGL(k_round_f32, dim3(1024), dim3(256), 0, s, nl, F.L.val.p, F.L.valf.p);
            hipLaunchKernelGGL(k_round_f32, dim3(1024), dim3(256), 0, s, nu, F.U.val.p, F.U.valf.p);
        } else {
            KRY_TRY(F.L.valh.alloc(nl));
            KRY_TRY(F.U.valh.alloc(nu));
            hipLaunchKernelGGL(k_round_bf16, dim3(1024), dim3(256), 0, s, nl, F.L.val.p, F.L.valh.p);
            hipLaunchKernelGGL(k_round_bf16, dim3(1024), dim3(256), 0, s, nu, F.U.val.p, F.U.valh.p);
        }
        KRY_HIP(hipGetLastError());
        // the FP64 planes are not needed by a reduced-precision apply
        F.L.val.release();
        F.U.val.release();
        F.dinv.release();
    }
    }
    // sweep state: forward output all-unwritten, counters zero
    const int64_t n = (int64_t)nb * bs;
    KRY_TRY(F.ctr.alloc(2 * GRID_QUEUES));
    if (prec == KRY_PREC_F64) {
        KRY_TRY(F.y64.alloc(n));
        hipLaunchKernelGGL(k_sweep_start<double>, dim3(1024), dim3(256), 0, s, n, F.y64.p, F.ctr.p);
    } else {
        KRY_TRY(F.y32.alloc(n));
        hipLaunchKernelGGL(k_sweep_start<float>, dim3(1024), dim3(256), 0, s, n, F.y32.p, F.ctr.p);
    }
    KRY_HIP(hipGetLastError());
    F.grid_waves = std::min(std::max(F.L.nslices, F.U.nslices), sweep_waves_cap());
    // the working copy is freed on return: wait for the kernels using it
    KRY_HIP(hipStreamSynchronize(s));
    return KRY_OK;
}

// ---------------------------------------------------------------------------
// apply
// ---------------------------------------------------------------------------
const char *sweep_timer_name(bool fwd, int bs, int factor_bytes, int add_mode) {
    // [bs == 3][precision f64/f32/bf16][fwd, bwd, bwd+add1, bwd+add2]
    static const char *const names[2][3][4] = {
        {{"ilu_fwd_csr_f64", "ilu_bwd_csr_f64", "ilu_bwd_csr_f64_add", "ilu_bwd_csr_f64_inject"},
         {"ilu_fwd_csr_f32", "ilu_bwd_csr_f32", "ilu_bwd_csr_f32_add", "ilu_bwd_csr_f32_inject"},
         {"ilu_fwd_csr_bf16", "ilu_bwd_csr_bf16", "ilu_bwd_csr_bf16_add", "ilu_bwd_csr_bf16_inject"}},
        {{"ilu_fwd_bsr3_f64", "ilu_bwd_bsr3_f64", "ilu_bwd_bsr3_f64_add", "ilu_bwd_bsr3_f64_inject"},
         {"ilu_fwd_bsr3_f32", "ilu_bwd_bsr3_f32", "ilu_bwd_bsr3_f32_add", "ilu_bwd_bsr3_f32_inject"},
         {"ilu_fwd_bsr3_bf16", "ilu_bwd_bsr3_bf16", "ilu_bwd_bsr3_bf16_add", "ilu_bwd_bsr3_bf16_inject"}},
    };
    const int p = factor_bytes == 8 ? 0 : factor_bytes == 4 ? 1 : 2;
    return names[bs == 3][p][fwd ? 0 : 1 + add_mode];
}

template <int BS, int W, typename TF, typename TD, typename TC, typename TIN, typename TO, int ADD,
          typename TAI, typename TAO>
static int sweep_rows(hipStream_t s, IluFactor &F, const TF *lval, const TF *uval, const TD *dinv,
                      TC *y, const TIN *b, TO *xo, const TAI *add_in, TAO *add_out, int *err) {
    const dim3 grid(F.L.nslices / RB_SLICES), block(RB_THREADS);
    {
        TimedScope t(F.timer_fwd ? F.timer_fwd : sweep_timer_name(true, BS, sizeof(TF), ADD), s);
        hipLaunchKernelGGL((k_ilu_fwd_rows<BS, W, TF, TC, TIN, TO>), grid, block,
                           F.Lrows.lds_bytes(BS, sizeof(TC)), s, F.Lrows.ncells, F.Lrows.perm,
                           F.Lrows.off, F.Lrows.cell, F.Lrows.woff, F.Lrows.words, lval, b, y, xo,
                           F.ctr.p, F.ctr.p + 1, err);
    }
    {
        TimedScope t(F.timer_bwd ? F.timer_bwd : sweep_timer_name(false, BS, sizeof(TF), ADD), s);
        hipLaunchKernelGGL((k_ilu_bwd_rows<BS, W, TF, TD, TC, TO, ADD, TAI, TAO>), grid, block,
                           F.Urows.lds_bytes(BS, sizeof(TO)), s, F.Urows.ncells, F.Urows.perm,
                           F.Urows.off, F.Urows.cell, F.Urows.woff, F.Urows.words, uval, dinv, y, xo,
                           add_in, add_out, F.ctr.p + 1, F.ctr.p, err);
    }
    KRY_HIP(hipGetLastError());
    return KRY_OK;
}

template <int BS, typename TF, typename TD, typename TC, typename TIN, typename TO, int ADD,
          typename TAI, typename TAO>
static int sweep_pair(hipStream_t s, IluFactor &F, const TF *lval, const TF *uval, const TD *dinv,
                      TC *y, const TIN *b, TO *xo, const TAI *add_in, TAO *add_out, int *err) {
    if (F.rows) {
        // three dependencies a row: a 7-point stencil's
        auto sweep = std::max(F.L.maxw, F.U.maxw) <= 3
                         ? sweep_rows<BS, 3, TF, TD, TC, TIN, TO, ADD, TAI, TAO>
                         : sweep_rows<BS, RB_WIDE, TF, TD, TC, TIN, TO, ADD, TAI, TAO>;
        return sweep(s, F, lval, uval, dinv, y, b, xo, add_in, add_out, err);
    }
    const dim3 grid((F.grid_waves + 3) / 4), block(256);
    {
        TimedScope t(F.timer_fwd ? F.timer_fwd : sweep_timer_name(true, BS, sizeof(TF), ADD), s);
        hipLaunchKernelGGL((k_ilu_fwd<BS, TF, TC, TIN, TO>), grid, block, 0, s, F.L.nslices,
                           F.L.perm.p, F.L.off.p, F.L.col.p, lval, b, y, xo, F.ctr.p,
                           F.ctr.p + 1, err);
    }
    {
        TimedScope t(F.timer_bwd ? F.timer_bwd : sweep_timer_name(false, BS, sizeof(TF), ADD), s);
        hipLaunchKernelGGL((k_ilu_bwd<BS, TF, TD, TC, TO, ADD, TAI, TAO>), grid, block, 0, s,
                           F.U.nslices, F.U.perm.p, F.U.off.p, F.U.col.p, uval, dinv, y, xo,
                           add_in, add_out, F.ctr.p + 1, F.ctr.p, err);
    }
    KRY_HIP(hipGetLastError());
    return KRY_OK;
}

// dispatch on the factor precision, then the vector types
template <int BS, typename TIN, typename TO>
static int apply_typed(hipStream_t s, IluFactor &F, const TIN *b, TO *xo, int add_mode,
                       const void *add_in, void *add_out, int *err) {
    if (F.prec == KRY_PREC_F64) {
        using TC = double;
        if (add_mode == 0)
            return sweep_pair<BS, double, double, TC, TIN, TO, 0, double, double>(
                s, F, F.L.val.p, F.U.val.p, F.dinv.p, F.y64.p, b, xo, nullptr, nullptr, err);
        if (add_mode == 1)
            return sweep_pair<BS, double, double, TC, TIN, TO, 1, TO, TO>(
                s, F, F.L.val.p, F.U.val.p, F.dinv.p, F.y64.p, b, xo, (const TO *)add_in,
                (TO *)add_out, err);
        return sweep_pair<BS, double, double, TC, TIN, TO, 2, TC, double>(
            s, F, F.L.val.p, F.U.val.p, F.dinv.p, F.y64.p, b, xo, (const TC *)add_in,
            (double *)add_out, err);
    }
    using TC = float;
    if (F.prec == KRY_PREC_F32) {
        if (add_mode == 0)
            return sweep_pair<BS, float, float, TC, TIN, TO, 0, float, float>(
                s, F, F.L.valf.p, F.U.valf.p, F.dinvf.p, F.y32.p, b, xo, nullptr, nullptr, err);
        if (add_mode == 1)
            return sweep_pair<BS, float, float, TC, TIN, TO, 1, TO, TO>(
                s, F, F.L.valf.p, F.U.valf.p, F.dinvf.p, F.y32.p, b, xo, (const TO *)add_in,
                (TO *)add_out, err);
        return sweep_pair<BS, float, float, TC, TIN, TO, 2, TC, double>(
            s, F, F.L.valf.p, F.U.valf.p, F.dinvf.p, F.y32.p, b, xo, (const TC *)add_in,
            (double *)add_out, err);
    }
    if (add_mode == 0)
        return sweep_pair<BS, uint16_t, float, TC, TIN, TO, 0, float, float>(
            s, F, F.L.valh.p, F.U.valh.p, F.dinvf.p, F.y32.p, b, xo, nullptr, nullptr, err);
    if (add_mode == 1)
        return sweep_pair<BS, uint16_t, float, TC, TIN, TO, 1, TO, TO>(
            s, F, F.L.valh.p, F.U.valh.p, F.dinvf.p, F.y32.p, b, xo, (const TO *)add_in,
            (TO *)add_out, err);
    return sweep_pair<BS, uint16_t, float, TC, TIN, TO, 2, TC, double>(
        s, F, F.L.valh.p, F.U.valh.p, F.dinvf.p, F.y32.p, b, xo, (const TC *)add_in,
        (double *)add_out, err);
}

template <int BS>
static int apply_bs(hipStream_t s, IluFactor &F, const void *b, int in_type, void *xscr,
                    int out_type, int add_mode, const void *add_in, void *add_out, int *err) {
    if (in_type == 0 && out_type == 0)
        return apply_typed<BS>(s, F, (const double *)b, (double *)xscr, add_mode, add_in, add_out, err);
    if (in_type == 0 && out_type == 1)
        return apply_typed<BS>(s, F, (const double *)b, (float *)xscr, add_mode, add_in, add_out, err);
    if (in_type == 1 && out_type == 0)
        return apply_typed<BS>(s, F, (const float *)b, (double *)xscr, add_mode, add_in, add_out, err);
    return apply_typed<BS>(s, F, (const float *)b, (float *)xscr, add_mode, add_in, add_out, err);
}

int ilu_apply(hipStream_t s, IluFactor &F, const void *b, int in_type, void *xscr, int out_type,
              int add_mode, const void *add_in, void *add_out, int *d_err) {
    if (F.nb == 0) return set_error(KRY_ERR_ARG, "ILU apply before setup");
    if (F.grid)
        return ilu_grid_apply(s, F, b, in_type, xscr, out_type, add_mode, add_in, add_out, d_err);
    if (F.bs == 1) return apply_bs<1>(s, F, b, in_type, xscr, out_type, add_mode, add_in, add_out, d_err);
    return apply_bs<3>(s, F, b, in_type, xscr, out_type, add_mode, add_in, add_out, d_err);
}

}  // namespace kry
