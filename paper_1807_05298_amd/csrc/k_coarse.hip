// Dense inverse of the coarsest pressure level (n <= kCoarseReg cells) in one
// launch of one workgroup: the 7-point rows are expanded, the matrix is
// inverted in place by Gauss-Jordan with partial pivoting, and the inverse is written row-major and transposed, in FP64 and FP32.
//
// Bound: a serial chain of n steps on one compute unit, each with the pivot
// search, a division and a rank-1 update.  The matrix therefore stays in
// registers, thread (ty, tx) of 16 x 16 holding rows ty + 16 i and columns
// tx + 16 j; a step reads the pivot column and row from LDS, where the owners
// left them after the step before (two buffers), so it costs one barrier.
// Only a step that exchanges rows, which the search finds by a ballot before
// it looks for the largest entry, adds another.  In place, the columns of the
// identity that the augmented form carries along are not stored or updated,
// and the build and the copies to the compact forms have no launches.
// 256 threads, as a larger workgroup waits for one compute unit with that
// many free wave slots while the smoother's set-up fills the GPU.
// Measured, one inverse on an otherwise busy GPU (the augmented matrix in LDS
// with four barriers a step, and the other two launches, before): 54 cells
// 28 us (143 + 9), 84 cells 61 to 73 us by what runs beside it (347 + 9);
// eight of 84 cells side by side 56 us (327 + 10).  Above kCoarseReg cells a
// thread's tile would not fit its registers, and k_gauss_jordan keeps the
// matrix in memory.
#include "pf_internal.h"

namespace pf {
namespace {

constexpr int kGjSide = 16;                           // thread grid of kGjSide^2
constexpr int kGjThreads = kGjSide * kGjSide;
constexpr int kGjTiles = kCoarseReg / kGjSide;        // rows and columns of a thread

struct GjShared {
    // the pivot column by (row mod 16, tile) and the pivot row by (column mod
    // 16, tile), in the tile order of the registers; a row to be exchanged
    alignas(16) double col[2 * kCoarseReg], row[2 * kCoarseReg], swap[kCoarseReg];
    int piv[kCoarseReg], order[kCoarseReg], place[kCoarseReg];
};

// Row (at least k) of the largest |f|, the lowest of equals (NaN never chosen;
// k when there is nothing else).  f[i]: row ty + 16 (i + kt) for i < tiles;
// the lanes of each wavefront hold every row, so all find the same one.
template <int TM>
__device__ __forceinline__ int gj_pivot(const double (&f)[TM], int tiles, int kt, int ty, int k, int n) {
    double best = -1.0;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int r = ty + kGjSide * (i + kt);
        if (i < tiles && r >= k && r < n) best = fmax(best, fabs(f[i]));      // fmax drops a NaN
    }
    for (int o = 32; o > 0; o >>= 1) best = fmax(best, __shfl_xor(best, o, 64));
    int p = n;
#pragma unroll
    for (int i = TM - 1; i >= 0; --i) {
        const int r = ty + kGjSide * (i + kt);
        if (i < tiles && r >= k && r < n && fabs(f[i]) == best) p = r;
    }
    for (int o = 32; o > 0; o >>= 1) p = min(p, __shfl_xor(p, o, 64));
    return p < n ? p : k;
}

// n <= 16 TM
template <int TM>
__device__ __forceinline__ void gauss_jordan(const Dims& g, int n, const double* __restrict__ A,
                                             double* __restrict__ inv, double* __restrict__ invt,
                                             float* __restrict__ inv32, float* __restrict__ invt32, GjShared& sh) {
    const int tid = threadIdx.x, tx = tid / kGjSide, ty = tid & (kGjSide - 1);
    const int gxy = g.nx * g.ny;
    double a[TM][TM];
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const int r = ty + kGjSide * i;
        const int iz = r / gxy, rem = r - iz * gxy, iy = rem / g.nx, ix = rem - iy * g.nx;
        // on one-cell-wide grids distances coincide, so each face is tested for itself
        const bool ex[7] = {true, ix > 0, ix + 1 < g.nx, iy > 0, iy + 1 < g.ny, iz > 0, iz + 1 < g.nz};
        const int at[7] = {0, -1, 1, -g.nx, g.nx, -gxy, gxy};
        double v[7];
#pragma unroll
        for (int q = 0; q < 7; ++q) v[q] = A[q * n + (r < n ? r : 0)];
#pragma unroll
        for (int j = 0; j < TM; ++j) {
            const int d = tx + kGjSide * j - r;
            a[i][j] = 0.0;
#pragma unroll
            for (int q = 0; q < 7; ++q)
                if (d == at[q] && ex[q] && r < n) a[i][j] += v[q];
        }
    }
    double* const my_col = &sh.col[ty * TM];       // this thread's rows of the pivot column
    double* const my_row = &sh.row[tx * TM];       // and columns of the pivot row
    for (int r = tid; r < n; r += kGjThreads) sh.piv[r] = r;
    if (tx == 0)
#pragma unroll
        for (int i = 0; i < TM; ++i) my_col[i] = a[i][0];
    if (ty == 0)
#pragma unroll
        for (int j = 0; j < TM; ++j) my_row[j] = a[0][j];
    __syncthreads();
    bool swapped = false;
    for (int kt = 0; kt * kGjSide < n; ++kt) {
        // The tiles are renumbered as the pivot passes from one to the next, so
        // that it is always tile 0 of its owners (registers have fixed names,
        // and a copy of the step for each tile would make the code six times as
        // long): register (i, j) holds tile ((i + kt) % TM, (j + kt) % TM).
        const int steps = min(kGjSide, n - kt * kGjSide);
        for (int kk = 0; kk < steps; ++kk) {
            const int k = kGjSide * kt + kk, cur = (k & 1) * kCoarseReg;
            double f[TM], pk[TM];
            const double akk = sh.col[cur + kk * TM];
#pragma unroll
            for (int i = 0; i < TM; ++i) f[i] = my_col[cur + i];
#pragma unroll
            for (int j = 0; j < TM; ++j) pk[j] = my_row[cur + j];
            double inv_p = 1.0 / akk;
            // the rows from k on: those of tile 0 below it and the tiles up to the last (the padding rows are zero)
            bool larger = ty > kk && !(fabs(akk) >= fabs(f[0]));
#pragma unroll
            for (int i = 1; i < TM; ++i) larger |= i + kt < TM && !(fabs(akk) >= fabs(f[i]));
            if (__ballot(larger) != 0) {
                // some entry is larger (or NaN)
                const int p = __builtin_amdgcn_readfirstlane(gj_pivot<TM>(f, TM - kt, kt, ty, k, n));
                if (p != k) {
                    // exchange rows k and p: row p becomes the pivot row, its owners take row k
                    swapped = true;
                    const int ps = p & (kGjSide - 1), pi = p / kGjSide - kt;      // p >= k: not renumbered past 0
                    if (tid == 0) sh.piv[k] = p;
                    inv_p = 1.0 / sh.col[cur + ps * TM + pi];
                    if (ty == ps)
#pragma unroll
                        for (int i = 0; i < TM; ++i)
                            if (i == pi) {
                                f[i] = akk;
#pragma unroll
                                for (int j = 0; j < TM; ++j) {
                                    sh.swap[tx * TM + j] = a[i][j];
                                    a[i][j] = pk[j];
                                }
                            }
                    __syncthreads();
#pragma unroll
                    for (int j = 0; j < TM; ++j) pk[j] = sh.swap[tx * TM + j];
                }
            }
            // the pivot column leaves as the identity's: 1 in the pivot row, 0 elsewhere
            if (tx == kk) {
                pk[0] = 1.0;
#pragma unroll
                for (int i = 0; i < TM; ++i) a[i][0] = 0.0;
            }
            // the pivot row itself becomes pk / pivot: 0 - (-1) pk / pivot
            if (ty == kk) {
                f[0] = -1.0;
#pragma unroll
                for (int j = 0; j < TM; ++j) a[0][j] = 0.0;
            }
#pragma unroll
            for (int j = 0; j < TM; ++j) {
                pk[j] *= inv_p;
#pragma unroll
                for (int i = 0; i < TM; ++i) a[i][j] -= f[i] * pk[j];
            }
            // column and row k + 1 for the next step (of the next tile: below)
            if (tx == kk + 1)
#pragma unroll
                for (int i = 0; i < TM; ++i) my_col[kCoarseReg - cur + i] = a[i][0];
            if (ty == kk + 1)
#pragma unroll
                for (int j = 0; j < TM; ++j) my_row[kCoarseReg - cur + j] = a[0][j];
            __syncthreads();
        }
        // to the next tile
        double t[TM][TM];
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TM; ++j) t[i][j] = a[(i + 1) % TM][(j + 1) % TM];
#pragma unroll
        for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TM; ++j) a[i][j] = t[i][j];
        if (tx == 0)
#pragma unroll
            for (int i = 0; i < TM; ++i) my_col[i] = a[i][0];
        if (ty == 0)
#pragma unroll
            for (int j = 0; j < TM; ++j) my_row[j] = a[0][j];
        __syncthreads();
    }
    if (swapped) {
        // the row exchanges, undone on the columns in reverse order
        if (tid == 0) {
            for (int c = 0; c < n; ++c) sh.order[c] = c;
            for (int k = n - 1; k >= 0; --k) {
                const int q = sh.order[k], p = sh.piv[k];
                sh.order[k] = sh.order[p];
                sh.order[p] = q;
            }
            for (int c = 0; c < n; ++c) sh.place[sh.order[c]] = c;
        }
        __syncthreads();
    }
    // the padded rows of the transpose are read as zeros (k_mg_tail)
    for (int q = n * n + tid; q < n * ((n + kCoarsePad - 1) / kCoarsePad * kCoarsePad); q += kGjThreads) {
        invt[q] = 0.0;
        if (inv32) invt32[q] = 0.0f;
    }
#pragma unroll
    for (int j = 0; j < TM; ++j) {
        const int c0 = tx + kGjSide * j;
        if (c0 >= n) continue;
        const int c = swapped ? sh.place[c0] : c0;
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const int r = ty + kGjSide * i;
            if (r >= n) continue;
            inv[r * n + c] = a[i][j];
            invt[c * n + r] = a[i][j];
            if (inv32) {
                inv32[r * n + c] = (float)a[i][j];
                invt32[c * n + r] = (float)a[i][j];
            }
        }
    }
}

__device__ __forceinline__ void k_coarse_inverse_d(const Blk&, Dims g, const double* __restrict__ A,
                                                   double* __restrict__ inv, double* __restrict__ invt,
                                                   float* __restrict__ inv32, float* __restrict__ invt32) {
    __shared__ GjShared sh;
    const int n = g.nx * g.ny * g.nz;
    static_assert(kGjTiles == 6, "one case per tile count");
    switch ((n + kGjSide - 1) / kGjSide) {
        case 1: gauss_jordan<1>(g, n, A, inv, invt, inv32, invt32, sh); break;
        case 2: gauss_jordan<2>(g, n, A, inv, invt, inv32, invt32, sh); break;
        case 3: gauss_jordan<3>(g, n, A, inv, invt, inv32, invt32, sh); break;
        case 4: gauss_jordan<4>(g, n, A, inv, invt, inv32, invt32, sh); break;
        case 5: gauss_jordan<5>(g, n, A, inv, invt, inv32, invt32, sh); break;
        default: gauss_jordan<6>(g, n, A, inv, invt, inv32, invt32, sh); break;
    }
}
__global__ __launch_bounds__(kGjThreads) void k_coarse_inverse(Dims g, const double* __restrict__ A,
                                                               double* __restrict__ inv, double* __restrict__ invt,
                                                               float* __restrict__ inv32, float* __restrict__ invt32) {
    k_coarse_inverse_d(PF_BLK, g, A, inv, invt, inv32, invt32);
}
struct F_k_coarse_inverse {
    static constexpr int kLB = kGjThreads;
    template <class... A>
    __device__ __forceinline__ void operator()(const Blk& wg, const A&... a) const {
        k_coarse_inverse_d(wg, a...);
    }
};

}  // namespace

void launch_coarse_inverse(Sim& s, hipStream_t st) {
    const MGLevel& L = s.mg.back();
    const bool mixed = s.opts.precision == PF_PREC_MIXED;
    launch<F_k_coarse_inverse>(s, st, k_coarse_inverse, dim3(1), dim3(kGjThreads), 0, Dims{L.nx, L.ny, L.nz, L.split},
                               (const double*)L.A, s.coarse_inv, s.coarse_inv_t,
                               mixed ? s.coarse_inv32 : (float*)nullptr, mixed ? s.coarse_inv_t32 : (float*)nullptr);
    PF_LAUNCH_CHECK();
}

}  // namespace pf
