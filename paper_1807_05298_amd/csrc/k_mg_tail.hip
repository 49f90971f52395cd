// The bottom of the pressure V-cycle in one workgroup.
//
// The levels of at most about a thousand cells are bound by latency, not by
// bytes: launched one by one, every sweep, restriction and coarsest solve
// takes 2-5 us (a launch, a round trip to memory, a segment composition
// through LDS), and a sweep of several inside one launch still 4 us.  Here one
// workgroup takes them all, its memory accesses in one batch: the coefficients
// of every level go to LDS by direct loads, all in flight together, and the
// sweeps then run on LDS and registers.  A column's segments sit in
// neighbouring lanes, so that their affine maps compose by a scan over
// registers (DPP row shifts) and a half-sweep costs one workgroup barrier.
// The upward pass is summed in LDS, so the prolongation above reads one level
// instead of all.
//
// Measured per V-cycle: 17.8 us for the 616- and 84-cell levels of the
// 60x220x85 grid (five sweeps) against 31 us in 3 launches before; 13.3 us for
// the 756-, 120- and 18-cell levels of 33x26x47 against 18 us in 5; all of the
// pressure stage of a 300-cell model 12.9 us in one launch against 11.  What
// is left is a first round trip to memory (about 3 us) and the issue of the
// instructions: a phase between two barriers is 0.3-0.7 us, the first pass
// through a level's code about 1.5 us.
//
// What bounds the size of the first level is that one compute unit draws only
// about 6 bytes a cycle from beyond its L2 cache (measured: 390 KB of a
// 4,928-cell level take 25 us, longer than the launches saved), so it has to
// fit the LDS with its coefficients.
#include "pf_internal.h"

#include <algorithm>

namespace pf {
namespace {

// 256 threads: one wavefront a SIMD (more would only queue for issue slots).
constexpr int kTailThreads = 256;
constexpr int kTailLevels = 8;
constexpr int kTailCoarse = 128;     // cells of the coarsest level, at most
constexpr int kTailPad = kCoarsePad; // columns of its inverse are padded to a multiple of this
constexpr int kTailLen = 4;          // layers of a segment, at most
constexpr int kTailSeg = 4;          // log2 of the segments of a column, at most (a row of 16 lanes)

// A smoothed level: its grid, its factors to the next coarser level, the
// segments of a column (1 << lseg of len layers each), pre-smoothing sweeps
// and its LDS offsets (elements): x, the residuals of colour 0, lateral
// couplings (4 planes) and line factors (3 planes).
struct TailLevel {
    int nx, ny, nz, hx, half;
    int cx, cy, cz;
    int lseg, len, sweeps;
    int xo, ro, ao, fo;
};

template <class T> struct Tail {
    int nl;                          // smoothed levels
    int cycles;                      // V-cycles (more than one only when the first level is the finest)
    int nc, cnx, cny;                // coarsest level: cells, row and layer lengths
    int xo, bo, po, fb;              // LDS offsets: its x, b and partial sums; the first level's b
    TailLevel lv[kTailLevels];
    const T* A[kTailLevels];
    const T* aux[kTailLevels];
    const T* inv;                    // coarsest inverse, transposed, zero rows up to a multiple of kTailPad
    const T* b;                      // right-hand side of the first level (null: formed from v or cv)
    const double* v;                 // the residual whose water and oil rows sum to it, natural layout ...
    CsVec cv;                        // ... or (v null) colour-split
    T* x;                            // out: the first level's correction with the coarser ones added (p null)
    T* p;                            // out: the same in natural cell order, or (cv) on the black cells
    // cv: the wells, whose pressures follow from their rows
    int nw;
    const int32_t *wp_first, *wp_idx, *perf_cell;
    const double *Cw, *Dw, *vw;
    double* pb;
};

// Lane i takes lane i - D (UP) or i + D of its row of 16 (DPP), 0 where there
// is none.
template <int D, bool UP>
__device__ __forceinline__ int lane_shift(int v) {
    return __builtin_amdgcn_update_dpp(0, v, (UP ? 0x110 : 0x100) + D, 0xf, 0xf, true);
}
template <int D, bool UP>
__device__ __forceinline__ float lane_shift(float v) {
    return __int_as_float(lane_shift<D, UP>(__float_as_int(v)));
}
template <int D, bool UP>
__device__ __forceinline__ double lane_shift(double v) {
    return __hiloint2double(lane_shift<D, UP>(__double2hiint(v)), lane_shift<D, UP>(__double2loint(v)));
}

// Composes the affine maps y -> a y + b of a column's segments, held by seg
// neighbouring lanes (a power of two, at most 16): returns the value that the
// maps of all segments before this one (UP) or after it give from 0.
template <class T, bool UP>
__device__ __forceinline__ T segment_scan(T a, T b, int s, int seg) {
    const int r = UP ? s : seg - 1 - s;          // segments before this one
#define PF_SCAN(D)                                                               \
    if (seg > D) {                                                               \
        const T pa = lane_shift<D, UP>(a), pb = lane_shift<D, UP>(b);            \
        if (r >= D) {                                                            \
            b = a * pb + b;                                                      \
            a = a * pa;                                                          \
        }                                                                        \
    }
    PF_SCAN(1) PF_SCAN(2) PF_SCAN(4) PF_SCAN(8)
#undef PF_SCAN
    const T prev = lane_shift<1, UP>(b);
    return r > 0 ? prev : (T)0;
}

// A thread's share of a level: segment s of column (ixh, iy) of each colour,
// and where its cells and their neighbours in the other colour's half lie.
struct TailItem {
    int s, iy, ixh, k0, cols;
    int len[2];                      // layers of its segment (0: no such column)
    int i0[2];                       // slot of the first one
    int nb[2][4];                    // slot of its -x, +x, -y, +y neighbour (its own: none)
    bool on;                         // the wavefront has any such column

    __device__ __forceinline__ TailItem(const TailLevel& g, int it) {
        const int hx = g.hx;
        cols = hx * g.ny;
        on = __builtin_amdgcn_readfirstlane(it) < cols << g.lseg;
        s = it & ((1 << g.lseg) - 1);
        const int col = it >> g.lseg;
        iy = col / hx;
        ixh = col - iy * hx;
        k0 = s * g.len;
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const int ix = 2 * ixh + ((iy + c) & 1), other = (1 - 2 * c) * g.half;
            len[c] = col < cols && ix < g.nx ? max(0, min(g.len, g.nz - k0)) : 0;
            const bool in = len[c] > 0;
            const int i = i0[c] = in ? c * g.half + col + k0 * cols : 0;
            nb[c][0] = in && ix > 0 ? i + other + (((ix - 1) >> 1) - ixh) : i;
            nb[c][1] = in && ix + 1 < g.nx ? i + other + (((ix + 1) >> 1) - ixh) : i;
            nb[c][2] = in && iy > 0 ? i + other - hx : i;
            nb[c][3] = in && iy + 1 < g.ny ? i + other + hx : i;
        }
    }
    // offset of layer j of the segment from its first one (0 past its end)
    __device__ __forceinline__ int step(int c, int j) const { return j < len[c] ? j * cols : 0; }
};

// Lateral couplings and line factors of a segment (past the end of the column
// those of its first layer, unused).
template <class T, int LM> struct TailCoef {
    T a[LM][4], f[LM][3];
    __device__ __forceinline__ TailCoef(const TailItem& t, int n, const T* lat, const T* fac, int c) {
#pragma unroll
        for (int j = 0; j < LM; ++j) {
            const int i = t.i0[c] + t.step(c, j);
#pragma unroll
            for (int q = 0; q < 4; ++q) a[j][q] = lat[q * n + i];
#pragma unroll
            for (int q = 0; q < 3; ++q) f[j][q] = fac[q * n + i];
        }
    }
};

// sum of the lateral couplings times the other colour's values (x in LDS is
// cleared first, and the coupling to a missing neighbour is 0)
template <class T, int LM>
__device__ __forceinline__ void tail_lateral(const TailItem& t, const TailCoef<T, LM>& k, const T* xs, int c,
                                             T (&r)[LM]) {
#pragma unroll
    for (int j = 0; j < LM; ++j) {
        const int o = t.step(c, j);
        r[j] = k.a[j][0] * xs[t.nb[c][0] + o] + k.a[j][1] * xs[t.nb[c][1] + o] + k.a[j][2] * xs[t.nb[c][2] + o] +
               k.a[j][3] * xs[t.nb[c][3] + o];
    }
}

// One z-line half-sweep over the columns of colour c: each column's
// tridiagonal rows are solved with the right-hand side b - lt by the Thomas
// recurrences, affine in the carried value and composed over the column's
// segments.  Layers past the end of the column come last: their forward
// values are set to 0, which is what the backward recurrence starts from.
template <class T, int LM>
__device__ __forceinline__ void tail_solve(const TailLevel& g, const TailItem& t, const TailCoef<T, LM>& k,
                                           const T (&b)[LM], const T (&lt)[LM], T* xs, int c) {
    const int seg = 1 << g.lseg;
    T r[LM], fa = 1, fb = 0;
#pragma unroll
    for (int j = 0; j < LM; ++j) {
        r[j] = j < t.len[c] ? (b[j] - lt[j]) * k.f[j][1] : (T)0;
        fb = k.f[j][2] * fb + r[j];
        fa = k.f[j][2] * fa;
    }
    T y = segment_scan<T, true>(fa, fb, t.s, seg);
    T ga = 1, gb = 0;
#pragma unroll
    for (int j = 0; j < LM; ++j) {
        y = k.f[j][2] * y + r[j];
        r[j] = j < t.len[c] ? y : (T)0;
    }
#pragma unroll
    for (int j = LM - 1; j >= 0; --j) {
        gb = r[j] - k.f[j][0] * gb;
        ga = -k.f[j][0] * ga;
    }
    T xin = segment_scan<T, false>(ga, gb, t.s, seg);
#pragma unroll
    for (int j = LM - 1; j >= 0; --j) {
        xin = r[j] - k.f[j][0] * xin;
        if (j < t.len[c]) xs[t.i0[c] + j * t.cols] = xin;
    }
}

// Right-hand side of a coarse cell: the fine residuals (colour 0; the
// colour-1 ones are zero) summed over its aggregate.  Branch-free, so that the
// reads of a thread's cells issue together; a cell that is not there reads 0.
template <class T>
__device__ __forceinline__ T tail_restrict(const TailLevel& f, const T* rs, bool in, int IX, int IY, int IZ) {
    T v[4];
    bool ok[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int dz = q >> 1, dy = q & 1;
        const int iz = IZ * f.cz + dz, iy = IY * f.cy + dy, ix0 = IX * f.cx, dx = (ix0 + iy) & 1, ix = ix0 + dx;
        ok[q] = in && dz < f.cz && dy < f.cy && dx < f.cx && iz < f.nz && iy < f.ny && ix < f.nx;
        v[q] = rs[ok[q] ? (iz * f.ny + iy) * f.hx + (ix >> 1) : 0];
    }
    T s = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) s += ok[q] ? v[q] : (T)0;
    return s;
}

// The sweeps of level l (colour 0, then 1) from its right-hand side (the first
// level's in LDS, the others' restricted from the level above, in the owner
// threads' registers), and its colour-0 residuals: the colour-1 rows have just
// been solved, and the colour-0 rows were with the previous colour-1 values,
// so b - A x there is the change of their lateral terms since.  zero: x is
// taken as 0.  A barrier precedes and follows.
template <class T, int LM>
__device__ __forceinline__ void tail_level(const Tail<T>& t, int l, int tid, T* lds, bool zero) {
    const TailLevel g = t.lv[l];
    const TailItem it(g, tid);
    const int n = 2 * g.half;
    T *xs = lds + g.xo, *rs = lds + g.ro;
    T b[2][LM], l0[LM], l1[LM];
    if (l > 0) {
        const TailLevel f = t.lv[l - 1];
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int j = 0; j < LM; ++j)
                b[c][j] = tail_restrict(f, lds + f.ro, j < it.len[c], 2 * it.ixh + ((it.iy + c) & 1), it.iy,
                                        it.k0 + j);
    } else {
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
            for (int j = 0; j < LM; ++j) b[c][j] = lds[t.fb + it.i0[c] + it.step(c, j)];
    }
    const TailCoef<T, LM> k0(it, n, lds + g.ao, lds + g.fo, 0), k1(it, n, lds + g.ao, lds + g.fo, 1);
#pragma unroll
    for (int j = 0; j < LM; ++j) l0[j] = 0;
    for (int w = 0; w < g.sweeps; ++w) {
        if (it.on) {
            if (w > 0 || !zero) tail_lateral<T, LM>(it, k0, xs, 0, l0);
            tail_solve<T, LM>(g, it, k0, b[0], l0, xs, 0);
        }
        __syncthreads();
        if (it.on) {
            tail_lateral<T, LM>(it, k1, xs, 1, l1);
            tail_solve<T, LM>(g, it, k1, b[1], l1, xs, 1);
        }
        __syncthreads();
    }
    if (it.on) {
        tail_lateral<T, LM>(it, k0, xs, 0, l1);
#pragma unroll
        for (int j = 0; j < LM; ++j)
            if (j < it.len[0]) rs[it.i0[0] + j * it.cols] = l0[j] - l1[j];
    }
    __syncthreads();
}

// x_l += P x_{l+1}; out: also the result.  A barrier precedes and follows.
template <class T, int LM>
__device__ __forceinline__ void tail_upward(const Tail<T>& t, int l, int tid, T* lds, bool out) {
    const TailLevel g = t.lv[l];
    const TailItem it(g, tid);
    const bool dense = l + 1 == t.nl;
    const TailLevel c = t.lv[dense ? l : l + 1];
    // the next level: colour-split (a half per colour, lines of hx), or the coarsest in natural order
    const int xo = dense ? t.xo : c.xo, line = dense ? t.cnx : c.hx, layer = line * (dense ? t.cny : c.ny);
    const int half = dense ? 0 : c.half, sh = dense ? 0 : 1;
    if (it.on) {
        T val[2][LM];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int ix = 2 * it.ixh + ((it.iy + q) & 1);
            const int X = g.cx == 2 ? ix >> 1 : ix, Y = g.cy == 2 ? it.iy >> 1 : it.iy;
            const int base = xo + ((X + Y) & 1) * half + Y * line + (X >> sh);
#pragma unroll
            for (int j = 0; j < LM; ++j) {
                const int iz = it.k0 + j, Z = g.cz == 2 ? iz >> 1 : iz;
                val[q][j] = lds[g.xo + it.i0[q] + it.step(q, j)] + lds[j < it.len[q] ? base + Z * layer : xo];
            }
        }
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int ix = 2 * it.ixh + ((it.iy + q) & 1);
#pragma unroll
            for (int j = 0; j < LM; ++j)
                if (j < it.len[q]) {
                    const int i = it.i0[q] + j * it.cols, iz = it.k0 + j;
                    if (!out || t.cv.b) lds[g.xo + i] = val[q][j];
                    if (out && !t.p) t.x[i] = val[q][j];
                    else if (out && !t.cv.b) t.p[ix + g.nx * (it.iy + g.ny * iz)] = val[q][j];
                    else if (out && ((q + iz) & 1)) t.p[i - q * g.half] = val[q][j];      // a black cell's slot
                }
        }
    }
    __syncthreads();
}

// Copies count elements to LDS without passing through registers: 16 bytes a
// lane (FP64: planes of an even number of elements, 16-byte aligned) or 4.
// The caller waits (s_waitcnt) before the barrier after which they are read.
template <class T>
__device__ __forceinline__ void tail_stage(const T* src, T* dst, int count, int tid) {
    using Src = const __attribute__((address_space(1))) void*;
    using Dst = __attribute__((address_space(3))) void*;
    constexpr int E = sizeof(T) == 8 ? 2 : 1;        // elements a lane
    const int lane = tid & 63;
    for (int i = __builtin_amdgcn_readfirstlane(tid) * E; i < count; i += kTailThreads * E)
        if (i + lane * E < count) {
            if constexpr (sizeof(T) == 8)
                __builtin_amdgcn_global_load_lds((Src)(src + i + lane * E), (Dst)(dst + i), 16, 0, 0);
            else
                __builtin_amdgcn_global_load_lds((Src)(src + i + lane * E), (Dst)(dst + i), 4, 0, 0);
        }
}

template <class T>
__device__ __forceinline__ void k_mg_tail_d(const Blk&, const Tail<T>& t) {
    extern __shared__ double tail_sm[];
    T* lds = reinterpret_cast<T*>(tail_sm);
    const int tid = (int)threadIdx.x;
    const TailLevel& g0 = t.lv[0];
    {
        // touch every line of the arguments at once: read one by one where they
        // are needed, each would be a round trip
        const int* w = reinterpret_cast<const int*>(&t);
        constexpr int kLines = (int)sizeof(Tail<T>) / 64;
        int sum = 0;
#pragma unroll
        for (int q = 0; q < kLines; ++q) sum += w[16 * q];
        asm volatile("" ::"s"(sum));
    }
    for (int l = 0; l < t.nl; ++l) {
        const TailLevel& g = t.lv[l];
        const int n = 2 * g.half;
        tail_stage<T>(t.A[l] + n, lds + g.ao, 4 * n, tid);
        tail_stage<T>(t.aux[l], lds + g.fo, 3 * n, tid);
    }
    for (int l = 0; l < t.nl; ++l) {
        const TailLevel& g = t.lv[l];
        for (int i = tid; i < 2 * g.half; i += kTailThreads) lds[g.xo + i] = 0;
    }
    // right-hand side of the first level
    if (t.b) {
        tail_stage<T>(t.b, lds + t.fb, 2 * g0.half, tid);
    } else {
        // it is the finest: b = water + oil rows of v
        const int layer = g0.nx * g0.ny, cells = layer * g0.nz, ns = g0.half;
        const double al = t.v ? 0.0 : *t.cv.alpha;
        for (int i = tid; i < cells; i += kTailThreads) {
            const int iz = i / layer, rem = i - iz * layer, iy = rem / g0.nx, ix = rem - iy * g0.nx;
            const int sl = (iz * g0.ny + iy) * g0.hx + (ix >> 1);
            double r;
            if (t.v) r = t.v[i] + t.v[cells + i];
            else if ((ix + iy + iz) & 1) r = t.cv.b[sl] + t.cv.b[ns + sl];
            else r = al * (t.cv.u[sl] + t.cv.u[ns + sl]);
            lds[t.fb + ((ix + iy) & 1) * g0.half + sl] = (T)r;
        }
    }
    // thread (q, r) takes its share of row r of the dense coarsest inverse
    const int nc = t.nc, r = tid & (kTailCoarse - 1), q = tid / kTailCoarse;
    constexpr int kQ = kTailThreads / kTailCoarse, kC = kTailCoarse / kQ, kG = kTailPad / kQ;
    T iv[kC];
#pragma unroll
    for (int e = 0; e < kC; ++e) iv[e] = 0;
    if (r < nc) {
        const T* inv = t.inv + (q * nc + r);
#pragma unroll
        for (int e = 0; e < kC; ++e)
            if (kQ * (e - e % kG) < nc) iv[e] = inv[kQ * e * nc];       // zero-padded to whole groups
    }
    __builtin_amdgcn_s_waitcnt(0);       // the staged coefficients
    __syncthreads();
    for (int cyc = 0; cyc < t.cycles; ++cyc) {
#pragma unroll 1
        for (int l = 0; l < t.nl; ++l) {
            const bool zero = l > 0 || cyc == 0;
            switch (t.lv[l].len) {
                case 1: tail_level<T, 1>(t, l, tid, lds, zero); break;
                case 2: tail_level<T, 2>(t, l, tid, lds, zero); break;
                case 3: tail_level<T, 3>(t, l, tid, lds, zero); break;
                default: tail_level<T, 4>(t, l, tid, lds, zero); break;
            }
        }
        if (tid < kTailCoarse) {
            const TailLevel f = t.lv[t.nl - 1];
            const int IZ = tid / (t.cnx * t.cny), rem = tid - IZ * t.cnx * t.cny, IY = rem / t.cnx;
            lds[t.bo + tid] = tail_restrict(f, lds + f.ro, tid < nc, rem - IY * t.cnx, IY, IZ);
        }
        __syncthreads();
        T sum = 0;
#pragma unroll
        for (int e = 0; e < kC; e += kG)
            if (kQ * e < nc) {
#pragma unroll
                for (int k = 0; k < kG; ++k) sum += iv[e + k] * lds[t.bo + q + kQ * (e + k)];
            }
        lds[t.po + q * kTailCoarse + r] = sum;
        __syncthreads();
        if (tid < nc) {
            T s = lds[t.po + tid];
#pragma unroll
            for (int e = 1; e < kQ; ++e) s += lds[t.po + e * kTailCoarse + tid];
            lds[t.xo + tid] = s;
        }
        __syncthreads();
        // upward, from the coarsest level
#pragma unroll 1
        for (int l = t.nl - 1; l >= 0; --l) {
            const bool out = l == 0 && cyc + 1 == t.cycles;
            if (t.lv[l].len <= 2) tail_upward<T, 2>(t, l, tid, lds, out);
            else tail_upward<T, kTailLen>(t, l, tid, lds, out);
        }
    }
    if (t.p && t.cv.b) {
        // pb_w = (v_w - sum_perf dW/dP * p_cell) / D_w, a wavefront per well
        for (int w = tid >> 6; w < t.nw; w += kTailThreads / 64) {
            double s = 0.0;
            for (int k = t.wp_first[w] + (tid & 63); k < t.wp_first[w + 1]; k += 64) {
                const int f = t.wp_idx[k], c = t.perf_cell[f], row = c / g0.nx, ix = c - row * g0.nx;
                const int iy = row % g0.ny;
                s += t.Cw[3 * f] * (double)lds[g0.xo + ((ix + iy) & 1) * g0.half + row * g0.hx + (ix >> 1)];
            }
            for (int o = 32; o > 0; o >>= 1) s += __shfl_down(s, o, 64);
            if ((tid & 63) == 0) t.pb[w] = (t.vw[w] - s) / t.Dw[w];
        }
    }
}
template <class T>
__global__ __launch_bounds__(kTailThreads) void k_mg_tail(Tail<T> t) {
    k_mg_tail_d<T>(PF_BLK, t);
}
template <class T>
struct F_k_mg_tail {
    static constexpr int kLB = kTailThreads;
    template <class... A>
    __device__ __forceinline__ void operator()(const Blk& wg, const A&... a) const {
        k_mg_tail_d<T>(wg, a...);
    }
};

template <class T> const T* lvA(const MGLevel& L);
template <> const double* lvA(const MGLevel& L) { return L.A; }
template <> const float* lvA(const MGLevel& L) { return L.A32; }
template <class T> const T* lvAux(const MGLevel& L);
template <> const double* lvAux(const MGLevel& L) { return L.aux; }
template <> const float* lvAux(const MGLevel& L) { return L.aux32; }
template <class T> T* lvX(const MGLevel& L);
template <> double* lvX(const MGLevel& L) { return L.x; }
template <> float* lvX(const MGLevel& L) { return L.x32; }
template <class T> T* lvB(const MGLevel& L);
template <> double* lvB(const MGLevel& L) { return L.b; }
template <> float* lvB(const MGLevel& L) { return L.b32; }
template <class T> const T* coarseInv(const Sim& s);
template <> const double* coarseInv(const Sim& s) { return s.coarse_inv_t; }
template <> const float* coarseInv(const Sim& s) { return s.coarse_inv_t32; }

// Segments of a column of a tail level: a power of two, as many as give every
// segment of a colour a thread (and at most one for each layer).  False where
// they do not fit the threads or the rows of lanes.
bool tail_segments(const MGLevel& L, int& lseg, int& len) {
    const int64_t cols = (int64_t)((L.nx + 1) / 2) * L.ny;
    lseg = 0;
    while (lseg < kTailSeg && (1 << lseg) < L.nz && (cols << (lseg + 1)) <= kTailThreads) ++lseg;
    len = (L.nz + (1 << lseg) - 1) >> lseg;
    return len <= kTailLen && cols <= kTailThreads;
}

// The shape of a tail from level l0 and its LDS offsets (elements); its LDS
// bytes, or 0 where a level does not fit.
template <class T>
size_t tail_plan(const Sim& s, int l0, Tail<T>& t) {
    const int nl = (int)s.mg.size();
    size_t off = 0;
    auto take = [&](int64_t n) {
        const size_t o = off;
        off += (size_t)((n + 3) & ~(int64_t)3);
        return (int)o;
    };
    t.nl = nl - 1 - l0;
    for (int l = l0; l + 1 < nl; ++l) {
        const MGLevel& L = s.mg[l];
        TailLevel& g = t.lv[l - l0];
        if (!tail_segments(L, g.lseg, g.len)) return 0;
        g.nx = L.nx; g.ny = L.ny; g.nz = L.nz;
        g.hx = (L.nx + 1) / 2;
        g.half = g.hx * L.ny * L.nz;
        g.cx = L.cx; g.cy = L.cy; g.cz = L.cz;
        g.sweeps = mg_pre_sweeps(s, l);
        g.xo = take(L.ns);
        g.ro = take(L.ns / 2);
        g.ao = take(4 * L.ns);
        g.fo = take(3 * L.ns);
    }
    const MGLevel& C = s.mg.back();
    t.nc = (int)C.n; t.cnx = C.nx; t.cny = C.ny;
    t.xo = take(kTailCoarse);
    t.bo = take(kTailCoarse);
    t.po = take(kTailThreads);
    t.fb = take(s.mg[l0].ns);
    return off * sizeof(T);
}

// The first level the launch takes: the finest that fits.  (Its segments are
// its own, so a caller who sets their length gets launches of their own.)
template <class T>
int tail_first(const Sim& s) {
    const int nl = (int)s.mg.size();
    if (nl < 2 || s.opts.mg_post > 0 || s.opts.zline_len > 0 || s.mg.back().n > kTailCoarse) return nl;
    Tail<T> t{};
    for (int l = std::max(0, nl - 1 - kTailLevels); l + 1 < nl; ++l) {
        if (s.mg[l].n > 2 * kTailLen * kTailThreads) continue;
        const size_t shm = tail_plan<T>(s, l, t);
        if (shm > 0 && shm <= (size_t)s.max_lds) return l;
    }
    return nl;
}

template <class T>
void tail_launch(Sim& s, int l0, int cycles, const double* v, const CsVec* cv, T* p) {
    Tail<T> t{};
    const size_t shm = tail_plan<T>(s, l0, t);
    for (int l = 0; l < t.nl; ++l) {
        t.A[l] = lvA<T>(s.mg[l0 + l]);
        t.aux[l] = lvAux<T>(s.mg[l0 + l]);
    }
    t.cycles = cycles;
    t.inv = coarseInv<T>(s);
    t.b = v || cv ? nullptr : lvB<T>(s.mg[l0]);
    t.v = v;
    if (cv) {
        t.cv = *cv;
        t.nw = s.m.nw;
        t.wp_first = s.wp_first; t.wp_idx = s.wp_idx; t.perf_cell = s.perf_cell;
        t.Cw = s.Cw; t.Dw = s.Dw;
        t.vw = cv->b + 3 * cs_ns(s.m);
        t.pb = s.pb;
    }
    t.x = lvX<T>(s.mg[l0]);
    t.p = p;
    launch<F_k_mg_tail<T>>(s, s.stream, k_mg_tail<T>, dim3(1), dim3(kTailThreads), shm, t);
    PF_LAUNCH_CHECK();
}

}  // namespace

int mg_tail_first(const Sim& s) {
    return s.opts.precision == PF_PREC_MIXED ? tail_first<float>(s) : tail_first<double>(s);
}

void launch_mg_tail(Sim& s, int l0, int cycles, const double* v, const CsVec* cv, double* p) {
    tail_launch<double>(s, l0, cycles, v, cv, p);
}
void launch_mg_tail(Sim& s, int l0, int cycles, const double* v, const CsVec* cv, float* p) {
    tail_launch<float>(s, l0, cycles, v, cv, p);
}

}  // namespace pf
