// Internal declarations of the polyflood HIP library (gfx950).
//
// Device data layout (all in the caller's workspace, 256-byte aligned):
//   state vectors   x, xn: 3N + nw doubles: planes P[N], S[N], C[N], then Pb[nw]
//   accumulation    Mn: 3N (water, oil, polymer planes)
//   residual        R: 3N + nw (row-scaled, see polyflood.h)
//   Jacobian        J: 63 planes of N: J[(d*9 + e)*N + i], d = 0 own block,
//                   1..6 = -x,+x,-y,+y,-z,+z neighbour blocks, e = 3*row + col
//   well border     B[3*np] (dR~_cell/dPb), Cw[3*np] (dW~/dx_cell), Dw[nw]
//   static          PVr[N], Tx/Ty/Tz[N] (to the + neighbour, 0 on the boundary)
#pragma once

#include <hip/hip_runtime.h>
#include <cstdint>
#include <cstddef>
#include <functional>
#include <string>
#include <vector>

#include "../../include/polyflood.h"

namespace pf {

constexpr double kBar = 1.0e5;
constexpr int kBlock = 256;          // threads per block for cell sweeps
constexpr int kMaxRestart = 64;
constexpr int kRedBlocks = 1024;     // largest partial-sum grid of the reductions
constexpr int kDotChunk = 16;        // dot products per multi-dot launch
constexpr int kPostFlag = 32;        // place of the flag in the read-back buffer
constexpr int kCoarseReg = 96;       // largest coarsest level inverted in registers (k_coarse)
constexpr int kCoarsePad = 16;       // rows of the transposed coarsest inverse: padded with zeros to a multiple
constexpr int kPartSlots = kMaxRestart + 2;   // partial-sum slots: restart + 2 dot products

// Everything a kernel needs to evaluate cell properties; passed by value.
struct DevModel {
    int32_t nx, ny, nz, nw;
    int64_t n, nxy;
    int64_t np;                      // perforations
    int64_t npc;                     // perforated cells
    double dx, dy, dz, top, vol;
    double cr, pref;
    double rho_w0, rho_o0, c_w, c_o, mu_w, mu_o, swc, sor, n_w, n_o, krw0, kro0, grav;
    double a1, a2, omega, cmax, mup_ref, ads_max, ads_b, rrf, ipv;
    double inv_den;                  // 1/(1 - swc - sor)
    double tl_pref;                  // mu_p^ref^(1-omega)  (Todd-Longstaff)
    double tl_pw;                    // mu_w^(1-omega)
    double c_ref;                    // polymer row scale concentration
    double inv_mu_o, inv_rho_w0, inv_vol, rk_slope;   // 1/mu_o, 1/rho_w0, 1/V, (RRF - 1)/A_max
    double inv_rho_o0, inv_c_ref;    // 1/rho_o0, 1/C_ref (row scales)
    int32_t corey2_w, corey2_o, omega1, pad;
    // property variants: mixing rule, tables (adsorption, viscosity multiplier, capillary pressure)
    int32_t mix_rule, n_ads, n_visc, n_pc;
    double mix_ln;                   // ln(mu_p^ref / mu_w) (PF_MIX_EXP)
    // device copy of the tables, kTabSlots x PF_TABLE_MAX doubles:
    // ads_c, ads_a, visc_c, visc_m, pc_s, pc_v, log10 of kperm_k, kperm_rrf, kperm_admax
    const double* tab;
    // retention and the rock table (null when not used): per cell the rock's
    // capacity A_d,max / ads_max, its (RRF - 1) / A_d,max, and the largest
    // past equilibrium adsorption
    int32_t n_kperm, pad2;
    double ads_res;
    const double* cell_cap;
    const double* cell_rks;
    const double* ads_hist;
};
enum { kTabAdsC = 0, kTabAdsA = 1, kTabViscC = 2, kTabViscM = 3, kTabPcS = 4, kTabPcV = 5, kTabKpK = 6,
       kTabKpRrf = 7, kTabKpAdm = 8, kTabSlots = 9 };


// ---- kernel launches: direct, or recorded for a fusion group --------------
// Every kernel is a __device__ body that takes the block index of its launch
// (Blk), with a __global__ wrapper for a direct launch and a functor
// F_<kernel> through which k_multi runs the same body for each simulator's
// share of a merged launch.  A simulator in a fusion group (pf_fusion_*)
// records its launches instead of issuing them; when every member has
// reached a synchronisation point the group issues the recorded work, one
// launch for the ops of the same kernel at the heads of the members' queues.
struct Blk {
    uint32_t x, n;                   // block index within this simulator's launch, its block count
};
#define PF_BLK (::pf::Blk{blockIdx.x, gridDim.x})

// Kernel arguments as a flat aggregate (host and device see one layout).
template <class... T> struct Pack {};
template <class H, class... T> struct Pack<H, T...> {
    H h;
    Pack<T...> t;
};
template <class... T> struct PackOf;
template <> struct PackOf<> {
    static Pack<> make() { return Pack<>{}; }
};
template <class H, class... T> struct PackOf<H, T...> {
    static Pack<H, T...> make(const H& h, const T&... t) { return Pack<H, T...>{h, PackOf<T...>::make(t...)}; }
};
template <class F, class... D>
__device__ __forceinline__ void pack_apply(const F& f, const Blk& wg, const Pack<>&, const D&... d) {
    f(wg, d...);
}
template <class F, class H, class... T, class... D>
__device__ __forceinline__ void pack_apply(const F& f, const Blk& wg, const Pack<H, T...>& p, const D&... d) {
    pack_apply(f, wg, p.t, d..., p.h);
}

// One simulator's share of a merged launch: nb blocks, from a first block
// that is a multiple of 8 (so that every block runs on the XCD it would run
// on alone), and the kernel's arguments.
template <class... P> struct MEntry {
    uint32_t nb, pad;
    Pack<P...> a;
};

// The table of a merged launch: the first blocks of its ns entries as one
// compact array (the block's search touches one or two cache lines), then
// the entries from byte multi_entries(ns).
__host__ __device__ inline size_t multi_entries(int ns) { return ((size_t)ns * 4 + 15) & ~(size_t)15; }

template <class F, class... P>
__global__ __launch_bounds__(F::kLB) void k_multi(const uint8_t* __restrict__ tab, int ns) {
    const uint32_t* __restrict__ b0 = reinterpret_cast<const uint32_t*>(tab);
    const MEntry<P...>* __restrict__ e = reinterpret_cast<const MEntry<P...>*>(tab + multi_entries(ns));
    const uint32_t b = blockIdx.x;
    int lo = 0, hi = ns - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (b0[mid] <= b) lo = mid;
        else hi = mid - 1;
    }
    const uint32_t lb = b - b0[lo];
    if (lb >= e[lo].nb) return;          // padding up to the next simulator's range
    pack_apply(F{}, Blk{lb, e[lo].nb}, e[lo].a);
}

using MultiFn = void (*)(const void* table, int n, unsigned blocks, unsigned threads, size_t shm, hipStream_t st);

template <class F, class... P>
void run_multi(const void* table, int n, unsigned blocks, unsigned threads, size_t shm, hipStream_t st) {
    hipLaunchKernelGGL((k_multi<F, P...>), dim3(blocks), dim3(threads), shm, st, static_cast<const uint8_t*>(table),
                       n);
}

// A recorded stream operation of a fusion-group member.
struct Op {
    MultiFn multi = nullptr;         // merged kernel launch, or null: a host-issued operation
    uint32_t nb = 0, threads = 0;    // this simulator's blocks, threads per block
    size_t shm = 0;                  // dynamic LDS bytes
    size_t off = 0, len = 0;         // its MEntry in the member's byte buffer
    std::function<void(hipStream_t)> host;
};

struct Fusion;                       // pf_fuse.hip

// Small device-side control block of FGMRES (Hessenberg, Givens, norms).
struct KrylovCtl {
    double H[(kMaxRestart + 1) * kMaxRestart];   // column-major, ld = kMaxRestart+1
    double cs[kMaxRestart], sn[kMaxRestart];
    double g[kMaxRestart + 1];
    double y[kMaxRestart];
    double h[kMaxRestart + 2];       // scratch column of dot products
    // colour-split solves: the red part of every Krylov vector is a multiple of
    // the cycle's residual's, V[k]_r = alpha[k] u, and gram = <u, u> (0 otherwise)
    double alpha[kMaxRestart + 2];
    double gram;
    double beta0;                    // initial residual norm of this solve
    double beta;                     // residual norm at the start of this cycle
    double wnorm0;                   // |w| before orthogonalisation
    double wnorm;                    // |w| after
    double inv_h;                    // 1 / h(j+1, j)
    double rel;                      // |g(j+1)| / beta0
    int32_t reorth;                  // second CGS pass requested
    int32_t breakdown;
    int32_t normalised;              // w was scaled to unit norm by the update itself
    int32_t pad;
};

// Grid dimensions of a multigrid level; split: colour-split slot order.
struct Dims { int nx, ny, nz, split; };

struct MGLevel {
    int32_t nx, ny, nz;
    int32_t split;                   // colour-split storage (every level but the coarsest)
    int64_t ns;                      // slots per plane (>= n)
    int32_t cx, cy, cz;              // aggregation factors to the next coarser level
    int64_t n;
    double* A;                       // 7 planes: diag, -x, +x, -y, +y, -z, +z
    double* aux;                     // smoother set-up data (inverse diagonal / line factors)
    double* x;
    double* b;
    double* r;
    float* A32;                      // mixed precision copies
    float* aux32;
    float* x32;
    float* b32;
    float* r32;
};

// Values for the host that a kernel writes itself, as its last act: to the
// pinned read-back buffer, then seq to its flag, for which the host polls
// (wait_post).  out null: nothing (a read-back buffer that is not pinned is
// filled by a copy).
struct HostPost {
    double* out;
    unsigned long long *flag, seq;
};
// by one thread, whose own stores the release orders
__device__ __forceinline__ void post_done(const HostPost& p) {
    __hip_atomic_store(p.flag, p.seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

struct Sim {
    DevModel m;
    pf_solver_opts opts;
    hipStream_t stream;
    hipStream_t aux = nullptr;       // side stream: the coarsest inverse overlaps the ILU set-up
    hipEvent_t ev_fork = nullptr, ev_join = nullptr;
    char* ws;
    size_t ws_bytes;
    int64_t nv;                      // 3N + nw

    // static
    double *poro, *kx, *ky, *kz;
    double *pvr, *Tx, *Ty, *Tz, *rscale;
    int32_t *perf_cell, *perf_well, *pc_cell, *pc_first, *wp_first, *wp_idx;
    int32_t *pc_map;                 // cell -> index into pc_cell, or -1
    int32_t *pc_map_cs;              // the same in the colour-split layout (FP64 red-black ILU(0))
    double *perf_wi, *perf_depth;
    int32_t *w_ctrl, *w_inj, *w_dir;
    double *w_target, *w_cinj, *w_gamma, *w_zref, *w_scale, *w_rw, *w_skin;

    // state / system
    double *x, *xn, *Mn, *R, *J, *B, *Cw, *Dw, *wv, *wdp;
    double *perf_q;                  // surface water and oil rate of each perforation (2 per perforation)
    double *cell_cap, *cell_rks;     // rock table per cell (n_kperm > 0)
    double *ads_hist;                // largest past equilibrium adsorption (ads_res > 0)
    double *tab;                     // property tables (kTabSlots x PF_TABLE_MAX)
    double *dx;                      // Newton update
    double *rhs;                     // linear right-hand side

    // solver
    double *V, *Z, *w, *t1, *t2;
    // Krylov vectors: length nx (nv, or nvc in the colour-split layout) and the
    // stride kst of the columns of V and Z (max(nv, nvc)); the Arnoldi process
    // works on nk entries of a column of V from entry ko (all of them, or the
    // black cells and wells)
    int64_t nx = 0, nk = 0, ko = 0, kst = 0, nvc = 0;
    double *bcs = nullptr, *xcs = nullptr;   // right-hand side and solution in the colour-split layout
    KrylovCtl* kc;
    double *part;                    // reduction partials
    double *red;                     // reduction results (64 doubles)
    double *Dinv;                    // block Jacobi: 9N natural; ILU(0): 2 x 9 colour-split planes
    double *Ap;                      // pressure operator (7N) = level 0 of MG
    double *coarse_aug;              // coarsest-level [A | I] -> [I | A^-1] (above kCoarseReg cells)
    double *coarse_inv;              // compact coarsest inverse (n x n)
    float *coarse_inv32;
    double *coarse_inv_t;            // ... and transposed
    float *coarse_inv_t32;
    float *Jp32;                     // mixed: FP32 P-columns of J (21 planes)
    double *Lc = nullptr;            // FP64 ILU: colour-split off-diagonal blocks (lc_at)
    double *Jdc;                     // FP64 ILU: colour-split diagonal blocks of J (2 x 9 planes)
    uint16_t *Joff16 = nullptr;      // mixed ILU: colour-split BF16 off-diagonal blocks (2 x 54 planes)
    float *Dinv32;                   // mixed: FP32 smoother inverse diagonals
    float *t32;                      // mixed: FP32 stage residual
    float *Z32;                      // mixed: FP32 preconditioned Krylov vectors
    double *pb;                      // well bottom-hole pressures of the pressure stage
    double *pnat;                    // pressure-stage correction in natural cell order
    float *pnat32;                   // the same, mixed precision
    std::vector<MGLevel> mg;
    int restart_cap;
    int max_lds = 65536;             // bytes of LDS a workgroup may allocate

    // host
    double* hbuf;                    // read-back buffer (64 doubles): pinned, or static (static_dev >= 0)
    unsigned long long post_seq = 0; // last post's number; its flag is hbuf[kPostFlag]
    int static_dev = -1;             // device whose static workspace this simulator holds (-1: caller's)
    int device = 0;                  // device current at creation (its workspace and stream)
    bool coarse_pending = false;     // the coarsest inverse may still run on the side stream
    bool j_cs = false;               // the last Jacobian is in the colour-split copies (Jdc, Lc) only
    bool j_nat = true;               // the natural-order planes of J hold the last Jacobian
    int newton_it;                   // Newton iterations in the current step
    double dt_next = 0.0;            // next sub-step length (0: the scheduled step)
    double last_upd;
    double last_bnorm;               // ||R~||_2 of the previous Newton iteration
    int prec_ready;
    std::vector<int32_t> h_perf_cell, h_perf_well, h_w_ctrl;
    // well controls: as given in the model (primary) and active (after BHP-limit switches)
    std::vector<int32_t> h_ctrl0, h_inj, h_wp_first;
    std::vector<double> h_target0, h_limit, h_target;
    std::vector<double> h_perf_wi;
    std::vector<int32_t> h_wktop;    // datum (top perforated) layer of every well

    // fusion group membership (pf_fusion_join): recorded operations
    Fusion* fu = nullptr;
    std::vector<Op> ops;
    std::vector<uint8_t> op_bytes;

    // kernel timing (pf_profile_begin/end)
    int prof_id = 0;
    int prof_used = 0;
    std::vector<hipEvent_t> prof_ev;     // start/stop pairs
};

// Brackets one launch with events when the simulator times this kernel.
struct ProfScope {
    Sim& s;
    bool on;
    ProfScope(Sim& sim, int id)
        : s(sim), on(!sim.fu && sim.prof_id == id && 2 * (sim.prof_used + 1) <= (int)sim.prof_ev.size()) {
        if (on) (void)hipEventRecord(s.prof_ev[2 * s.prof_used], s.stream);
    }
    ~ProfScope() {
        if (on) {
            (void)hipEventRecord(s.prof_ev[2 * s.prof_used + 1], s.stream);
            ++s.prof_used;
        }
    }
};

// Bump allocator over the workspace; with base == nullptr it only measures.
struct Bump {
    char* base;
    size_t used = 0;
    template <class T>
    T* take(size_t count) {
        used = (used + 255) & ~size_t(255);
        T* p = base ? reinterpret_cast<T*>(base + used) : nullptr;
        used += (count > 0 ? count : 1) * sizeof(T);
        return p;
    }
};

// ---- kernels launchers (k_physics.hip) ----------------------------------
void launch_static(Sim& s);
void launch_accum(Sim& s, const double* x, double* M);
void launch_assemble(Sim& s, double dt, bool with_jacobian);
void launch_norms(Sim& s, const double* v, double* out, const HostPost& post);   // out[0..5]
void launch_update(Sim& s, const double* dx, double* out, bool cs, const HostPost& post);   // out[0..4]; cs: dx colour-split
void launch_kperm(Sim& s);                                          // per-cell RRF, A_d,max
void launch_ads_hist(Sim& s);                                       // take in the current state
void launch_equilibrium(Sim& s, double datum_depth, double datum_p, double fwl_depth);

// Blocks of a reduction over n entries: one entry a thread up to kRedBlocks
// blocks, a grid-stride loop beyond.  (Entries fall to the same partial sums
// as with the full grid, whose other blocks would only add zeros: for eight
// members of 26 to 44 thousand cells at once the products of a column took
// 22.7 us with it and take 10.7, the update 12.3 and 7.0.)
inline int red_grid(int64_t n) {
    const int64_t g = (n + kBlock - 1) / kBlock;
    return (int)(g < 1 ? 1 : g > kRedBlocks ? kRedBlocks : g);
}

// ---- linear algebra (k_linalg.hip) ----------------------------------------
void launch_spmv(Sim& s, const double* x, double* y);
void launch_spmv(Sim& s, const float* x, double* y);
void launch_residual(Sim& s, const double* v, const double* x, double* t);        // t = v - J x
void launch_residual(Sim& s, const double* v, const float* x, double* t);
void launch_pc_map_cs(Sim& s);        // pc_map_cs from pc_map
void launch_to_cs(Sim& s, const double* x, double* y, double scale = 1.0);   // natural -> colour-split, times scale
void launch_from_cs(Sim& s, const double* x, double* y);          // colour-split -> natural layout
void launch_axpby(Sim& s, int64_t n, double a, const double* x, double b, double* y);
void launch_copy(Sim& s, int64_t n, const double* x, double* y);
void launch_fill(Sim& s, int64_t n, double v, double* y);
// J in the colour-split layout only (FP64 red-black ILU(0), PF order), and
// the natural-order planes formed from it when a kernel needs them
bool j_colour_split_mode(const Sim& s);
void ensure_j_natural(Sim& s);
void launch_bjac_setup(Sim& s);
// Krylov helpers
void launch_norm_to_ctl(Sim& s, const double* v, int which, const HostPost& post);   // which 0: beta0+beta, 1: beta
void launch_scale_by_ctl(Sim& s, const double* v, double* out, int which);  // which 0: 1/beta, 1: inv_h
// first CGS pass of w against V[0..j], and the second pass (when requested);
// posts rel, then (int32) reorth, breakdown, normalised of the control block
void launch_arnoldi(Sim& s, int j, double* w, const HostPost& post);
void launch_arnoldi_second(Sim& s, int j, double* w, const HostPost& post);
void launch_normalise(Sim& s, int j, double* w);                   // V[j+1] = w / h(j+1, j)
void launch_solve_small(Sim& s, int k);                             // y = H(0:k,0:k)^{-1} g
void launch_zcomb(Sim& s, int k, double* dx, bool first = false);   // dx += Z y (first: dx = Z y)

// ---- CPR (k_cpr.hip) ---------------------------------------------------------
void cpr_choose_levels(Sim& s);     // host: multigrid hierarchy shape
void cpr_plan(Sim& s, Bump& b);      // workspace of the preconditioner
void cpr_setup(Sim& s);
void cpr_apply(Sim& s, const double* v, double* z);
void cpr_apply(Sim& s, const double* v, float* z);      // mixed precision
// A vector of the colour-split layout (black cells and wells at b, red cells
// alpha times u), and z = M^{-1} v with the black rows and wells of w = J z (wb)
struct CsVec {
    const double *u, *b, *alpha;
};
void cpr_apply_spmv(Sim& s, const CsVec& v, double* z, double* wb);
void cpr_apply_spmv(Sim& s, const double* v, double* z, double* w);   // natural layout: z = M^{-1} v, w = J z
bool cpr_colour_split(const Sim& s);  // the FP64 solve runs in the colour-split layout
void mg_smooth_once(Sim& s, int level, int colour, int zero_init);   // test hook
int64_t mg_slot(const MGLevel& L, int ix, int iy, int iz);             // cell -> slot of a level
int mg_pre_sweeps(const Sim& s, int level);                            // pre-smoothing sweeps of a level
// test hook: what takes a level on the way down of a pressure stage's cycle
// (PF_MG_*), k_mg_down's tile, and whether the next level's first half-sweep goes with it
struct MgRoute {
    int32_t kind, tx, ty, next;
};
MgRoute mg_route(const Sim& s, int level, int cycle);
void mg_cycles_once(Sim& s, const double* v);   // test hook: s.pnat(32) = V-cycles(Pi_r v)
void smoother_once(Sim& s, const double* f);    // test hook: s.t1 (FP64) / s.Z32 (mixed) = S f

// ---- the bottom of the V-cycle in one workgroup (k_mg_tail.hip) ------------
// First level that its launch takes (the number of levels: none)
int mg_tail_first(const Sim& s);
// cycles V-cycles from that level l0 down; l0 > 0: from the level's right-hand
// side to its correction with the coarser ones added; l0 == 0: from v (natural
// layout) or cv (colour-split) to p, in natural cell order or the black cells
// alone with the well pressures
void launch_mg_tail(Sim& s, int l0, int cycles, const double* v, const CsVec* cv, double* p);
void launch_mg_tail(Sim& s, int l0, int cycles, const double* v, const CsVec* cv, float* p);

// the coarsest level's dense inverse on stream st (k_coarse.hip; at most kCoarseReg cells)
void launch_coarse_inverse(Sim& s, hipStream_t st);

// ---- errors -----------------------------------------------------------------
void set_error(const std::string& msg);
struct HipError { std::string msg; };
#define PF_HIP(call)                                                              \
    do {                                                                          \
        hipError_t e_ = (call);                                                   \
        if (e_ != hipSuccess)                                                     \
            throw ::pf::HipError{std::string(#call) + ": " + hipGetErrorString(e_)}; \
    } while (0)
#define PF_LAUNCH_CHECK() PF_HIP(hipGetLastError())

// ---- fusion group hooks (pf_fuse.hip) -----------------------------------------
void fusion_record(Sim& s, MultiFn f, uint32_t nb, uint32_t threads, size_t shm, const void* entry, size_t len);
void fusion_host(Sim& s, std::function<void(hipStream_t)> op);
int64_t fusion_cells(const Sim& s);  // cells of the group's members together (its own without a group)
void fusion_sync(Sim& s);            // every member at a synchronisation point: the group's work is issued

// Launch of kernel k (functor F) on stream st, or its record in s's fusion group.
template <class F, class... P, class... A>
void launch(Sim& s, hipStream_t st, void (*k)(P...), dim3 grid, dim3 block, size_t shm, const A&... a) {
    static_assert(sizeof...(P) == sizeof...(A), "argument count");
    if (!s.fu) {
        hipLaunchKernelGGL(k, grid, block, shm, st, a...);
        PF_LAUNCH_CHECK();
        return;
    }
    if (grid.y != 1 || grid.z != 1 || block.y != 1 || block.z != 1) {
        fusion_host(s, [=](hipStream_t q) { hipLaunchKernelGGL(k, grid, block, shm, q, a...); });
        return;
    }
    using E = MEntry<P...>;
    static_assert(sizeof(E) % alignof(E) == 0 && alignof(E) <= 16, "entries of one launch are an array");
    const E e{grid.x, 0u, PackOf<P...>::make(static_cast<P>(a)...)};
    fusion_record(s, &run_multi<F, P...>, grid.x, block.x, shm, &e, sizeof(e));
}

// Host <-> device copies and stream synchronisation of a simulator's stream
// (recorded in a fusion group: host sources are copied at record time).
void copy_h2d(Sim& s, void* dst, const void* src, size_t bytes);
void copy_d2h(Sim& s, void* dst, const void* src, size_t bytes);
void stream_sync(Sim& s);
// Waits until *flag == seq, which the last kernel on the stream writes: polls,
// and leaves a longer wait (or an error) to the runtime.
void poll_flag(const unsigned long long* flag, unsigned long long seq, hipStream_t stream);

// Colour-split vector layout of the FP64 red-black ILU(0) path (PF order): the
// three planes (P, S, C) of the red cells ((ix+iy+iz) even), ns entries each,
// then those of the black cells, both in the slot order of the smoother's
// colour-split factors (x-lines of ceil(nx/2) slots, lines in natural order;
// where nx is odd every other line has a pad slot, which holds zero), then the
// wells.  A kernel over the cells of one colour writes whole cache lines, and
// the black cells and wells, which is what the Arnoldi process works on, are
// one run of 3 ns + nw entries.
__host__ __device__ __forceinline__ int64_t cs_ns(const DevModel& m) {
    return (int64_t)((m.nx + 1) / 2) * m.ny * m.nz;
}
// offset of the P entry of the cell with natural index i (S and C: ns and 2 ns on)
__device__ __forceinline__ int64_t cs_index(const DevModel& m, int64_t i) {
    const int64_t iz = i / m.nxy;
    const int64_t rem = i - iz * m.nxy;
    const int64_t iy = rem / m.nx;
    const int64_t ix = rem - iy * m.nx;
    return ((ix + iy + iz) & 1) * 3 * cs_ns(m) + (iy + m.ny * iz) * ((m.nx + 1) >> 1) + (ix >> 1);
}

// Storage of the off-diagonal blocks in that order (Lc).  Of a face's block,
// rows water, oil, polymer by columns P, S, C, the entry (oil, C) is zero, and
// as the polymer travels with the water the polymer row's P and S entries are
// those of the water row times one factor g (the upstream concentration, the
// viscosities' ratio and the rows' scales).  So kFaceVals values are kept:
// water P, S, C, oil P, S, g and polymer C.  They lie in blocks of 64 slots,
// all faces' values of a block together: a wavefront reads one run of 21.5 KB
// instead of 42 runs of 512 bytes in as many pages (reads of 48 values a slot
// alone: 5.55 TB/s for 5.26).  On 300^3, against eight values in planes: the
// assembly 3.34 ms for 3.95, k_ilu_diag 2.71 for 3.03, the smoother's and the
// product's kernels 9-10 % less.  Value v of face q of a slot is at
// lc_at(...) + (q kFaceVals + v) 64.
constexpr int kFaceVals = 7;
__host__ __device__ __forceinline__ int64_t lc_colour(int64_t ns) { return (ns + 63) / 64 * (64 * 6 * kFaceVals); }
__device__ __forceinline__ int64_t lc_at(int64_t ns, int64_t colour, int64_t s) {
    return colour * lc_colour(ns) + (s >> 6) * (64 * 6 * kFaceVals) + (s & 63);
}

// Whether the kernels stream J past the caches (non-temporal loads): where it
// does not stay in the 256 MB memory-side cache from one of them to the next
// beside what the other kernels read, which it would only push out.  The lines
// are those of whole timesteps (ms with streamed / plain loads, by the size of
// J): colour-split copies, FP64, 85 MB 3.93 / 3.83, 111 MB 5.81 / 5.68, 133 MB
// 5.51 / 5.46, 145 MB 4.88 / 4.89, 158 MB 7.05 / 7.13, 168 MB 7.28 / 7.40, 221
// MB 8.31 / 8.62, 327 MB 9.63 / 10.09; natural-order planes, block Jacobi in
// Algorithm 2's order, 114 MB 5.19 / 5.01, 148 MB 6.31 / 6.11, 163 MB 6.15 /
// 6.15, 178 MB 7.35 / 7.27, 194 MB 6.55 / 6.60, 224 MB 8.06 / 8.31, 435 MB
// 12.82 / 13.27, and mixed precision 163 MB 5.23 / 5.14, 178 MB 6.06 / 6.00,
// 194 MB 5.30 / 5.32, 224 MB 8.01 / 8.11.  (By themselves the kernels gain from
// plain loads up to 200 and 250 MB: 168 MB, four of them, 91.2 / 83.9 us.  From
// 13.5M cells on, 4.5 GB, the two are the same to 1 %.)  The members of a
// fusion group take turns at the cache, kernel by kernel, so theirs count
// together (a timestep of a group: 8 members of 50k cells, 136 MB in all, 8.61
// / 8.58; 8 of 101k, 271 MB, 8.62 / 9.04; 4 of 202k, 271 MB, 11.34 / 11.91; 4
// of 397k, 533 MB, 14.86 / 15.21; 16 of 397k 48.2 / 48.6).  The values loaded
// and their order are the same either way.
inline bool past_caches(const Sim& s, int64_t bytes, double line) {
    return (double)bytes * (double)fusion_cells(s) > line * (double)s.m.n;
}
bool stream_split(const Sim& s);     // the colour-split copies (k_cpr.hip)
inline bool stream_natural(const Sim& s) { return past_caches(s, 56 * s.m.n * (int64_t)sizeof(double), 185e6); }

// XCD-aware block order: workgroups are dispatched round-robin over the 8
// XCDs (each with its own L2); renumbering them so that XCD x processes one
// contiguous range of blocks keeps stencil neighbours in the same L2.
__device__ __forceinline__ int64_t xcd_block(const Blk& wg) {
    const int64_t nb = wg.n, b = wg.x;
    const int64_t q = nb >> 3, r = nb & 7, x = b & 7, j = b >> 3;
    return x * q + (x < r ? x : r) + j;
}

// y-strip order of a grid of lines of w entries (line = iy + ny*iz): strips
// of kStripLines lines in y, each taken layer by layer, a strip-layer being
// one contiguous run of entries.  Maps a thread index v to an entry (a
// bijection on [0, w*ny*nz)); the last strip may hold fewer lines.  Kernels
// whose threads read neighbours one layer up or down use it on grids with
// large layers, so that those neighbours were read a strip-layer earlier
// (within the reach of the L2 cache) rather than a whole layer earlier.
constexpr int64_t kStripLines = 16;
__device__ __forceinline__ int64_t strip_order(int64_t v, int64_t w, int64_t ny, int64_t nz) {
    if (ny <= kStripLines) return v;
    const int64_t full = kStripLines * w * nz;          // entries of a strip of kStripLines lines
    const int64_t st = v / full;
    const int64_t y0 = st * kStripLines;
    const int64_t lines = min(kStripLines, ny - y0);
    const int64_t r = v - st * full;
    const int64_t per_layer = lines * w;
    const int64_t iz = r / per_layer;
    const int64_t r2 = r - iz * per_layer;
    return (y0 + ny * iz) * w + r2;                     // line (y0 + r2 / w, iz), entry r2 % w
}

// The cell a natural-order kernel's thread v takes: y-strips on grids whose
// layers hold at least kStripCells cells, natural order otherwise.
constexpr int64_t kStripCells = 65536;
__device__ __forceinline__ int64_t strip_cell(const DevModel& m, int64_t v) {
    if (m.nxy < kStripCells) return v;
    return strip_order(v, m.nx, m.ny, m.nz);
}

inline unsigned grid_for(int64_t n, int block = kBlock) {
    int64_t g = (n + block - 1) / block;
    return (unsigned)(g > 0 ? g : 1);
}

}  // namespace pf

// the simulator behind a handle of the C interface
pf::Sim& pf_sim_state(pf_sim* h);
