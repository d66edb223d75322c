// henry_device.hpp -- gfx950 device code for batched Henry solves.
//
// One workgroup, or for a large grid a cluster of 2-8 workgroups on one XCD,
// owns one solve (one random sample on one grid) and runs its whole
// implicit time loop (Sec. 2.3: implicit Euler, fixed tau).  Each step
// is a defect correction on the FP64 nonlinear residual of the cell-centred
// discretisation of e_cont_eq / e_tran_eq / e_Darcy_vel (Sec. 2.1):
//
//   repeat
//     R = R(p, c)                                   FP64, scaled max norms
//     stop if both norms <= tol
//     unless |R^p| <= tol:
//       (A_pp) dp = -R^p  one V(2,2) cycle, red-black Gauss-Seidel   inner T
//       p += dp                                                       FP64
//     R = R(p, c), S = R^c - c R^p                                    FP64
//     stop if both norms <= tol
//     (A_cc) dc = -S      one V-cycle, zebra x-lines before the coarse
//                         correction, x- (global levels) or y-lines
//                         (LDS levels) after                      inner T
//     c += dc                                                         FP64
//
// Each step starts from an extrapolation through the last converged states
// (interpolating polynomials up to cubic, then on long solves the
// least-squares cubic through five states; see implicit_step).
//
// A_pp = -div(rho K / mu grad .) with the seawater Dirichlet face.  The salt
// block is driven by S = R^c - c R^p, an exact recombination of the two
// equations (same discrete solution): S is the non-conservative upwind form
// of e_tran_eq, in which a mass-flux error of an inexact pressure solve no
// longer appears as a salt source.  A_cc, its frozen-flux derivative, is an
// M-matrix with the stored-mass term (h^2/tau) phi rho(c^n) on the diagonal
// and upwind inflow plus diffusion couplings.  The inner precision T is float (the
// mixed path) or double (the plain FP64 path): one code path, two
// instantiations.  Memory: per-solve FP64 state and per-level inner arrays
// in a caller-provided workspace (L2 / Infinity-Cache resident for the
// grid sizes of an MLMC hierarchy); line systems are solved in registers by
// segmented elimination with a cyclic-reduction interface solve across the
// lanes of a wavefront.
#pragma once

#include <type_traits>

#include <hip/hip_runtime.h>
#include <stdint.h>

// The namespace and the FP32 kernel's workgroup bound of this build: the
// library compiles this header twice, as henry with 1024-thread bounds
// (henry_api.hip) and as henry512 with 512-thread bounds (henry_solve512.hip),
// so that each build's device functions get their own register budget.
#ifndef HENRY_NS
#define HENRY_NS henry
#endif
#ifndef HENRY_FP32_THREADS
#define HENRY_FP32_THREADS 1024
#endif
// Grids of at least HENRY_RES_FIELDS_NX columns (0: none): the residual
// pass forms the face coefficients and the norm scale from K and phi (5 FP64
// loads per cell instead of 9, and three FP64 divisions); smaller ones load
// the stored ones.  Both give the same bits.
#ifndef HENRY_RES_FIELDS_NX
#define HENRY_RES_FIELDS_NX 0
#endif
// Cells per thread gathered by the grid transfers of the builds with at most
// 512 threads (the 1024-thread build takes one).
#ifndef HENRY_TRANSFER_BATCH
#define HENRY_TRANSFER_BATCH 1
#endif

namespace HENRY_NS {

// Cells per thread whose operands a transfer between levels (restriction,
// prolongation, coefficient coarsening) from a finer level in global memory
// gathers before it writes any, so that their loads are in flight together;
// the 1024-thread build has no registers to spare for more than one.
constexpr int kTBatch = HENRY_FP32_THREADS <= 512 ? HENRY_TRANSFER_BATCH : 1;
// strips of eight cells per thread take more registers than the 1024-thread build has
constexpr bool kStripWide = HENRY_FP32_THREADS <= 512;

constexpr int kMaxLevels = 12;  // ny <= 512 -> at most 10 multigrid levels
constexpr int kWave = 64;

struct Phys {
    double rho0, rho1, mu, g, D, phi0, k0, q_in, T;
};

// One solve of a batch.  Offsets are in bytes from the workspace base
// (ws_off) or in elements of the packed field arrays (field_off).
struct SolveDesc {
    int32_t nx, ny, nsteps, nlev;
    int32_t reserved;
    int32_t index;       // position in the caller's solve list
    int64_t ws_off;
    int64_t field_off;
    int64_t adj_off;     // adjoint region (adjoint calls only)
};

struct Launch {
    const SolveDesc* descs;
    uint8_t* ws;
    const double* xi;    // [nsolves][3] or null
    const double* phi_in;
    const double* logk_in;
    const double* qin_in;
    const double* c0;
    double* c_out;
    double* p_out;
    double* qoi_out;
    int32_t* status;
    int32_t* iters;
    Phys ph;
    double tol;
    int32_t max_outer;
    int32_t predictor;       // henry_opts_t.predictor
    int32_t field_kind;
    int32_t g_begin, g_end;  // global step range of this launch
    int32_t g_total;         // global steps of the whole batch (max nsteps)
    int32_t lds_cells;       // multigrid levels with at most this many cells live in LDS (wavefront 0)
    int32_t lds_block_cells; // levels 1.. with at most this many cells also live in LDS (whole workgroup)
    int32_t lds_bytes;       // dynamic LDS of the launch (the LDS levels, or the line staging if larger)
    int32_t xi_dim;          // coefficients per solve in xi (3 closed form, 41 KL)
    const double* kl_modes;  // KL: sqrt(lam_k) e_k at the cells of this group's grid, [20][n]
    double kl_sigma_phi, kl_sigma_logk;
    int32_t nsolves;         // solves of this launch (descs[0 .. nsolves-1])
    int32_t cluster;         // workgroups per solve (1, 2, 4 or 8)
    uint64_t cluster_wait;   // bound of one cluster-barrier wait, ticks of the 100 MHz wall clock
    int32_t redo;            // a solve whose cluster's wait runs out is left to another launch (henry_redo_kernel)
    // time series (forward solves only; trace == nullptr: none): record k =
    // 1..trace_nrec after step ceil(k nsteps / trace_nrec), holding the
    // fresh-water area and c at trace_npts points, at
    // trace[index][k-1][0 .. trace_npts]
    double* trace;
    int32_t trace_nrec, trace_npts;
    double trace_fresh;             // c threshold of the fresh-water indicator
    double trace_pts[2 * 16];       // (x, y) of each point
};

constexpr int kMaxTracePoints = 16;
constexpr int kStatusSync = 3;  // HENRY_STATUS_SYNC

// ------------------------------------------------------------------ layout
__host__ __device__ inline int64_t align256(int64_t b) { return (b + 255) & ~int64_t(255); }

__host__ __device__ inline int num_levels(int ny) {
    int L = 1;
    while (ny > 1) { ny >>= 1; ++L; }
    return L;
}

// Per-level inner arrays, in this order, each nx_l*ny_l elements of T:
//   x, b, r, te, tn, acc, mx, my, dx, dy
// followed by four row arrays of ny_l elements: dl, dr, mr, ml
// (left diffusion, right diffusion, right mass flux, left inflow).
constexpr int kLevelArrays = 10;
constexpr int kRowArrays = 4;

template <typename T>
__host__ __device__ inline int64_t level_bytes(int nx, int ny) {
    return align256((int64_t)(kLevelArrays * nx * ny + kRowArrays * ny) * (int64_t)sizeof(T));
}

// FP64 arrays: p, c, cn, phi, K, pp (previous p), then the face
// coefficients that depend only on the fields, set once per solve:
//   tx, ty  east / north face K_f / mu (harmonic K; 2 K_P / mu on the
//           seawater face; 0 above the top row),
//   wx, wy  east / north face phi_f D (harmonic phi; 2 phi_P D on the
//           seawater face; 0 above the top row),
//   isc     residual scale tau / (h^2 phi_P rho0),
// then the older states c2, p2 (u^{n-2}), c3, p3 (u^{n-3}) and c4, p4
// (u^{n-4}) of the extrapolated initial guess (their roles rotate: bind_history), then kScratch doubles of
// scratch: [0] recharge, [1] status, [2] outer iterations, [3] converged states in a row, [4] the history's
// rotation at the end of a launch, [6] the arrivals and failures of a cluster on one XCD, [8..31]
// phase timers of builds with HENRY_PHASE_TIMERS, [32..63] the state of a cluster of workgroups sharing the solve (the members'
// 32-bit arrival counts in [32..35], the error flag in [36], barriers passed [37], the members' XCD
// ids [40..47], their partial residual norms [48..63]).
enum : int { kP, kC, kCn, kPhi, kK, kPp, kTx, kTy, kWx, kWy, kIsc, kC2, kP2, kC3, kP3, kC4, kP4, kF64Arrays };
constexpr int kScratch = 64;
constexpr int kClusterHere = 6, kClusterFlags = 32, kClusterErr = 36, kClusterGen = 37, kClusterXcc = 40, kClusterSlots = 48;
constexpr int kMaxCluster = 8;
// the barrier polls the K arrival counts and the error flag in one load:
// the flag sits past the last count, within one wavefront's lanes
static_assert((kClusterErr - kClusterFlags) * 2 >= kMaxCluster && (kClusterErr - kClusterFlags) * 2 < 64,
              "cluster error flag placement");

template <typename T>
__host__ __device__ inline int64_t solve_bytes(int nx, int ny) {
    int64_t b = align256((int64_t)kF64Arrays * nx * ny * 8 + kScratch * 8);
    int lx = nx, ly = ny;
    const int L = num_levels(ny);
    for (int l = 0; l < L; ++l) {
        b += level_bytes<T>(lx, ly);
        lx >>= 1; ly >>= 1;
    }
    return b;
}

template <typename T>
struct Level {
    using value_type = T;
    int nx, ny;
    T *x, *b, *r, *te, *tn, *acc, *mx, *my, *dx, *dy, *dl, *dr, *mr, *ml;
};

// Address-space-typed view of a level for the smoothers and transfers: AS 1
// (global memory) or 3 (LDS) lets the compiler emit global_* / ds_*
// instructions instead of flat ones; AS 0 keeps generic pointers.
template <typename T, int AS> struct AsPtr { using type = T*; };
template <typename T> struct AsPtr<T, 1> { using type = __attribute__((address_space(1))) T*; };
template <typename T> struct AsPtr<T, 3> { using type = __attribute__((address_space(3))) T*; };
template <int AS, typename T>
__device__ inline typename AsPtr<T, AS>::type as_ptr(T* p) { return (typename AsPtr<T, AS>::type)p; }

template <typename T, int AS>
struct LV {
    using value_type = T;
    using P = typename AsPtr<T, AS>::type;
    int nx, ny;
    P x, b, r, te, tn, acc, mx, my, dx, dy, dl, dr, mr, ml;
    __device__ explicit LV(const Level<T>& v)
        : nx(v.nx), ny(v.ny), x(as_ptr<AS>(v.x)), b(as_ptr<AS>(v.b)), r(as_ptr<AS>(v.r)), te(as_ptr<AS>(v.te)),
          tn(as_ptr<AS>(v.tn)), acc(as_ptr<AS>(v.acc)), mx(as_ptr<AS>(v.mx)), my(as_ptr<AS>(v.my)),
          dx(as_ptr<AS>(v.dx)), dy(as_ptr<AS>(v.dy)), dl(as_ptr<AS>(v.dl)), dr(as_ptr<AS>(v.dr)),
          mr(as_ptr<AS>(v.mr)), ml(as_ptr<AS>(v.ml)) {}
};

template <typename T>
struct Solve {
    int nx, ny, n, nsteps, L;
    int lds_from;  // first level whose arrays live in LDS and that wavefront 0 runs alone
    int lb;        // first level whose arrays live in LDS (lb <= lds_from)
    int lc;        // levels 0 .. lc-1 are run by the whole cluster (0 with one workgroup)
    int hand;      // level lc is in LDS and fed by the cluster through its global copy hg
    int hist;      // rotation of the state history (see bind_history)
    double h, tau;
    double q;  // recharge (m/s)
    Phys ph;
    double *p, *c, *cn, *phi, *K, *pp, *tx, *ty, *wx, *wy, *isc, *c2, *p2, *c3, *p3, *c4, *p4, *scratch;
    Level<T> lv[kMaxLevels];
    Level<T> hg;  // the global-memory arrays of level lb
    T* wave;      // LDS of the levels wavefront 0 runs (henry_wave.hpp)
    double *rout_p, *rout_c;  // residual outputs (henry_residual_kernel)
};

// Levels in LDS: every level of at most `lds_cells` cells (run by
// wavefront 0), and levels 1.. of at most `lds_block_cells` cells (run by
// the whole workgroup; level 0 always stays in global memory, where the
// FP64 residual pass of the whole cluster writes it).
__host__ __device__ inline bool level_in_lds(int l, int cells, int lds_cells, int lds_block_cells) {
    return cells <= lds_cells || (l >= 1 && cells <= lds_block_cells);
}

// One wave level of NX x NX/2 cells: x with a halo of one cell around it
// (pressure: two colours of H cells per row, each with its own halo;
// transport: rows of NX cells from column 2 on), the residual that the
// restriction reads (red cells, or even rows), and for the levels below the
// first the coefficients and right-hand side.  Levels lie one after another
// from the coarsest up, so their places do not depend on which is first.
constexpr int ilog2(int v) { return v > 1 ? 1 + ilog2(v / 2) : 0; }
constexpr int round4(int v) { return (v + 3) & ~3; }
template <int NX>
struct WaveDim {
    static constexpr int NY = NX / 2, H = NX / 2, N = NX * NY;
    static constexpr int CS = H + 2;       // colour stride (pressure)
    static constexpr int RS = NX + 4;      // row stride of x
    static constexpr int kX = (NY + 2) * RS;
    static constexpr int kR = (NY + 2) * CS;  // red cells; the even rows (NY/2 + 1) * RS take no more
    static constexpr int kXR = round4(kX + kR);
    static constexpr int kCoef = round4(6 * N + 4 * NY);
    static constexpr int base() {
        if constexpr (NX == 2) return 0;
        else return WaveDim<NX / 2>::base() + WaveDim<NX / 2>::kXR + WaveDim<NX / 2>::kCoef;
    }
};
// Elements of the wave region below a first level of nx columns.
__host__ __device__ inline int wave_region_elems(int nx) {
    switch (nx) {
        case 2: return WaveDim<2>::base() + WaveDim<2>::kXR;
        case 4: return WaveDim<4>::base() + WaveDim<4>::kXR;
        case 8: return WaveDim<8>::base() + WaveDim<8>::kXR;
        case 16: return WaveDim<16>::base() + WaveDim<16>::kXR;
        default: return WaveDim<32>::base() + WaveDim<32>::kXR;
    }
}

// The first level that wavefront 0 runs keeps its arrays but r in LDS (the
// rest of the workgroup, or the cluster, writes its coefficients and
// right-hand side and reads its x); what it and the coarser levels need
// besides lives in the wave region after them (henry_wave.hpp).
template <typename T>
__host__ __device__ inline int64_t wave_top_bytes(int nx, int ny) {
    return align256((int64_t)((kLevelArrays - 1) * nx * ny + kRowArrays * ny) * (int64_t)sizeof(T));
}
template <typename T>
__host__ __device__ inline int64_t wave_region_bytes(int nx) {
    return align256((int64_t)wave_region_elems(nx) * (int64_t)sizeof(T));
}

// Dynamic LDS bytes for the LDS levels of an nx x ny hierarchy.
template <typename T>
__host__ __device__ inline int64_t lds_level_bytes(int nx, int ny, int lds_cells, int lds_block_cells) {
    int64_t b = 0;
    int lx = nx, ly = ny;
    const int L = num_levels(ny);
    for (int l = 0; l < L; ++l) {
        if (lx * ly <= lds_cells) return b + wave_top_bytes<T>(lx, ly) + wave_region_bytes<T>(lx);
        if (level_in_lds(l, lx * ly, lds_cells, lds_block_cells)) b += level_bytes<T>(lx, ly);
        lx >>= 1; ly >>= 1;
    }
    return b;
}

// The state history: five arrays per field hold the iterate and the four
// converged states before it, u^n .. u^{n-3} (the roles c / cn / c2 / c3 /
// c4 and p / pp / p2 / p3 / p4).  A step's extrapolated start overwrites the
// oldest state in place (each cell reads only its own history) and the roles
// then rotate by one: role k is array (k + hist) mod 5 of the field, and a
// step takes hist to hist + 4 mod 5.  One write per cell and field instead of
// five (the older states are never copied).
template <typename T>
__device__ inline void bind_history(Solve<T>& S, uint8_t* base) {
    double* f = reinterpret_cast<double*>(base);
    const int64_t n = (int64_t)S.nx * S.ny;
    const int cs[5] = {kC, kCn, kC2, kC3, kC4}, ps[5] = {kP, kPp, kP2, kP3, kP4};
    double** cr[5] = {&S.c, &S.cn, &S.c2, &S.c3, &S.c4};
    double** pr[5] = {&S.p, &S.pp, &S.p2, &S.p3, &S.p4};
    for (int k = 0; k < 5; ++k) {
        *cr[k] = f + (int64_t)cs[(k + S.hist) % 5] * n;
        *pr[k] = f + (int64_t)ps[(k + S.hist) % 5] * n;
    }
}

// Binds the solve's arrays.  The LDS levels (level_in_lds) get their inner
// arrays in the workgroup's LDS (`lds`): they are rebuilt every iteration,
// so nothing there has to survive a launch.  Every level keeps its region
// in the workspace too (S.hg views that of level lb).  lds_cells >= 2, so
// the coarsest level (2 x 1) is always in LDS and S.lds_from < S.L; the
// levels after S.lds_from are places of the wave region and are not bound.
template <typename T>
__device__ inline void bind_solve(Solve<T>& S, uint8_t* base, int nx, int ny, uint8_t* lds, int lds_cells,
                                  int lds_block_cells) {
    S.nx = nx; S.ny = ny; S.n = nx * ny; S.L = num_levels(ny);
    S.h = 1.0 / ny;
    double* f = reinterpret_cast<double*>(base);
    const int n = nx * ny;
    auto arr = [&](int k) { return f + (int64_t)k * n; };
    S.phi = arr(kPhi); S.K = arr(kK);
    S.tx = arr(kTx); S.ty = arr(kTy); S.wx = arr(kWx); S.wy = arr(kWy); S.isc = arr(kIsc);
    S.scratch = arr(kF64Arrays);
    S.hist = 0;
    bind_history(S, base);
    uint8_t* q = base + align256((int64_t)kF64Arrays * n * 8 + kScratch * 8);
    uint8_t* ql = lds;
    int lx = nx, ly = ny;
    S.lds_from = S.L;
    S.lb = S.L;
    S.lc = 0;
    S.hand = 0;
    S.wave = nullptr;
    auto bind_level = [](Level<T>& v, T* a, int lx, int ly, bool with_r = true) {
        const int m = lx * ly;
        v.nx = lx; v.ny = ly;
        v.x = a; v.b = a + m;
        T* f = a + (with_r ? 3 : 2) * m;
        v.r = with_r ? a + 2 * m : nullptr;
        v.te = f; v.tn = f + m; v.acc = f + 2 * m; v.mx = f + 3 * m; v.my = f + 4 * m; v.dx = f + 5 * m;
        v.dy = f + 6 * m;
        f += 7 * m;
        v.dl = f; v.dr = f + ly; v.mr = f + 2 * ly; v.ml = f + 3 * ly;
    };
    for (int l = 0; l < S.L; ++l) {
        const bool in_lds = level_in_lds(l, lx * ly, lds_cells, lds_block_cells);
        if (in_lds && S.lb == S.L) {
            S.lb = l;
            bind_level(S.hg, reinterpret_cast<T*>(q), lx, ly);
        }
        if (lx * ly <= lds_cells) {
            S.lds_from = l;
            bind_level(S.lv[l], reinterpret_cast<T*>(ql), lx, ly, false);
            S.wave = reinterpret_cast<T*>(ql + wave_top_bytes<T>(lx, ly));
            break;
        }
        bind_level(S.lv[l], reinterpret_cast<T*>(in_lds ? ql : q), lx, ly);
        if (in_lds) ql += level_bytes<T>(lx, ly);
        q += level_bytes<T>(lx, ly);
        lx >>= 1; ly >>= 1;
    }
}

// ------------------------------------------------------------------ reductions
// max that propagates NaN (fmax would drop it)
__device__ inline double nanmax(double a, double b) { return (a > b || a != a) ? a : b; }

__device__ inline double wave_max(double v) {
    for (int o = kWave / 2; o > 0; o >>= 1) v = nanmax(v, __shfl_xor(v, o));
    return v;
}
__device__ inline double wave_sum(double v) {
    for (int o = kWave / 2; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

// Block-wide max / sum in a fixed order; `red` holds >= nwaves doubles.
// Ends with every thread holding the result.
__device__ inline double block_max(double v, double* red) {
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave, nw = blockDim.x / kWave;
    v = wave_max(v);
    __syncthreads();
    if (lane == 0) red[w] = v;
    __syncthreads();
    double r = red[0];
    for (int k = 1; k < nw; ++k) r = nanmax(r, red[k]);
    return r;
}
__device__ inline void block_max2(double& a, double& b, double* red) {
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave, nw = blockDim.x / kWave;
    a = wave_max(a);
    b = wave_max(b);
    __syncthreads();
    if (lane == 0) { red[2 * w] = a; red[2 * w + 1] = b; }
    __syncthreads();
    double ra = red[0], rb = red[1];
    for (int k = 1; k < nw; ++k) { ra = nanmax(ra, red[2 * k]); rb = nanmax(rb, red[2 * k + 1]); }
    a = ra;
    b = rb;
}
__device__ inline double block_sum(double v, double* red) {
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave, nw = blockDim.x / kWave;
    v = wave_sum(v);
    __syncthreads();
    if (lane == 0) red[w] = v;
    __syncthreads();
    double r = red[0];
    for (int k = 1; k < nw; ++k) r += red[k];
    return r;
}

// Every level's nx and ny are powers of two: cell coordinates come from
// shifts and masks instead of integer division.
__device__ inline int log2i(int v) { return __builtin_ctz((unsigned)v); }

// Division inside the FP32 inner solves uses the hardware reciprocal (about
// 1 ulp; the solves only precondition the FP64 defect correction); the FP64
// path divides exactly.
template <typename T>
__device__ inline T qdiv(T a, T b) {
    if constexpr (sizeof(T) == 4) return a * __builtin_amdgcn_rcpf(b);
    else return a / b;
}

// ------------------------------------------------------------------ vectors and lanes
template <typename T> using LdsPtr = typename AsPtr<T, 3>::type;
template <typename T> using Vec2 = T __attribute__((ext_vector_type(2)));
template <typename T> using Vec4 = T __attribute__((ext_vector_type(4)));

template <typename T>
__device__ inline Vec2<T> lds_load2(LdsPtr<T> p) { return *(typename AsPtr<Vec2<T>, 3>::type)p; }
template <typename T>
__device__ inline void lds_store2(LdsPtr<T> p, T a, T b) {
    Vec2<T> v = {a, b};
    *(typename AsPtr<Vec2<T>, 3>::type)p = v;
}

// Value of the lane kN below (above) within its row of 16 lanes; 0 where
// the row ends.
template <int kCtrl>
__device__ inline float dpp_row(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), kCtrl, 0xf, 0xf, true));
}
template <int kCtrl>
__device__ inline double dpp_row(double v) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), kCtrl, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), kCtrl, 0xf, 0xf, true);
    return __hiloint2double(hi, lo);
}
// Value of the lane below / above in the wavefront; `end` where it ends.
template <int kCtrl>
__device__ inline double dpp_wave(double v, double end) {
    const int lo = __builtin_amdgcn_update_dpp(__double2loint(end), __double2loint(v), kCtrl, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(__double2hiint(end), __double2hiint(v), kCtrl, 0xf, 0xf, false);
    return __hiloint2double(hi, lo);
}
__device__ inline double wave_below(double v, double end) { return dpp_wave<0x138>(v, end); }  // wave_shr:1
__device__ inline double wave_above(double v, double end) { return dpp_wave<0x130>(v, end); }  // wave_shl:1

// Values that every lane of the wavefront holds alike, in scalar registers.
__device__ inline int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ inline double uniform(double v) {
    return __hiloint2double(uniform(__double2hiint(v)), uniform(__double2loint(v)));
}
template <typename P>
__device__ inline P* uniform(P* p) {
    const uint64_t v = reinterpret_cast<uint64_t>(p);
    return reinterpret_cast<P*>((uint64_t)(uint32_t)uniform((int)(uint32_t)v) |
                                ((uint64_t)(uint32_t)uniform((int)(v >> 32)) << 32));
}
// v of lane t (uniform)
__device__ inline double lane_value(double v, int t) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), t),
                            __builtin_amdgcn_readlane(__double2loint(v), t));
}

template <int kN, typename T> __device__ inline T lane_below(T v) { return dpp_row<0x110 + kN>(v); }  // row_shr
template <int kN, typename T> __device__ inline T lane_above(T v) { return dpp_row<0x100 + kN>(v); }  // row_shl

// ------------------------------------------------------------------ rounding
// A product that is rounded before it is added to anything.
template <typename T>
__device__ inline T rounded_mul(T a, T b) {
#pragma clang fp contract(off)
    const T p = a * b;
    return p;
}

// Where a sum of two products could be fused either way, the choice is
// written out, so that the code that runs a level does not change its
// rounding.
__device__ inline float fused(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ inline double fused(double a, double b, double c) { return __builtin_fma(a, b, c); }

// Bilinear prolongation weights 9/16, 3/16, 3/16, 1/16.
template <typename T>
__device__ inline T prolonged(T near, T side, T up, T far) {
    return fused((T)0.0625, far, fused((T)0.5625, near, rounded_mul((T)0.1875, side + up)));
}

// Diagonal as the smoother divides by it: its reciprocal for float (qdiv's),
// itself for double.
template <typename T>
__device__ inline T diag_prep(T d) {
    if constexpr (sizeof(T) == 4) return __builtin_amdgcn_rcpf(d);
    else return d;
}
template <typename T>
__device__ inline T diag_div(T a, T prep) {
    if constexpr (sizeof(T) == 4) return rounded_mul(a, prep);  // not fused into what it is added to next
    else return a / prep;
}

// ------------------------------------------------------------------ teams
// The threads that run one multigrid operation together: the whole
// workgroup (levels in global memory), or wavefront 0 alone (the coarse
// levels in LDS, where barrier latency would dominate the little work).
// Within one wavefront the lanes execute in lockstep and LDS operations of
// the wavefront complete in issue order, so a wavefront-scope fence (which
// keeps the compiler from moving memory operations across it) is the whole
// synchronisation.
struct BlockTeam {
    __device__ static int rank() { return threadIdx.x; }
    __device__ static int size() { return blockDim.x; }
    __device__ static void sync() { __syncthreads(); }
};
struct WaveTeam {
    __device__ static void sync() {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
};

// ------------------------------------------------------------------ clusters
// A large grid's solve can be shared by K workgroups (a cluster, K = 2, 4
// or 8), one per CU: the fine levels (0 .. S.lc-1) are split over all
// K x blockDim threads, while member 0 (the leader) runs the coarse levels
// alone.  Every cell and every line is computed by the same arithmetic
// whatever the split, and the residual norms are maxima, so a solve gives
// bitwise the same result for every K.
//
// Members of a cluster are placed on one XCD: the workgroups of a launch
// are dealt to the eight XCDs round robin (block b on XCD b mod 8), so the
// members of cluster c on XCD x are K consecutive blocks of that XCD's
// sequence.  Each launch checks the placement (hardware XCC id, exchanged
// under an agent-scope barrier).  Clusters whose members share one XCD, and
// so one L2, synchronise through an atomic counter in that L2: each member's
// arrival is one atomic that returns the count, so the last to arrive does
// not poll, and the others poll with atomics too (the texture cache does not
// hold them); then the L1 is invalidated.  Any other cluster uses
// agent-scope stores and loads of the members' counts, with a release (L2
// write-back) before.  Blocks of one XCD are dispatched in order, so the
// lowest cluster not yet complete always gets its members.  Every wait is
// bounded (Launch::cluster_wait, 10 s by default): past it a member raises
// the cluster's error flag, every later barrier of the cluster returns at
// once, and the solve reports HENRY_STATUS_SYNC.
struct ClusterState {
    int K, member, base, size;
    unsigned* flags; // [K] barriers each member has arrived at
    unsigned* err;   // sticky error flag
    unsigned long long* here;  // members on one XCD: arrivals of this launch, failures from bit 56 on
    double* slots;   // [2K] partial norms
    unsigned gen;    // barriers passed
    unsigned long long gen_here;  // of them through `here`, this launch
    int local;       // all members on one XCD
    int failed;
    int redo;        // Launch::redo
    uint64_t wait;   // bound of one wait (wall-clock ticks)
    uint8_t* stage;  // the dynamic LDS, as line staging buffers on the cluster levels
    int stage_waves; // wavefronts whose staging buffer fits in it
    int stage_bytes; // its size
};
__shared__ ClusterState g_cl;

__device__ inline int xcc_id() { return __builtin_amdgcn_s_getreg(20 | (0 << 6) | (3 << 11)); }

// Adds v to a cluster's counter in the L2 of the calling XCD and returns the
// value before.  Written out, with its wait, because the atomic must be
// performed in that L2 (no sc1: device scope would send it past it, to the
// point where the XCDs meet) and by the one lane that calls it (the
// compiler would add a scan over the lanes).
__device__ inline unsigned long long l2_fetch_add(unsigned long long* p, unsigned long long v) {
    unsigned long long old;
    asm volatile("global_atomic_add_x2 %0, %1, %2, off sc0\n\ts_waitcnt vmcnt(0)"
                 : "=&v"(old)
                 : "v"(p), "v"(v)
                 : "memory");
    return old;
}

// The same without the value before.
__device__ inline void l2_add(unsigned long long* p, unsigned long long v) {
    asm volatile("global_atomic_add_x2 %0, %1, off\n\ts_waitcnt vmcnt(0)" : : "v"(p), "v"(v) : "memory");
}

constexpr int kFailBit = 56;

// The bound of a wait: the wall clock is first read after a poll that found
// the members missing (reading it before would delay every barrier by its
// latency), then every 8 polls.
struct WaitClock {
    uint64_t t0;
    unsigned polls = 0;
    __device__ inline bool expired(uint64_t wait) {
        if ((polls++ & 7u) != 0u) return false;
        const uint64_t t = wall_clock64();
        if (polls == 1u) t0 = t;
        return t - t0 > wait;
    }
};

// Every workgroup of a cluster waits until all K members have arrived; all
// memory operations before the call are visible to every member after it.
// On one XCD lane 0 of wavefront 0 arrives and polls (256x128 at K = 8, 24
// barriers an iteration: 215 -> 208 us).  Elsewhere wavefront 0 publishes the
// member's arrival count and polls the K counts and the cluster's error flag
// with one load per lane (lane k < K: member k's count; the lane at the error
// flag's offset: the flag), so that one poll is one round trip.  One acquire
// fence after the members are all there makes their stores visible.
__device__ inline void cluster_barrier() {
    __builtin_amdgcn_s_waitcnt(0);  // this thread's stores have reached L2
    __syncthreads();
    if (threadIdx.x < kWave) {
        const int lane = (int)threadIdx.x;
        const unsigned gen = g_cl.gen + 1u;
        bool failed = false;
        if (g_cl.local && !g_cl.failed) {
            if (lane == 0) {
                unsigned long long* here = g_cl.here;
                const unsigned long long all = (g_cl.gen_here + 1ull) * (unsigned)g_cl.K;
                unsigned long long v = l2_fetch_add(here, 1ull) + 1ull;
                WaitClock clk;
                while (v < all || (v >> kFailBit) != 0ull) {
                    if ((v >> kFailBit) != 0ull || clk.expired(g_cl.wait)) {
                        failed = true;
                        break;
                    }
                    v = l2_fetch_add(here, 0ull);
                }
                if (failed) {
                    l2_add(here, 1ull << kFailBit);
                    __hip_atomic_store(g_cl.err, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    g_cl.failed = 1;
                }
                g_cl.gen_here += 1ull;
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        } else if (!g_cl.failed) {
            if (lane == 0) __hip_atomic_store(g_cl.flags + g_cl.member, gen, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
            const int eoff = (int)(g_cl.err - g_cl.flags);  // the error flag's offset (>= K)
            const bool is_err = lane == eoff;
            const unsigned* f = g_cl.flags + (lane < g_cl.K || is_err ? lane : 0);
            WaitClock clk;
            for (;;) {
                const unsigned v = __hip_atomic_load(f, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (__any(is_err && v != 0u)) {
                    failed = true;
                    break;
                }
                if (__all(is_err || (int)(v - gen) >= 0)) break;
                if (clk.expired(g_cl.wait)) {
                    failed = true;
                    break;
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
            if (failed && lane == 0) {
                __hip_atomic_store(g_cl.err, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                g_cl.failed = 1;
            }
        }
        if (lane == 0) g_cl.gen = gen;
    }
    __syncthreads();
}

// All K x blockDim threads of the cluster (the workgroup when K = 1).
struct ClusterTeam {
    __device__ static int rank() { return g_cl.base + (int)threadIdx.x; }
    __device__ static int size() { return g_cl.size; }
    __device__ static void sync() {
        if (g_cl.K == 1) __syncthreads();
        else cluster_barrier();
    }
};

// The launch's dynamic LDS as line staging buffers (thread 0; read after the
// next workgroup barrier).
__device__ inline void cluster_stage(uint8_t* lds, int lds_bytes, int64_t per_wave) {
    g_cl.stage = lds;
    g_cl.stage_waves = (int)(lds_bytes / per_wave);
    g_cl.stage_bytes = lds_bytes;
}

// Cluster of one workgroup (the adjoint kernel, small grids).
__device__ inline void cluster_init_single() {
    if (threadIdx.x == 0) {
        g_cl.K = 1; g_cl.member = 0; g_cl.base = 0; g_cl.size = (int)blockDim.x;
        g_cl.flags = nullptr; g_cl.err = nullptr; g_cl.here = nullptr; g_cl.slots = nullptr;
        g_cl.gen = 0u; g_cl.gen_here = 0ull; g_cl.local = 1; g_cl.failed = 0; g_cl.wait = 0;
        g_cl.stage = nullptr; g_cl.stage_waves = 0; g_cl.stage_bytes = 0;  // no line staging unless cluster_stage says so
    }
    __syncthreads();
}

// Binds member `member` of a K-cluster to the cluster state in the solve's
// scratch `sp` and checks the members' placement.
__device__ inline void cluster_init(int K, int member, double* sp, uint64_t wait, int redo) {
    if (threadIdx.x == 0) {
        g_cl.wait = wait;
        g_cl.redo = redo;
        g_cl.K = K; g_cl.member = member; g_cl.base = member * (int)blockDim.x; g_cl.size = K * (int)blockDim.x;
        g_cl.flags = reinterpret_cast<unsigned*>(sp + kClusterFlags);
        g_cl.err = reinterpret_cast<unsigned*>(sp + kClusterErr);
        g_cl.slots = sp + kClusterSlots;
        g_cl.gen = (unsigned)sp[kClusterGen];
        g_cl.gen_here = 0ull;
        g_cl.here = reinterpret_cast<unsigned long long*>(sp + kClusterHere);
        if (member == 0) *g_cl.here = 0ull;  // in the L2 of a cluster on one XCD before any member passes the next barrier
        g_cl.local = 0;  // the placement check itself uses the agent-scope protocol
        g_cl.failed = 0;
        g_cl.stage = nullptr; g_cl.stage_waves = 0; g_cl.stage_bytes = 0;  // no line staging unless cluster_stage says so
        sp[kClusterXcc + member] = (double)xcc_id();
    }
    cluster_barrier();
    if (threadIdx.x == 0) {
        // a cluster that failed in an earlier launch stays failed
        if (__hip_atomic_load(g_cl.err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0u) g_cl.failed = 1;
        int same = 1;
        const double x0 = sp[kClusterXcc];
        for (int k = 1; k < K; ++k) same &= sp[kClusterXcc + k] == x0 ? 1 : 0;
        g_cl.local = same;
    }
    __syncthreads();
}

// Maxima of two per-thread values over the whole cluster, in a fixed order
// (NaN propagates); every thread of every member gets the same pair.
__device__ inline void cluster_max2(double a, double b, double* red, double& ra, double& rb) {
    double pa = a, pb = b;
    block_max2(pa, pb, red);
    if (g_cl.K == 1) {
        ra = pa; rb = pb;
        return;
    }
    if (threadIdx.x == 0) {
        g_cl.slots[2 * g_cl.member] = pa;
        g_cl.slots[2 * g_cl.member + 1] = pb;
    }
    cluster_barrier();
    ra = g_cl.slots[0];
    rb = g_cl.slots[1];
    for (int k = 1; k < g_cl.K; ++k) {
        ra = nanmax(ra, g_cl.slots[2 * k]);
        rb = nanmax(rb, g_cl.slots[2 * k + 1]);
    }
}

// Neighbour indices of (i, j), clamped to the cell itself at the boundary.
struct Nb {
    int idx, w, e, s, n;
    bool hw, he, hs, hn;
    __device__ Nb(int i, int j, int nx, int ny) {
        idx = j * nx + i;
        hw = i > 0; he = i + 1 < nx; hs = j > 0; hn = j + 1 < ny;
        w = hw ? idx - 1 : idx; e = he ? idx + 1 : idx;
        s = hs ? idx - nx : idx; n = hn ? idx + nx : idx;
    }
};

// Layout of the pressure cycle's level arrays (x, b, r, te, tn while the
// pressure V-cycle runs): every row stores its red cells ((i + j) even)
// first and its black cells after them, each in order of i, so that a
// red-black half-sweep reads and writes whole cache lines.  The transport
// cycle keeps the natural row-major order.
__device__ inline int pidx(int i, int j, int nx) { return j * nx + (((i + j) & 1) ? (nx >> 1) : 0) + (i >> 1); }

// Cell (i, j) at storage position s of the colour-split layout (nx = 2^sx).
__device__ inline void pcell(int s, int nx, int sx, int& i, int& j) {
    j = s >> sx;
    const int r = s & (nx - 1), half = nx >> 1;
    const int col = r >= half ? 1 : 0;
    i = 2 * (r - col * half) + ((j + col) & 1);
}

// Neighbour storage positions of (i, j) in the colour-split layout,
// clamped to the cell itself at the boundary.
struct NbS {
    int idx, w, e, s, n;
    bool hw, he, hs, hn;
    __device__ NbS(int i, int j, int nx, int ny) {
        hw = i > 0; he = i + 1 < nx; hs = j > 0; hn = j + 1 < ny;
        idx = pidx(i, j, nx);
        w = hw ? pidx(i - 1, j, nx) : idx; e = he ? pidx(i + 1, j, nx) : idx;
        s = hs ? pidx(i, j - 1, nx) : idx; n = hn ? pidx(i, j + 1, nx) : idx;
    }
};

// ------------------------------------------------------------------ physics (FP64)
__device__ inline double rho_of(const Phys& ph, double c) { return ph.rho0 + (ph.rho1 - ph.rho0) * c; }

// Mass and salt flux through a face, per metre of depth: harmonic K and phi
// on the face (precomputed: K_f / mu, phi_f D), arithmetic rho; donor cell.
struct FaceFlux { double M, F, lam, dif; };

// Wall-clock accumulators of the phases of one step (builds with
// HENRY_PHASE_TIMERS only; wall_clock64 runs at a constant 100 MHz).
// Slots 0..7, 13, 15, 21, 23: phases of the outer iteration (the residual
// passes split into the pass and its reduction or barrier); 8..12, 14 and
// 16..20, 22: parts of the pressure and of the transport V-cycle.
struct PhaseClock {
#ifdef HENRY_PHASE_TIMERS
    uint64_t acc[24];
    uint64_t last;
    __device__ void init() {
        for (int k = 0; k < 24; ++k) acc[k] = 0;
        last = wall_clock64();
    }
    __device__ void tick(int k) {
        const uint64_t t = wall_clock64();
        acc[k] += t - last;
        last = t;
    }
#else
    __device__ void init() {}
    __device__ void tick(int) {}
#endif
};

// ------------------------------------------------------------------ FP64 residual
// Face coefficients between cells a and b: t = K_f / mu and w = phi_f D with
// the harmonic means K_f = 2 Ka Kb / (Ka + Kb) and phi_f = 2 fa fb / (fa + fb),
// both from one division.  At the seawater boundary (half a cell from the
// centre) the coefficients are 2 K / mu and 2 phi D: twice the pair of the
// cell with itself.  With the scale of a cell's residual in the norms, the
// fields kernel stores them; the residual pass may form them again from K and
// phi with the same operations.
struct FacePair { double t, w; };
__device__ inline FacePair face_pair(const Phys& ph, double Ka, double Kb, double fa, double fb) {
    const double sK = (Ka + Kb) * ph.mu, sf = fa + fb;
    const double r = 1.0 / (sK * sf);
    return {2.0 * Ka * Kb * sf * r, 2.0 * fa * fb * ph.D * sK * r};
}
__device__ inline double res_scale(const Phys& ph, double tau, double h, double f) { return tau / (h * h * f * ph.rho0); }

// Rows whose operands the residual pass of the largest grids (kFields) loads
// before it uses any of them: its rows are a chain (the flux through a row's
// south face comes from the row below), and each would wait for its own loads
// from HBM.  32 KL solves of 1024x512, 40 steps, with 1, 2, 4, 8: 752, 730,
// 718, 721 ms.  On the smaller grids, whose operands come from L2 and the
// Infinity Cache, 2 and 4 change nothing and 8 costs 5 %.
constexpr int kResRows = 4;

struct ResNorms { double p, c; };  // scaled max |R^p|, |R^c|

// Mass and salt flux of an interior or boundary face: rf the face density,
// dp the pressure difference (with the gravity term on north faces), ca and
// cb the upstream candidates of the two directions.
__device__ inline FaceFlux face_flux(double rf, double dp, double ca, double cb, double kf, double wf) {
    FaceFlux f;
    f.lam = rf * kf;
    f.dif = rf * wf;
    f.M = rounded_mul(-f.lam, dp);
    f.F = fused(f.M, f.M >= 0.0 ? ca : cb, -rounded_mul(f.dif, cb - ca));
    return f;
}
// Interior face a|b; on a north face Darcy's law with gravity (0,-g) adds
// rho_f g h to the pressure difference.
template <bool kNorth>
__device__ inline FaceFlux face_flux(const Phys& ph, double h, double ra, double rb, double pa, double pb, double ca,
                                     double cb, double kf, double wf) {
    const double rf = 0.5 * (ra + rb);
    return face_flux(rf, kNorth ? fused(rf * ph.g, h, pb - pa) : pb - pa, ca, cb, kf, wf);
}

// Max of |v| and a maximum so far, on the bit patterns: those of the
// non-negative doubles are ordered, and a NaN's is above infinity's.
__device__ inline void abs_max(unsigned long long& m, double v) {
    const unsigned long long b = (unsigned long long)__double_as_longlong(v) & 0x7fffffffffffffffull;
    m = b > m ? b : m;
}

// The rows of one residual pass (see residual_pass): level 0's inner arrays
// are in address space AS0.  Bound by FP64 and address arithmetic on the
// grids whose operands stay in L2 (five hundred cycles a row and wavefront
// before), by HBM on the largest.  Each lane forms the flux through its
// east and its north face; the west one is the lane below's east one (two
// values through DPP shifts), the south one the row below's north one.  Where
// a wavefront ends inside a row, the flux into its first cell and the state
// beyond its last are formed once per 64 rows, lane t those of row t, and
// handed out row by row.  A seawater face is the east face with the boundary
// state's density, concentration and pressure difference; both boundaries'
// terms are formed only by the wavefronts that have one.  Its own function,
// so that its registers are not the solve kernel's.
// kFields: the face coefficients and the norm scale formed from K and phi (5
// FP64 loads per cell instead of 9, and three FP64 divisions), with the same
// operations as the fields kernel's stored ones, so both variants give the
// same bits.  Per outer iteration, with the two residual passes inlined in
// the solve kernel (a division per cell, four fluxes and both boundaries'
// for every cell) and here: 128x64 165 -> 150 us, 64x32 84 -> 80, 4096 solves
// of 16x8 44 -> 38; on clusters the same within 1 %.
template <typename T, int kMode, bool kFields, int AS0>
__device__ __attribute__((noinline)) ResNorms residual_rows(Solve<T>& S) {
    using GP = __attribute__((address_space(1))) double*;
    auto arr = [](double* a) { return as_ptr<1>(uniform(a)); };
    auto at = [](GP a, uint32_t off) { return *(GP)((__attribute__((address_space(1))) char*)a + off); };
    Phys ph;
    ph.rho0 = uniform(S.ph.rho0); ph.rho1 = uniform(S.ph.rho1); ph.mu = uniform(S.ph.mu); ph.g = uniform(S.ph.g);
    ph.D = uniform(S.ph.D); ph.phi0 = 0.0; ph.k0 = 0.0; ph.q_in = 0.0; ph.T = 0.0;
    const int nx = uniform(S.nx), ny = uniform(S.ny), half = nx >> 1;
    const double h = uniform(S.h), tau = uniform(S.tau), drho = ph.rho1 - ph.rho0;
    const double h2t = uniform(h * h / tau), q = uniform(S.q);
    const GP ap = arr(S.p), ac = arr(S.c), acn = arr(S.cn), aphi = arr(S.phi), aK = arr(S.K), atx = arr(S.tx),
             awx = arr(S.wx), aty = arr(S.ty), awy = arr(S.wy), aisc = arr(S.isc);
    const LV<T, AS0> L0(S.lv[0]);
    auto rho = [&](double c) { return fused(drho, c, ph.rho0); };
    const int bs = uniform(ClusterTeam::size()), rk = ClusterTeam::rank();
    const int cw = nx < bs ? nx : bs;  // both powers of two
    const int G = bs / cw;
    const int band = (ny + G - 1) / G;
    const int lane = threadIdx.x & (kWave - 1);
    const int g = rk / cw, ci = rk - g * cw;
    const int j0 = g * band;
    const uint32_t row8 = 8u * (uint32_t)nx;
    unsigned long long mp = 0, mc = 0;
    for (int cx = 0; cx < nx; cx += cw) {
        const int i = cx + ci;
        const bool hw = i > 0, he = i + 1 < nx;
        const bool sea = __any(!he), recharge = __any(!hw);
        // ends of the wavefront inside a row
        const int i0 = uniform(i);
        const bool endw = nx > kWave && i0 > 0, ende = nx > kWave && i0 + kWave < nx;
        // rows below and at the start of the band (clamped into the grid)
        const int jb = j0 < ny ? j0 : ny - 1;
        const int js = jb > 0 ? jb - 1 : jb;
        const uint32_t ob = (uint32_t)(jb * nx + i) * 8u, os = (uint32_t)(js * nx + i) * 8u;
        const double pS = at(ap, os), cS = at(ac, os);
        double pP = at(ap, ob), cP = at(ac, ob);
        double KP = 0.0, fP = 0.0, tyS = 0.0, wyS = 0.0;
        if constexpr (kFields) {
            KP = at(aK, ob);
            fP = at(aphi, ob);
            if (jb > 0) {  // the first row's south face (none at j = 0)
                const FacePair fy = face_pair(ph, at(aK, os), KP, at(aphi, os), fP);
                tyS = fy.t;
                wyS = fy.w;
            }
        } else {
            tyS = at(aty, os);
            wyS = at(awy, os);
        }
        double rP = rho(cP);
        // the flux through the south face of the band's first row
        const FaceFlux f0 = face_flux<true>(ph, h, rho(cS), rP, pS, pP, cS, cP, tyS, wyS);
        double sM = f0.M, sF = f0.F;
        for (int tb = 0; tb < band; tb += kWave) {
            double wM0 = 0.0, wF0 = 0.0, pE0 = 0.0, cE0 = 0.0, KE0 = 0.0, fE0 = 0.0;
            const int je = min(j0 + tb + lane, ny - 1);
            if (endw) {
                const uint32_t o = (uint32_t)(je * nx + i0) * 8u;
                const double p0 = at(ap, o - 8u), p1 = at(ap, o), c0 = at(ac, o - 8u), c1 = at(ac, o);
                const FaceFlux f = face_flux<false>(ph, h, rho(c0), rho(c1), p0, p1, c0, c1, at(atx, o - 8u), at(awx, o - 8u));
                wM0 = f.M;
                wF0 = f.F;
            }
            if (ende) {
                const uint32_t o = (uint32_t)(je * nx + i0 + kWave) * 8u;
                pE0 = at(ap, o);
                cE0 = at(ac, o);
                if constexpr (kFields) {
                    KE0 = at(aK, o);
                    fE0 = at(aphi, o);
                }
            }
            const int tn = min(kWave, band - tb);
            struct RowIn { double pN, cN, cn, a, b, tx, wx, ty, wy; };  // a, b: phi and isc, or K and phi of the row above
            auto load_row = [&](int t) {
                const int j = j0 + tb + t, jc = j < ny ? j : ny - 1;
                const uint32_t o = (uint32_t)(jc * nx + i) * 8u, on = jc + 1 < ny ? o + row8 : o;
                RowIn r;
                r.pN = at(ap, on); r.cN = at(ac, on); r.cn = at(acn, o);
                if constexpr (kFields) {
                    r.a = at(aK, on); r.b = at(aphi, on);
                    r.tx = r.wx = r.ty = r.wy = 0.0;
                } else {
                    r.a = at(aphi, o); r.b = at(aisc, o);
                    r.tx = at(atx, o); r.wx = at(awx, o); r.ty = at(aty, o); r.wy = at(awy, o);
                }
                return r;
            };
            auto row = [&](int t, const RowIn& in) {
                const int j = j0 + tb + t;
                const bool active = j < ny;
                const int jc = active ? j : ny - 1;
                const bool hs = jc > 0, hn = jc + 1 < ny;
                const double pN = in.pN, cN = in.cN, cn = in.cn;
                double KN = 0.0, fN = 0.0, phiP, tx, wx, ty, wy, sc;
                if constexpr (kFields) {
                    KN = in.a;
                    fN = in.b;
                    phiP = fP;
                    const double KE = wave_above(KP, lane_value(KE0, t)), fE = wave_above(fP, lane_value(fE0, t));
                    const FacePair fx = face_pair(ph, KP, he ? KE : KP, fP, he ? fE : fP);
                    const FacePair fy = face_pair(ph, KP, KN, fP, fN);
                    tx = he ? fx.t : 2.0 * fx.t;
                    wx = he ? fx.w : 2.0 * fx.w;
                    ty = hn ? fy.t : 0.0;
                    wy = hn ? fy.w : 0.0;
                    sc = res_scale(ph, tau, h, fP);
                } else {
                    phiP = in.a;
                    tx = in.tx; wx = in.wx; ty = in.ty; wy = in.wy;
                    sc = in.b;
                }
                // east face: interior, or the seawater boundary at half a
                // cell's distance (p_B = -rho1 g y, c_B = 1)
                double cE = wave_above(cP, ende ? lane_value(cE0, t) : 0.0);
                double dE = wave_above(pP, ende ? lane_value(pE0, t) : 0.0) - pP;
                double rE = rho(cE);
                if (sea) {
                    const double y = fused(jc + 0.5, h, -1.0);
                    const double dB = fused(-ph.rho1 * ph.g, y, -pP);
                    cE = he ? cE : 1.0;
                    rE = he ? rE : ph.rho1;
                    dE = he ? dE : dB;
                }
                const FaceFlux fe = face_flux(0.5 * (rP + rE), dE, cP, cE, tx, wx);
                // west face: out of the west neighbour, or the recharge
                double wM = wave_below(fe.M, endw ? lane_value(wM0, t) : 0.0);
                double wF = wave_below(fe.F, endw ? lane_value(wF0, t) : 0.0);
                double ldif = 0.0, lM = 0.0;
                if (recharge) {  // inflow rho0 q h of fresh water (c_B = 0)
                    const double rB = 0.5 * (rP + ph.rho0);
                    ldif = 2.0 * rB * phiP * ph.D;
                    lM = -ph.rho0 * q * h;
                    wM = hw ? wM : -lM;
                    wF = hw ? wF : -rounded_mul(ldif, cP);
                }
                // north face (the top is impermeable)
                const double rN = rho(cN);
                const FaceFlux fn = face_flux<true>(ph, h, rP, rN, pP, pN, cP, cN, ty, wy);
                const double st = h2t * phiP, rn = rho(cn);
                double Rp = fused(rP - rn, st, fe.M);
                double Rc = fused(fused(cP, rP, -rounded_mul(cn, rn)), st, fe.F);
                Rp -= wM;
                Rc -= wF;
                Rp += hn ? fn.M : 0.0;
                Rc += hn ? fn.F : 0.0;
                Rp -= hs ? sM : 0.0;
                Rc -= hs ? sF : 0.0;
                if (active) {
                    if constexpr (kMode != 2) {
                        abs_max(mp, Rp * sc);
                        abs_max(mc, Rc * sc);
                    }
                    if constexpr (kMode == 0) {
                        const int ps = jc * nx + ((i ^ jc) & 1) * half + (i >> 1);  // pidx: colour-split
                        L0.te[ps] = (T)fe.lam;
                        L0.tn[ps] = (T)(hn ? fn.lam : 0.0);
                        L0.b[ps] = (T)(-Rp);
                        L0.x[ps] = (T)0;
                    } else if constexpr (kMode == 1) {
                        const int idx = jc * nx + i;
                        L0.mx[idx] = (T)(he ? fe.M : 0.0);
                        L0.dx[idx] = (T)(he ? fe.dif : 0.0);
                        L0.my[idx] = (T)(hn ? fn.M : 0.0);
                        L0.dy[idx] = (T)(hn ? fn.dif : 0.0);
                        if (!he) { L0.dr[jc] = (T)fe.dif; L0.mr[jc] = (T)fe.M; }
                        if (!hw) { L0.dl[jc] = (T)ldif; L0.ml[jc] = (T)(-lM); }
                        L0.acc[idx] = (T)(st * rn);
                        L0.b[idx] = (T)(-(Rc - cP * Rp));
                        L0.x[idx] = (T)0;
                    } else {
                        S.rout_p[jc * nx + i] = Rp;
                        S.rout_c[jc * nx + i] = Rc;
                    }
                }
                // carry up one row
                if (active) { sM = fn.M; sF = fn.F; }
                pP = pN; cP = cN; rP = rN;
                KP = KN; fP = fN;
            };
            constexpr int kAhead = kFields ? kResRows : 1;
            int t = 0;  // the same trip counts in every lane (shifts)
            for (; t + kAhead <= tn; t += kAhead) {
                RowIn in[kAhead];
#pragma unroll
                for (int r = 0; r < kAhead; ++r) in[r] = load_row(t + r);
#pragma unroll
                for (int r = 0; r < kAhead; ++r) row(t + r, in[r]);
            }
            if (kAhead > 1)
                for (; t < tn; ++t) row(t, load_row(t));
        }
    }
    return {__longlong_as_double((long long)mp), __longlong_as_double((long long)mc)};
}

template <typename T, int kMode, bool kFields>
__device__ inline ResNorms residual_rows(Solve<T>& S) {
    if (kMode != 2 && S.lds_from == 0) return residual_rows<T, kMode, false, 3>(S);
    return residual_rows<T, kMode, kFields, 1>(S);
}

// mode 0: R^p and R^c, pressure coefficients te/tn at level 0, and the
//         scaled max norms (block max).
// mode 1: the salt defect S = R^c - c R^p with the transport coefficients
//         at level 0.
// (residual_rows' mode 2: R^p and R^c into S.rout_p, S.rout_c, the residual
// entry point.)
// Thread layout: lanes along x (cw = min(nx, blockDim) columns), the
// blockDim / cw row groups each march up their own band of rows.  A cell
// takes p and c of the row below from the registers of the previous row and
// its east and west neighbours' values from the adjacent lanes: 9 loads per
// cell.  Grids of at least HENRY_RES_FIELDS_NX columns form the face
// coefficients from K and phi instead (their passes are bound by bandwidth);
// on smaller ones, whose passes wait on load latency, the divisions would
// lengthen the wait.
// The row bands are spread over all threads of the cluster; mode 0 ends
// with the cluster-wide norms, mode 1 with a cluster barrier only.
template <typename T>
__device__ inline void residual_pass(Solve<T>& S, int mode, double* red, double& np_out, double& nc_out,
                                     PhaseClock* pcx = nullptr) {
    constexpr bool kF = HENRY_RES_FIELDS_NX > 0;
    ResNorms m;
    if (kF && S.nx >= HENRY_RES_FIELDS_NX) m = mode == 0 ? residual_rows<T, 0, kF>(S) : residual_rows<T, 1, kF>(S);
    else m = mode == 0 ? residual_rows<T, 0, false>(S) : residual_rows<T, 1, false>(S);
    if (pcx) pcx->tick(mode == 0 ? 23 : 21);
    cluster_max2(m.p, m.c, red, np_out, nc_out);
    __syncthreads();
}

// ------------------------------------------------------------------ coefficient coarsening
// One level of each hierarchy from the level below it (Team loops; the
// caller synchronises the team before the level is read).
template <typename T, class Team, int ASF, int ASC, int KB>
__device__ inline void coarsen_pressure_level_kb(const LV<T, ASF>& F, const LV<T, ASC>& C) {
    const int nc = C.nx * C.ny;
    const int sx = log2i(C.nx);
    const int ts = Team::size();
    for (int k0 = Team::rank(); k0 < nc; k0 += KB * ts) {
        T e0[KB], e1[KB], n0[KB], n1[KB];
#pragma unroll
        for (int u = 0; u < KB; ++u) {
            const int k = k0 + u * ts;
            const int idx = k < nc ? k : 0;
            int I, J;  // colour-split layout on both levels
            pcell(idx, C.nx, sx, I, J);
            e0[u] = F.te[pidx(2 * I + 1, 2 * J, F.nx)];
            e1[u] = F.te[pidx(2 * I + 1, 2 * J + 1, F.nx)];
            n0[u] = F.tn[pidx(2 * I, 2 * J + 1, F.nx)];
            n1[u] = F.tn[pidx(2 * I + 1, 2 * J + 1, F.nx)];
        }
#pragma unroll
        for (int u = 0; u < KB; ++u) {
            const int k = k0 + u * ts;
            if (k < nc) {
                C.te[k] = (T)0.5 * (e0[u] + e1[u]);
                C.tn[k] = (T)0.5 * (n0[u] + n1[u]);
            }
        }
    }
}

template <typename T, class Team, int ASF, int ASC>
__device__ void coarsen_pressure_level(const Level<T>& F0, Level<T>& C0) {
    const LV<T, ASF> F(F0);
    const LV<T, ASC> C(C0);
    if (kTBatch > 1 && ASF == 1 && C.nx * C.ny > Team::size())
        coarsen_pressure_level_kb<T, Team, ASF, ASC, kTBatch>(F, C);
    else coarsen_pressure_level_kb<T, Team, ASF, ASC, 1>(F, C);
}

template <typename T, class Team, int ASF, int ASC, int KB>
__device__ inline void coarsen_transport_level_kb(const LV<T, ASF>& F, const LV<T, ASC>& C) {
    const int nc = C.nx * C.ny;
    const int sx = log2i(C.nx);
    const int ts = Team::size();
    for (int k0 = Team::rank(); k0 < nc; k0 += KB * ts) {
        T a00[KB], a01[KB], a10[KB], a11[KB], mx0[KB], mx1[KB], dx0[KB], dx1[KB], my0[KB], my1[KB], dy0[KB],
            dy1[KB];
#pragma unroll
        for (int u = 0; u < KB; ++u) {
            const int k = k0 + u * ts;
            const int idx = k < nc ? k : 0;
            const int I = idx & (C.nx - 1), J = idx >> sx;
            const int f0 = (2 * J) * F.nx + 2 * I, f1 = f0 + F.nx;
            a00[u] = F.acc[f0]; a01[u] = F.acc[f0 + 1]; a10[u] = F.acc[f1]; a11[u] = F.acc[f1 + 1];
            mx0[u] = F.mx[f0 + 1]; mx1[u] = F.mx[f1 + 1]; dx0[u] = F.dx[f0 + 1]; dx1[u] = F.dx[f1 + 1];
            my0[u] = F.my[f1]; my1[u] = F.my[f1 + 1]; dy0[u] = F.dy[f1]; dy1[u] = F.dy[f1 + 1];
        }
#pragma unroll
        for (int u = 0; u < KB; ++u) {
            const int k = k0 + u * ts;
            if (k < nc) {
                const int I = k & (C.nx - 1), J = k >> sx;
                C.acc[k] = (a00[u] + a01[u]) + (a10[u] + a11[u]);
                // mass fluxes through the two fine faces add; diffusion
                // transmissibilities (length/distance = 1 on every level) average
                C.mx[k] = (I + 1 < C.nx) ? mx0[u] + mx1[u] : (T)0;
                C.dx[k] = (I + 1 < C.nx) ? (T)0.5 * (dx0[u] + dx1[u]) : (T)0;
                C.my[k] = (J + 1 < C.ny) ? my0[u] + my1[u] : (T)0;
                C.dy[k] = (J + 1 < C.ny) ? (T)0.5 * (dy0[u] + dy1[u]) : (T)0;
            }
        }
    }
    for (int J = Team::rank(); J < C.ny; J += ts) {
        C.dl[J] = (T)0.5 * (F.dl[2 * J] + F.dl[2 * J + 1]);
        C.dr[J] = (T)0.5 * (F.dr[2 * J] + F.dr[2 * J + 1]);
        C.mr[J] = F.mr[2 * J] + F.mr[2 * J + 1];
        C.ml[J] = F.ml[2 * J] + F.ml[2 * J + 1];
    }
}

template <typename T, class Team, int ASF, int ASC>
__device__ void coarsen_transport_level(const Level<T>& F0, Level<T>& C0) {
    const LV<T, ASF> F(F0);
    const LV<T, ASC> C(C0);
    if (kTBatch > 1 && ASF == 1 && C.nx * C.ny > Team::size())
        coarsen_transport_level_kb<T, Team, ASF, ASC, kTBatch>(F, C);
    else coarsen_transport_level_kb<T, Team, ASF, ASC, 1>(F, C);
}

template <typename T, bool kTransport, class Team, int ASF, int ASC>
__device__ void coarsen_level(const Level<T>& F, Level<T>& C) {
    if constexpr (kTransport) coarsen_transport_level<T, Team, ASF, ASC>(F, C);
    else coarsen_pressure_level<T, Team, ASF, ASC>(F, C);
}

// Re-discretised coarse coefficients.  The cluster forms levels 1 .. lc
// (from cluster levels; level lc into its global copy when the leader runs
// it in LDS; no barrier after the last, whose next reader, the leader's
// part of the V-cycle, comes after the restriction's barrier).
template <typename T, bool kTransport>
__device__ void coarsen_cluster(Solve<T>& S) {
    for (int l = 1; l <= S.lc; ++l) {
        if (l > 1) ClusterTeam::sync();
        coarsen_level<T, kTransport, ClusterTeam, 1, 1>(S.lv[l - 1], (S.hand && l == S.lc) ? S.hg : S.lv[l]);
    }
}

// Levels `from` .. lds_from, by the leader's workgroup alone; wavefront 0's
// cycle forms the coarser ones itself.
template <typename T, bool kTransport>
__device__ void coarsen_leader(Solve<T>& S, int from) {
    const int lw = S.lds_from, lb = S.lb;
    for (int l = from > 1 ? from : 1; l < S.L && l <= lw; ++l) {
        if (l < lb) coarsen_level<T, kTransport, BlockTeam, 1, 1>(S.lv[l - 1], S.lv[l]);
        else if (l == lb) coarsen_level<T, kTransport, BlockTeam, 1, 3>(S.lv[l - 1], S.lv[l]);
        else coarsen_level<T, kTransport, BlockTeam, 3, 3>(S.lv[l - 1], S.lv[l]);
        __syncthreads();
    }
}

template <typename T, bool kTransport>
__device__ void handoff_in(Solve<T>& S);

// Every level down to lds_from, complete on return (the adjoint's transposed
// solves reuse the coefficients over several cycles; a level handed from the
// cluster to the leader's LDS is copied there first).
template <typename T, bool kTransport>
__device__ void coarsen(Solve<T>& S) {
    coarsen_cluster<T, kTransport>(S);
    if (S.lc > 0) ClusterTeam::sync();
    if (g_cl.member == 0) {
        if (S.hand) {
            handoff_in<T, kTransport>(S);
            __syncthreads();
        }
        coarsen_leader<T, kTransport>(S, S.lc + 1);
    }
    ClusterTeam::sync();
}

template <typename T>
__device__ void coarsen_pressure(Solve<T>& S) { coarsen<T, false>(S); }

template <typename T>
__device__ void coarsen_transport(Solve<T>& S) { coarsen<T, true>(S); }

// ------------------------------------------------------------------ stencils
// Pressure: (A x)_P = diag x_P - sum_nb t_nb x_nb; te of the last column is
// the seawater Dirichlet coefficient (diagonal only); tn of the top row is 0.
// The operations below load every operand from a clamped (always valid)
// index and zero the missing neighbours afterwards: loads under boundary
// branches would each wait for their own round trip.
template <typename T>
struct Stencil { T d, w, e, s, n; };


template <class V, class Q, typename T = typename V::value_type>
__device__ inline Stencil<T> pstencil(const V& v, const Q& q) {
    Stencil<T> st;
    const T te = v.te[q.idx], tw = v.te[q.w], tn = v.tn[q.idx], ts = v.tn[q.s];
    st.e = q.he ? te : (T)0;
    st.w = q.hw ? tw : (T)0;
    st.n = tn;
    st.s = q.hs ? ts : (T)0;
    st.d = te + st.w + st.n + st.s;
    return st;
}

// Transport (non-conservative upwind form): a neighbour couples only
// through inflow across the shared face plus diffusion; the diagonal is
// the stored mass plus the sum of the couplings and the boundary inflow /
// diffusion terms.  mx/my are the mass fluxes leaving (i,j) east/north.
// max(a, 0), 0 for NaN; for float the median with 0 and infinity, one
// instruction (a maximum would first quiet its operand).
__device__ inline double pos(double a) { return a > 0.0 ? a : 0.0; }
__device__ inline float pos(float a) { return __builtin_amdgcn_fmed3f(a, 0.0f, __builtin_inff()); }

template <class V, typename T = typename V::value_type>
__device__ inline Stencil<T> cstencil(const V& v, const Nb& q, int j) {
    Stencil<T> st;
    const T a = v.acc[q.idx];
    const T mE = v.mx[q.idx], dE = v.dx[q.idx], mW = v.mx[q.w], dW = v.dx[q.w];
    const T mN = v.my[q.idx], dN = v.dy[q.idx], mS = v.my[q.s], dS = v.dy[q.s];
    const T bE = pos(-v.mr[j]) + v.dr[j], bW = v.dl[j] + v.ml[j];
    T d = a;
    st.e = q.he ? pos(-mE) + dE : (T)0;
    d += q.he ? st.e : bE;
    st.w = q.hw ? pos(mW) + dW : (T)0;
    d += q.hw ? st.w : bW;
    st.n = q.hn ? pos(-mN) + dN : (T)0;
    d += st.n;
    st.s = q.hs ? pos(mS) + dS : (T)0;
    d += st.s;
    st.d = d;
    return st;
}

// Transpose of the transport operator (adjoint solves): a cell couples to
// a neighbour with that neighbour's coupling to it; the diagonal is the same.
template <class V, typename T = typename V::value_type>
__device__ inline Stencil<T> cstencil_t(const V& v, const Nb& q, int j) {
    Stencil<T> st;
    const T a = v.acc[q.idx];
    const T mE = v.mx[q.idx], dE = v.dx[q.idx], mW = v.mx[q.w], dW = v.dx[q.w];
    const T mN = v.my[q.idx], dN = v.dy[q.idx], mS = v.my[q.s], dS = v.dy[q.s];
    const T bE = pos(-v.mr[j]) + v.dr[j], bW = v.dl[j] + v.ml[j];
    T d = a;
    d += q.he ? pos(-mE) + dE : bE;
    st.e = q.he ? pos(mE) + dE : (T)0;
    d += q.hw ? pos(mW) + dW : bW;
    st.w = q.hw ? pos(-mW) + dW : (T)0;
    d += q.hn ? pos(-mN) + dN : (T)0;
    st.n = q.hn ? pos(mN) + dN : (T)0;
    d += q.hs ? pos(mS) + dS : (T)0;
    st.s = q.hs ? pos(-mS) + dS : (T)0;
    st.d = d;
    return st;
}

template <typename T, bool kTransport, bool kTrans = false, class V, class Q>
__device__ inline Stencil<T> stencil(const V& v, const Q& q, int j) {
    if constexpr (kTransport) {
        if constexpr (kTrans) return cstencil_t(v, q, j);
        else return cstencil(v, q, j);
    } else {
        return pstencil(v, q);
    }
}

// ------------------------------------------------------------------ grid transfer
// Prolongation: bilinear with constant extrapolation at the boundary,
// x_f += P x_c.  Restriction is its exact transpose (full weighting with
// weights (1,3,3,1)/4 per direction, boundary weights folded in).
// kSplit: both levels in the colour-split layout (pressure cycle).
template <typename T, class Team, int ASC, int ASF, bool kSplit, int KB>
__device__ inline void prolong_add_kb(const LV<T, ASC>& C, const LV<T, ASF>& F) {
    const int n = F.nx * F.ny;
    const int sx = log2i(F.nx);
    const int ts = Team::size();
    auto cat = [&](int I, int J) { return kSplit ? pidx(I, J, C.nx) : J * C.nx + I; };
    for (int k0 = Team::rank(); k0 < n; k0 += KB * ts) {
        T v[KB], xf[KB];
#pragma unroll
        for (int u = 0; u < KB; ++u) {
            const int k = k0 + u * ts;
            const int idx = k < n ? k : 0;
            int i, j;
            if constexpr (kSplit) pcell(idx, F.nx, sx, i, j);
            else { i = idx & (F.nx - 1); j = idx >> sx; }
            const int I = i >> 1, J = j >> 1;
            const int In = (i & 1) ? min(I + 1, C.nx - 1) : max(I - 1, 0);
            const int Jn = (j & 1) ? min(J + 1, C.ny - 1) : max(J - 1, 0);
            v[u] = (T)0.5625 * C.x[cat(I, J)] + (T)0.1875 * (C.x[cat(In, J)] + C.x[cat(I, Jn)]) +
                   (T)0.0625 * C.x[cat(In, Jn)];
            xf[u] = F.x[idx];
        }
#pragma unroll
        for (int u = 0; u < KB; ++u)
            if (k0 + u * ts < n) F.x[k0 + u * ts] = xf[u] + v[u];
    }
}

// Prolongation: bilinear with constant extrapolation at the boundary,
// x_f += P x_c.  Restriction is its exact transpose (full weighting with
// weights (1,3,3,1)/4 per direction, boundary weights folded in).
// kSplit: both levels in the colour-split layout (pressure cycle).
template <typename T, class Team = BlockTeam, int ASC = 0, int ASF = 0, bool kSplit = false>
__device__ void prolong_add(const Level<T>& C0, Level<T>& F0) {
    const LV<T, ASC> C(C0);
    const LV<T, ASF> F(F0);
    if (kTBatch > 1 && ASF == 1 && F.nx * F.ny > Team::size())
        prolong_add_kb<T, Team, ASC, ASF, kSplit, kTBatch>(C, F);
    else prolong_add_kb<T, Team, ASC, ASF, kSplit, 1>(C, F);
}

// 1D restriction weight of fine index I2 = 2I - 1 + a (a = 0..3) for coarse
// index I of n: (1,3,3,1)/4, with the boundary ghost weight folded in.
__device__ inline float rweight(int I, int n, int a) {
    float w = (a == 0 || a == 3) ? 0.25f : 0.75f;
    if (a == 1 && I == 0) w += 0.25f;
    if (a == 2 && I == n - 1) w += 0.25f;
    return w;
}

template <typename T, class Team, int ASF, int ASC, bool kSplit, int KB>
__device__ inline void restrict_residual_kb(const LV<T, ASF>& F, const LV<T, ASC>& C) {
    const int n = C.nx * C.ny;
    const int sx = log2i(C.nx);
    const int ts = Team::size();
    // fine cells whose residual the level residual left out (zero): black
    // cells (aq + bq odd) in the pressure cycle, odd rows (bq even) in the
    // transport cycle
    auto live = [](int aq, int bq) { return kSplit ? ((aq + bq) & 1) == 0 : (bq & 1) == 1; };
    for (int k0 = Team::rank(); k0 < n; k0 += KB * ts) {
        T rv[KB][4][4];
        int cI[KB], cJ[KB];
#pragma unroll
        for (int u = 0; u < KB; ++u) {
            const int k = k0 + u * ts;
            const int idx = k < n ? k : 0;
            int I, J;
            if constexpr (kSplit) pcell(idx, C.nx, sx, I, J);
            else { I = idx & (C.nx - 1); J = idx >> sx; }
            cI[u] = I; cJ[u] = J;
            // fine rows / columns outside the level get weight 0 (their load
            // is clamped to a valid cell)
#pragma unroll
            for (int bq = 0; bq < 4; ++bq) {
                const int jf = min(max(2 * J - 1 + bq, 0), F.ny - 1);
#pragma unroll
                for (int aq = 0; aq < 4; ++aq) {
                    const int ifn = min(max(2 * I - 1 + aq, 0), F.nx - 1);
                    rv[u][bq][aq] = live(aq, bq) ? F.r[kSplit ? pidx(ifn, jf, F.nx) : jf * F.nx + ifn] : (T)0;
                }
            }
        }
#pragma unroll
        for (int u = 0; u < KB; ++u) {
            const int I = cI[u], J = cJ[u];
            // terms outside the level are selected away, not weighted by
            // zero: their clamped load may land on a cell whose residual was
            // never written
            T s = (T)0;
#pragma unroll
            for (int bq = 0; bq < 4; ++bq) {
                const int jf = 2 * J - 1 + bq;
                const bool jin = jf >= 0 && jf < F.ny;
                T row = (T)0;
#pragma unroll
                for (int aq = 0; aq < 4; ++aq) {
                    const int ifn = 2 * I - 1 + aq;
                    const bool iin = ifn >= 0 && ifn < F.nx;
                    row += iin ? (T)rweight(I, C.nx, aq) * rv[u][bq][aq] : (T)0;
                }
                s += jin ? (T)rweight(J, C.ny, bq) * row : (T)0;
            }
            const int k = k0 + u * ts;
            if (k < n) {
                C.b[k] = s;
                C.x[k] = (T)0;
            }
        }
    }
}

// Value of the lane below / above in the wavefront (0 at its ends).
template <typename T> __device__ inline T wave_below(T v) { return dpp_row<0x138>(v); }  // wave_shr:1
template <typename T> __device__ inline T wave_above(T v) { return dpp_row<0x130>(v); }  // wave_shl:1

// The same for fine rows of 64 to 256 cells, two coarse cells 2m and 2m + 1 per
// thread: the residuals of their six fine columns are one vector load per
// fine row and a value of the neighbouring lane each side (the row's lanes lie
// in one wavefront), where a cell by itself gathered eight values from
// clamped indices.  Per iteration, level 0 down: 128x64 in one workgroup 11.5
// and 12.4 -> 10.2 and 11.6 us (pressure, transport), 256x128 on 8 workgroups
// 11.9 and 10.1 -> 10.9 and 9.2.
// Coarse rows J0 .. J1 - 1 by `size` threads.
template <typename T, int ASF, int ASC, bool kSplit>
__device__ inline void restrict_pairs(typename AsPtr<T, ASF>::type r, int nx, int ny, const LV<T, ASC>& C, int J0, int J1,
                                      int rank, int size) {
    using V2 = T __attribute__((ext_vector_type(2)));
    const int hc = C.nx >> 1, n = hc * (J1 - J0), sh = log2i(hc);
    for (int k = rank; k < n; k += size) {  // whole rows
        const int J = J0 + (k >> sh), m = k & (hc - 1);
        T s[2] = {};
#pragma unroll
        for (int bq = 0; bq < 4; ++bq) {
            if (!kSplit && !(bq & 1)) continue;  // odd fine rows: zero
            const int jf = 2 * J - 1 + bq;
            const bool jin = jf >= 0 && jf < ny;
            const int jc = min(max(jf, 0), ny - 1);
            T f[6] = {};  // fine columns 4m - 1 .. 4m + 4
            if constexpr (kSplit) {
                const V2 a = *(typename AsPtr<V2, ASF>::type)(r + jc * nx + 2 * m);
                if (bq & 1) { f[1] = a[0]; f[3] = a[1]; f[5] = wave_above((T)a[0]); }
                else { f[0] = wave_below((T)a[1]); f[2] = a[0]; f[4] = a[1]; }
            } else {
                const Vec4<T> a = *(typename AsPtr<Vec4<T>, ASF>::type)(r + jc * nx + 4 * m);
                f[0] = wave_below((T)a[3]); f[5] = wave_above((T)a[0]);
#pragma unroll
                for (int q = 0; q < 4; ++q) f[1 + q] = a[q];
            }
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int I = 2 * m + u;
                T row = (T)0;
#pragma unroll
                for (int aq = 0; aq < 4; ++aq) {
                    if (kSplit && ((aq + bq) & 1)) continue;  // black cells: zero
                    const int ifn = 2 * I - 1 + aq;
                    row += ifn >= 0 && ifn < nx ? rounded_mul((T)rweight(I, C.nx, aq), f[2 * u + aq]) : (T)0;
                }
                s[u] += jin ? rounded_mul((T)rweight(J, C.ny, bq), row) : (T)0;
            }
        }
        if constexpr (kSplit) {
            const int at = J * C.nx + m, o = (J & 1) * hc;  // cell 2m is red in the even rows
            C.b[at + o] = s[0];
            C.b[at + hc - o] = s[1];
            C.x[at + o] = (T)0;
            C.x[at + hc - o] = (T)0;
        } else {
            *(typename AsPtr<V2, ASC>::type)(C.b + J * C.nx + 2 * m) = V2{s[0], s[1]};
            *(typename AsPtr<V2, ASC>::type)(C.x + J * C.nx + 2 * m) = V2{};
        }
    }
}

template <typename T, class Team = BlockTeam, int ASF = 0, int ASC = 0, bool kSplit = false>
__device__ void restrict_residual(const Level<T>& F0, Level<T>& C0) {
    const LV<T, ASF> F(F0);
    const LV<T, ASC> C(C0);
    if (F.nx >= 64 && F.nx <= 256)
        return restrict_pairs<T, ASF, ASC, kSplit>(F.r, F.nx, F.ny, C, 0, C.ny, Team::rank(), Team::size());
    if (kTBatch > 1 && ASF == 1 && C.nx * C.ny > Team::size())
        restrict_residual_kb<T, Team, ASF, ASC, kSplit, kTBatch>(F, C);
    else restrict_residual_kb<T, Team, ASF, ASC, kSplit, 1>(F, C);
}

// r = b - A x on one level after the pre-smoothing (operands of kRBatch
// cells gathered first), on the cells smoothed first only: the cells the
// smoother updated last (black cells of the red-black sweep, odd rows of the
// zebra x-line sweep) satisfy their equations with the current neighbours,
// so their residual is zero to rounding, and the restriction skips them.
// Pressure: red cells, the first half of each row of the colour-split
// layout; transport: the even rows.
constexpr int kRBatch = 2;
template <typename T, bool kTransport, bool kTrans, class Team, int AS, int KB>
__device__ inline void level_residual_kb(const LV<T, AS>& v) {
    const int half = v.nx >> 1;
    const int n = kTransport ? v.nx * ((v.ny + 1) >> 1) : half * v.ny;  // live cells
    const int ts = Team::size();
    const int sx = log2i(v.nx);
    for (int k0 = Team::rank(); k0 < n; k0 += KB * ts) {
        T res[KB];
        int at[KB];
#pragma unroll
        for (int u = 0; u < KB; ++u) {
            const int k = k0 + u * ts;
            const int kk = k < n ? k : 0;
            int i, j, idx;
            if constexpr (kTransport) {
                i = kk & (v.nx - 1); j = 2 * (kk >> sx);
                idx = j * v.nx + i;
            } else {
                j = kk >> (sx - 1);
                const int kr = kk & (half - 1);
                i = 2 * kr + (j & 1);
                idx = j * v.nx + kr;
            }
            at[u] = idx;
            using Q = typename std::conditional<kTransport, Nb, NbS>::type;
            const Q q(i, j, v.nx, v.ny);
            const Stencil<T> st = stencil<T, kTransport, kTrans>(v, q, j);
            const T xP = v.x[idx], xW = v.x[q.w], xE = v.x[q.e], xS = v.x[q.s], xN = v.x[q.n];
            const T bP = v.b[idx];
            // missing neighbours have zero couplings
            T ax = st.d * xP;
            ax -= st.w * xW;
            ax -= st.e * xE;
            ax -= st.s * xS;
            ax -= st.n * xN;
            res[u] = bP - ax;
        }
#pragma unroll
        for (int u = 0; u < KB; ++u)
            if (k0 + u * ts < n) v.r[at[u]] = res[u];
    }
}

// One cell per thread when one pass of the team covers the live cells.
template <typename T, bool kTransport, bool kTrans = false, class Team = BlockTeam, int AS = 0>
__device__ void level_residual(Level<T>& v0) {
    const LV<T, AS> v(v0);
    const int n = kTransport ? v.nx * ((v.ny + 1) >> 1) : (v.nx >> 1) * v.ny;
    if (n <= Team::size()) level_residual_kb<T, kTransport, kTrans, Team, AS, 1>(v);
    else level_residual_kb<T, kTransport, kTrans, Team, AS, kRBatch>(v);
}

// ------------------------------------------------------------------ smoothers
// Red-black Gauss-Seidel (pressure): colour (i + j) & 1.  Cells of one
// colour are independent; each thread gathers the operands of kBatch cells
// before it writes any of them, so their loads are in flight together.
constexpr int kBatch = 4;

// One half-sweep (colour col) with KB cells gathered per thread.
template <typename T, class Team, int AS, int KB>
__device__ inline void rbgs_colour(const LV<T, AS>& v, int col) {
    const int nx = v.nx, ny = v.ny;
    const int half = nx >> 1;  // nx is even on every level
    const int sh = log2i(half);
    const int m = half * ny;
    const auto te = v.te;
    const auto tn = v.tn;
    const auto b = v.b;
    const auto x = v.x;
    for (int k0 = Team::rank(); k0 < m; k0 += KB * Team::size()) {
        T num[KB], den[KB];
        int at[KB];
#pragma unroll
        for (int u = 0; u < KB; ++u) {
            const int k = k0 + u * Team::size();
            const int kk = k < m ? k : 0;
            const int j = kk >> sh;
            const int i = 2 * (kk & (half - 1)) + ((j + col) & 1);
            const NbS q(i, j, nx, ny);  // q.idx = j nx + col half + (kk mod half)
            at[u] = k < m ? q.idx : -1;
            const T tE = te[q.idx], tWl = te[q.w], tN = tn[q.idx], tSl = tn[q.s];
            const T xW = x[q.w], xE = x[q.e], xS = x[q.s], xN = x[q.n];
            const T bP = b[q.idx];
            const T tW = q.hw ? tWl : (T)0, tS = q.hs ? tSl : (T)0;
            const T tEc = q.he ? tE : (T)0;  // the seawater coefficient is diagonal only
            T a = bP;
            a += tW * xW;
            a += tEc * xE;
            a += tS * xS;
            a += tN * xN;
            num[u] = a;
            den[u] = tE + tW + tN + tS;
        }
#pragma unroll
        for (int u = 0; u < KB; ++u)
            if (at[u] >= 0) x[at[u]] = qdiv(num[u], den[u]);
    }
}

// A colour that one pass of the team covers takes one cell per thread
// (the coarse levels: a fixed batch would issue the loads and arithmetic of
// kBatch cells per lane for one useful cell or none); larger ones take
// kBatch.  The cells and their arithmetic are the same either way.
template <typename T, class Team = BlockTeam, int AS = 0>
__device__ void rbgs(Level<T>& v0, int sweeps) {
    const LV<T, AS> v(v0);
    const bool one = (v.nx >> 1) * v.ny <= Team::size();
    for (int s = 0; s < sweeps; ++s)
        for (int col = 0; col < 2; ++col) {
            if (one) rbgs_colour<T, Team, AS, 1>(v, col);
            else rbgs_colour<T, Team, AS, kBatch>(v, col);
            Team::sync();
        }
}

// Segmented line solve.  Every line of one colour is split over T lanes of
// one wavefront (T a power of two dividing 64), lane t owning the m = len/T
// consecutive rows t*m .. t*m+m-1 of the line.  The lane's last row is an
// interface unknown iota_t; its m-1 interior rows are eliminated locally
// (Thomas, three right-hand sides: the line rhs and the unit couplings to
// iota_{t-1} and iota_t), which leaves a tridiagonal system in the T
// interface unknowns.  That reduced system is solved by parallel cyclic
// reduction across the T lanes with wavefront shuffles, then every lane
// back-substitutes its interior rows.  All coefficients live in registers;
// a colour of lines is one block-wide phase.
// MS = rows per lane (a power of two, 2 to 16, chosen by line_sweep); line
// lengths are powers of two, so TL = len/MS <= 64 lanes per line.
// Each instantiation is its own function, so the register budget of the
// long-line variants does not weigh on the short ones.
template <typename T, bool kXLine, bool kTrans, int MS, class Team, int AS>
__device__ __attribute__((noinline)) void line_sweep_m(Level<T>& v0, int col) {
    const LV<T, AS> v(v0);
    const int len = kXLine ? v.nx : v.ny;
    const int other = kXLine ? v.ny : v.nx;
    const int nlines = (other - col + 1) >> 1;
    const int m = MS;                   // rows per lane
    const int TL = len / m;             // lanes per line
    const int stl = log2i(TL);
    const int lane = threadIdx.x & (kWave - 1);
    const int t = lane & (TL - 1);
    const int need = nlines * TL;
    for (int base = 0; base < need; base += Team::size()) {
        const int g = base + Team::rank();
        const int li = g >> stl;
        const bool active = li < nlines;
        const int fixed = col + 2 * (active ? li : 0);
        // w (the response to iota_t) is zero above row m-2 before the back
        // substitution, so afterwards w[q] = w[m-2] * prod_{k=q}^{m-3} (-cp[k]):
        // it is carried as a running product instead of an array
        T cp[MS], y[MS], u[MS];
        T wlast = (T)0;
        T ar = (T)0, br = (T)1, cr = (T)0, dr = (T)0;
        // forward elimination of the interior rows, interface row kept aside
#pragma unroll
        for (int q = 0; q < MS; ++q) {
            if (q < m) {
                const int k = t * m + q;
                const int i = kXLine ? k : fixed, j = kXLine ? fixed : k;
                const Nb nb(i, j, v.nx, v.ny);
                const Stencil<T> st = stencil<T, true, kTrans>(v, nb, j);
                T rhs = v.b[nb.idx];
                T a, c;
                // off-line neighbours; missing ones have zero couplings
                if (kXLine) {
                    const T xS = v.x[nb.s], xN = v.x[nb.n];
                    rhs += st.s * xS;
                    rhs += st.n * xN;
                    a = -st.w; c = -st.e;
                } else {
                    const T xW = v.x[nb.w], xE = v.x[nb.e];
                    rhs += st.w * xW;
                    rhs += st.e * xE;
                    a = -st.s; c = -st.n;
                }
                if (q < m - 1) {
                    const T den = (q > 0) ? st.d - a * cp[q > 0 ? q - 1 : 0] : st.d;
                    const T inv = qdiv((T)1, den);
                    const T yprev = (q > 0) ? y[q > 0 ? q - 1 : 0] : (T)0;
                    const T uprev = (q > 0) ? u[q > 0 ? q - 1 : 0] : (T)0;
                    cp[q] = c * inv;
                    y[q] = (rhs - a * yprev) * inv;
                    u[q] = ((q == 0 ? -a : (T)0) - a * uprev) * inv;
                    if (q == m - 2) wlast = (-c - a * (T)0) * inv;
                } else {
                    ar = a; br = st.d; cr = c; dr = rhs;
                }
            }
        }
        // back substitution of the interior rows (coupling to iota_t: the
        // running product wrun, w[q] = 0 - cp[q] w[q + 1])
        T wrun = wlast;
#pragma unroll
        for (int q = MS - 2; q >= 0; --q) {
            if (q < m - 2) {
                y[q] -= cp[q] * y[q + 1];
                u[q] -= cp[q] * u[q + 1];
                wrun = (T)0 - cp[q] * wrun;
            }
        }
        // interior rows next to the interfaces
        T yL = (T)0, uL = (T)1, wL = (T)0;  // row before the interface (m == 1: iota_{t-1} itself)
        T yF = (T)0, uF = (T)0, wF = (T)1;  // first row of this lane (m == 1: iota_t itself)
#pragma unroll
        for (int q = 0; q < MS; ++q) {
            if (q == m - 2) { yL = y[q]; uL = u[q]; wL = wlast; }
        }
        if (m >= 2) { yF = y[0]; uF = u[0]; wF = m >= 2 ? wrun : (T)1; }
        // first row of the next lane of the same line
        const bool last = (t == TL - 1);
        const int src = last ? lane : lane + 1;
        T yN = __shfl(yF, src, kWave), uN = __shfl(uF, src, kWave), wN = __shfl(wF, src, kWave);
        if (last) { yN = (T)0; uN = (T)0; wN = (T)0; cr = (T)0; }
        T A = ar * uL;
        T B = br + ar * wL + cr * uN;
        T C = cr * wN;
        T D = dr - ar * yL - cr * yN;
        // parallel cyclic reduction over the TL interface equations
        for (int sft = 1; sft < TL; sft <<= 1) {
            const bool hasL = t >= sft, hasR = t + sft < TL;
            const int l = hasL ? lane - sft : lane, r = hasR ? lane + sft : lane;
            const T Al = __shfl(A, l, kWave), Bl = __shfl(B, l, kWave), Cl = __shfl(C, l, kWave),
                    Dl = __shfl(D, l, kWave);
            const T Ar = __shfl(A, r, kWave), Br = __shfl(B, r, kWave), Cr = __shfl(C, r, kWave),
                    Dr = __shfl(D, r, kWave);
            T nA = (T)0, nB = B, nC = (T)0, nD = D;
            if (hasL) {
                const T k1 = qdiv(A, Bl);
                nA = -Al * k1;
                nB -= Cl * k1;
                nD -= Dl * k1;
            }
            if (hasR) {
                const T k2 = qdiv(C, Br);
                nC = -Cr * k2;
                nB -= Ar * k2;
                nD -= Dr * k2;
            }
            A = nA; B = nB; C = nC; D = nD;
        }
        const T iota = qdiv(D, B);
        const T left0 = __shfl(iota, t > 0 ? lane - 1 : lane, kWave);
        const T left = t > 0 ? left0 : (T)0;
        if (active) {
            // rows from the bottom up, rebuilding w[q] as in the back substitution
            T wq = wlast;
#pragma unroll
            for (int q = MS - 1; q >= 0; --q) {
                if (q < m) {
                    const int k = t * m + q;
                    const int i = kXLine ? k : fixed, j = kXLine ? fixed : k;
                    if (q < m - 2) wq = (T)0 - cp[q] * wq;
                    v.x[j * v.nx + i] = (q < m - 1) ? y[q] + u[q] * left + wq * iota : iota;
                }
            }
        }
    }
    Team::sync();
}

// x-lines of 512 and 1024 cells on the cluster levels (one wavefront per
// line, MS = 8 or 16 rows per lane).  line_sweep_m gathers a lane's MS
// consecutive cells, so each of its load instructions touches 32 cache lines
// at 8 bytes each, and the lines are gone from L1 and L2 before the lane
// comes back for the rest of them.  Here the wavefront forms each row's
// coefficients (the same stencil arithmetic) from coalesced loads, 64
// consecutive cells per instruction, into its own LDS buffer, and each lane
// reads its segment back from there for the same elimination (results are
// bitwise those of line_sweep_m).  A 1024-cell row is staged in two halves
// of 512 (lanes 0-31 eliminate the first, 32-63 the second).  The buffers
// overlay the LDS levels, which are dead while the cluster runs its levels
// in the forward solve: every cycle's leader rebuilds them (coarse_coeffs)
// after the cluster's downward leg and is done with them before its upward
// leg.  The adjoint's transposed cycles keep them from cycle to cycle, so
// its kernel turns the staging off (g_cl.stage_waves = 0).  Padding of one
// element per segment keeps the segment reads free of bank conflicts (lane
// stride MS + 1).
constexpr int kStageCells = 512;
constexpr int kStageElems = kStageCells + kStageCells / 8;  // one pad per segment of >= 8 cells
template <typename T>
__host__ __device__ constexpr int64_t line_stage_bytes_per_wave() { return 4 * (int64_t)kStageElems * (int64_t)sizeof(T); }

template <typename T, bool kTrans, int MS>
__device__ __attribute__((noinline)) void line_sweep_x_staged(Level<T>& v0, int col) {
    static_assert(MS == 8 || MS == 16, "staged x-lines are 512 or 1024 cells");
    constexpr int NH = kWave * MS / kStageCells;  // halves of a row
    const LV<T, 1> v(v0);
    const int nlines = (v.ny - col + 1) >> 1;
    const int lane = threadIdx.x & (kWave - 1);
    T* buf = reinterpret_cast<T*>(g_cl.stage) + (int64_t)(threadIdx.x / kWave) * 4 * kStageElems;
    auto As = as_ptr<3>(buf);
    auto Cs = as_ptr<3>(buf + kStageElems);
    auto Ds = as_ptr<3>(buf + 2 * kStageElems);
    auto Rs = as_ptr<3>(buf + 3 * kStageElems);
    const int waves = ClusterTeam::size() / kWave, wrank = ClusterTeam::rank() / kWave;
    const int t = lane;
    for (int l0 = 0; l0 < nlines; l0 += waves) {  // the same trip count in every lane
        const int li = l0 + wrank;
        const bool active = li < nlines;
        const int j = col + 2 * (active ? li : 0);
        T cp[MS], y[MS], u[MS];
        T wlast = (T)0;
        T ar = (T)0, br = (T)1, cr = (T)0, dr = (T)0;
        for (int hh = 0; hh < NH; ++hh) {
            // coefficients of cells hh * 512 + r * 64 + lane, coalesced
#pragma unroll 2
            for (int r = 0; r < kStageCells / kWave; ++r) {
                const int kl = r * kWave + lane;
                const Nb nb(hh * kStageCells + kl, j, v.nx, v.ny);
                const Stencil<T> st = stencil<T, true, kTrans>(v, nb, j);
                T rhs = v.b[nb.idx];
                const T xS = v.x[nb.s], xN = v.x[nb.n];
                rhs += st.s * xS;
                rhs += st.n * xN;
                const int si = kl + kl / MS;
                As[si] = -st.w;
                Cs[si] = -st.e;
                Ds[si] = st.d;
                Rs[si] = rhs;
            }
            WaveTeam::sync();
            // forward elimination of the lanes whose segment lies in this half
            if (t * MS / kStageCells == hh) {
                const int s0 = (t * MS - hh * kStageCells) / MS * (MS + 1);
#pragma unroll
                for (int q = 0; q < MS; ++q) {
                    const T a = As[s0 + q], c = Cs[s0 + q], d = Ds[s0 + q], rhs = Rs[s0 + q];
                    if (q < MS - 1) {
                        const T den = (q > 0) ? d - a * cp[q > 0 ? q - 1 : 0] : d;
                        const T inv = qdiv((T)1, den);
                        const T yprev = (q > 0) ? y[q > 0 ? q - 1 : 0] : (T)0;
                        const T uprev = (q > 0) ? u[q > 0 ? q - 1 : 0] : (T)0;
                        cp[q] = c * inv;
                        y[q] = (rhs - a * yprev) * inv;
                        u[q] = ((q == 0 ? -a : (T)0) - a * uprev) * inv;
                        if (q == MS - 2) wlast = (-c - a * (T)0) * inv;
                    } else {
                        ar = a; br = d; cr = c; dr = rhs;
                    }
                }
            }
            WaveTeam::sync();  // the buffer is refilled by the next half or line
        }
        // back substitution of the interior rows (coupling to iota_t: the
        // running product wrun, w[q] = 0 - cp[q] w[q + 1])
        T wrun = wlast;
#pragma unroll
        for (int q = MS - 2; q >= 0; --q) {
            if (q < MS - 2) {
                y[q] -= cp[q] * y[q + 1];
                u[q] -= cp[q] * u[q + 1];
                wrun = (T)0 - cp[q] * wrun;
            }
        }
        const T yL = y[MS - 2], uL = u[MS - 2], wL = wlast;
        const T yF = y[0], uF = u[0], wF = wrun;
        // first row of the next lane of the same line
        const bool last = (t == kWave - 1);
        const int src = last ? lane : lane + 1;
        T yN = __shfl(yF, src, kWave), uN = __shfl(uF, src, kWave), wN = __shfl(wF, src, kWave);
        if (last) { yN = (T)0; uN = (T)0; wN = (T)0; cr = (T)0; }
        T A = ar * uL;
        T B = br + ar * wL + cr * uN;
        T C = cr * wN;
        T D = dr - ar * yL - cr * yN;
        // parallel cyclic reduction over the 64 interface equations
        for (int sft = 1; sft < kWave; sft <<= 1) {
            const bool hasL = t >= sft, hasR = t + sft < kWave;
            const int l = hasL ? lane - sft : lane, r = hasR ? lane + sft : lane;
            const T Al = __shfl(A, l, kWave), Bl = __shfl(B, l, kWave), Cl = __shfl(C, l, kWave),
                    Dl = __shfl(D, l, kWave);
            const T Ar = __shfl(A, r, kWave), Br = __shfl(B, r, kWave), Cr = __shfl(C, r, kWave),
                    Dr = __shfl(D, r, kWave);
            T nA = (T)0, nB = B, nC = (T)0, nD = D;
            if (hasL) {
                const T k1 = qdiv(A, Bl);
                nA = -Al * k1;
                nB -= Cl * k1;
                nD -= Dl * k1;
            }
            if (hasR) {
                const T k2 = qdiv(C, Br);
                nC = -Cr * k2;
                nB -= Ar * k2;
                nD -= Dr * k2;
            }
            A = nA; B = nB; C = nC; D = nD;
        }
        const T iota = qdiv(D, B);
        const T left0 = __shfl(iota, t > 0 ? lane - 1 : lane, kWave);
        const T left = t > 0 ? left0 : (T)0;
        if (active) {
            // rows from the bottom up, rebuilding w[q] as in the back substitution
            T wq = wlast;
#pragma unroll
            for (int q = MS - 1; q >= 0; --q) {
                if (q < MS - 2) wq = (T)0 - cp[q] * wq;
                v.x[j * v.nx + t * MS + q] = (q < MS - 1) ? y[q] + u[q] * left + wq * iota : iota;
            }
        }
    }
    ClusterTeam::sync();
}

// x-lines of 64, 128 and 256 cells: line_sweep_m's solve with four rows per
// lane, TL = 16, 32 or 64 lanes per line.  With one load per cell and array
// (12 of them), a wavefront's loads lay 16 bytes apart and each took the
// texture unit 16 clocks for a quarter of the bytes it moved; that, not the
// elimination, was the phase.  Here a lane loads its four cells of an array
// as one vector (the flux into the segment's first cell comes from the lane
// before), 10 loads instead of 48: an outer iteration of 128x64 (one
// workgroup) 190 -> 172 us, its level 0 transport legs 22.2 -> 15.7 and 14.9
// -> 8.8 us.
//
// Lane l of a line's rows of 16 holds segment t = (l mod 16) R + l / 16,
// R = TL / 16: a shift by a multiple of R segments is then a shift within
// rows of 16 lanes, a DPP operand, and only the log2(R) shortest shifts of
// the cyclic reduction go through the LDS crossbar.  A reduction step's two
// reciprocals are one, formed before the shift.
template <int TL>
struct LineLanes {
    static constexpr int R = TL / 16;
    __device__ static inline int segment(int lane) { return (lane & 15) * R + ((lane >> 4) & (R - 1)); }
    __device__ static inline int line(int lane) { return (lane >> 4) / R; }
    __device__ static inline int lane_of(int lane, int t) { return (lane & ~(TL - 1)) | ((t & (R - 1)) << 4) | (t / R); }
    // value of segment t - kS (below), t + kS (above) of the same line; any
    // finite value of this wavefront's where there is none
    template <int kS, typename T>
    __device__ static inline T below(T v, int lane) {
        if constexpr (kS % R == 0) return lane_below<kS / R>(v);
        else { const int t = segment(lane); return __shfl(v, t >= kS ? lane_of(lane, t - kS) : lane, kWave); }
    }
    template <int kS, typename T>
    __device__ static inline T above(T v, int lane) {
        if constexpr (kS % R == 0) return lane_above<kS / R>(v);
        else { const int t = segment(lane); return __shfl(v, t + kS < TL ? lane_of(lane, t + kS) : lane, kWave); }
    }
};

// One step of the cyclic reduction over a line's segments and those after
// it (segments without a partner have a zero coupling to it).
template <int kS, int TL, typename T>
__device__ inline void line_pcr(T& A, T& B, T& C, T& D, int lane) {
    if constexpr (kS < TL) {
        using LL = LineLanes<TL>;
        T k1, k2;
        if constexpr (sizeof(T) == 4) {
            const T rB = __builtin_amdgcn_rcpf(B);
            k1 = A * LL::template below<kS>(rB, lane);
            k2 = C * LL::template above<kS>(rB, lane);
        } else {
            const int t = LL::segment(lane);
            const T Bl = LL::template below<kS>(B, lane), Br = LL::template above<kS>(B, lane);
            k1 = t >= kS ? A / Bl : (T)0;
            k2 = t + kS < TL ? C / Br : (T)0;
        }
        const T Al = LL::template below<kS>(A, lane), Cl = LL::template below<kS>(C, lane),
                Dl = LL::template below<kS>(D, lane);
        const T Ar = LL::template above<kS>(A, lane), Cr = LL::template above<kS>(C, lane),
                Dr = LL::template above<kS>(D, lane);
        T nB = B, nD = D;
        nB -= Cl * k1;
        nD -= Dl * k1;
        nB -= Ar * k2;
        nD -= Dr * k2;
        A = -Al * k1;
        C = -Cr * k2;
        B = nB;
        D = nD;
        line_pcr<2 * kS, TL>(A, B, C, D, lane);
    }
}

// One segment of a line: four cells' couplings, diagonals, right-hand sides
// and solution.
template <typename T>
struct Segment {
    int j, k0;     // row, first cell's index
    bool active;   // the line exists
    T w[4], e[4], s[4], n[4], d[4], b[4];
    Vec4<T> x;
};

// What the rows beside a line hold: zero, v.x, or (first colour after the
// coarse levels) v.x and the correction prolonged from level c.
struct BesideZero {
    template <class L, typename T>
    __device__ inline void operator()(const L&, int, int, int, int, T&, T&) const {}
};
struct BesideX {
    template <typename T, int AS>
    __device__ inline void operator()(const LV<T, AS>& v, int, int, int ks, int kn, Vec4<T>& xS, Vec4<T>& xN) const {
        xS = *(typename AsPtr<Vec4<T>, AS>::type)(v.x + ks);
        xN = *(typename AsPtr<Vec4<T>, AS>::type)(v.x + kn);
    }
};
template <typename T, int TL, int ASC>
struct BesideProlonged {
    const LV<T, ASC>& c;
    // a line of an even row 2J: the rows beside it are the upper ones of
    // coarse rows J - 1 and J
    template <int AS>
    __device__ inline void operator()(const LV<T, AS>& v, int lane, int j, int ks, int kn, Vec4<T>& xS, Vec4<T>& xN) const {
        using LL = LineLanes<TL>;
        using V2 = T __attribute__((ext_vector_type(2)));
        constexpr int nc = 2 * TL;
        const int t = LL::segment(lane), J = j >> 1;
        T cc[3][4];  // coarse cells 2t - 1 .. 2t + 2 of rows J - 1, J, J + 1
#pragma unroll
        for (int r = 0; r < 3; ++r) {
            const int Jr = min(max(J + r - 1, 0), c.ny - 1);
            const V2 o = *(typename AsPtr<V2, ASC>::type)(c.x + Jr * nc + 2 * t);
            const T w = LL::template below<1>((T)o[1], lane), e = LL::template above<1>((T)o[0], lane);
            cc[r][0] = t > 0 ? w : (T)o[0];
            cc[r][1] = o[0];
            cc[r][2] = o[1];
            cc[r][3] = t < TL - 1 ? e : (T)o[1];
        }
        BesideX{}(v, lane, j, ks, kn, xS, xN);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int m = 1 + (q >> 1), w = (q & 1) ? m + 1 : m - 1;
            xS[q] = xS[q] + prolonged(cc[0][m], cc[0][w], cc[1][m], cc[1][w]);
            xN[q] = xN[q] + prolonged(cc[1][m], cc[1][w], cc[2][m], cc[2][w]);
        }
    }
};

// Solves this wavefront's lines of colour col from line (base + rank) / TL
// on.
template <typename T, bool kTrans, int TL, class Team, int AS, class Beside>
__device__ inline void line_solve_x(const LV<T, AS>& v, int col, int base, Segment<T>& g, const Beside& beside) {
    constexpr bool kZero = std::is_same<Beside, BesideZero>::value;
    using LL = LineLanes<TL>;
    using V4 = Vec4<T>;
    constexpr int MS = 4, nx = MS * TL;
    const int ny = v.ny;
    const int nlines = (ny - col + 1) >> 1;
    const int lane = threadIdx.x & (kWave - 1);
    const int t = LL::segment(lane);
    const bool first = t == 0, last = t == TL - 1;
    auto load4 = [](typename LV<T, AS>::P p) { return *(typename AsPtr<V4, AS>::type)p; };
    const int li = (base + Team::rank() - lane) / TL + LL::line(lane);
    g.active = li < nlines;
    const int j = col + 2 * (g.active ? li : 0);
    const bool hs = j > 0, hn = j + 1 < ny;
    const int k0 = j * nx + MS * t, ks = hs ? k0 - nx : k0, kn = hn ? k0 + nx : k0;
    g.j = j;
    g.k0 = k0;
    const V4 acc = load4(v.acc + k0), mE = load4(v.mx + k0), dE = load4(v.dx + k0), mN = load4(v.my + k0),
             dN = load4(v.dy + k0), mS = load4(v.my + ks), dS = load4(v.dy + ks), bq = load4(v.b + k0);
    V4 xS = {}, xN = {};
    beside(v, lane, j, ks, kn, xS, xN);
    const T bE = pos(-v.mr[j]) + v.dr[j], bW = v.dl[j] + v.ml[j];
    const T mW0 = LL::template below<1>((T)mE[3], lane), dW0 = LL::template below<1>((T)dE[3], lane);
    T cp[MS], y[MS], u[MS];
    T wlast = (T)0;
    T ar = (T)0, br = (T)1, cr = (T)0, dr = (T)0;
#pragma unroll
    for (int q = 0; q < MS; ++q) {
        const bool he = q < MS - 1 || !last, hw = q > 0 || !first;
        const T mW = q == 0 ? mW0 : mE[q > 0 ? q - 1 : 0], dW = q == 0 ? dW0 : dE[q > 0 ? q - 1 : 0];
        // cstencil's / cstencil_t's couplings and diagonal
        const T ce = pos(-mE[q]) + dE[q], cw = pos(mW) + dW, cn = pos(-mN[q]) + dN[q], cs = pos(mS[q]) + dS[q];
        T d = acc[q];
        d += he ? ce : bE;
        d += hw ? cw : bW;
        d += hn ? cn : (T)0;
        d += hs ? cs : (T)0;
        const T e = he ? (kTrans ? pos(mE[q]) + dE[q] : ce) : (T)0, w = hw ? (kTrans ? pos(-mW) + dW : cw) : (T)0,
                n = hn ? (kTrans ? pos(mN[q]) + dN[q] : cn) : (T)0,
                s = hs ? (kTrans ? pos(-mS[q]) + dS[q] : cs) : (T)0;
        g.w[q] = w; g.e[q] = e; g.s[q] = s; g.n[q] = n; g.d[q] = d; g.b[q] = bq[q];
        T rhs = bq[q];
        if constexpr (!kZero) {
            rhs += s * xS[q];
            rhs += n * xN[q];
        }
        const T a = -w, c = -e;
        if (q < MS - 1) {
            const T den = (q > 0) ? d - a * cp[q > 0 ? q - 1 : 0] : d;
            const T inv = qdiv((T)1, den);
            const T yprev = (q > 0) ? y[q > 0 ? q - 1 : 0] : (T)0;
            const T uprev = (q > 0) ? u[q > 0 ? q - 1 : 0] : (T)0;
            cp[q] = c * inv;
            y[q] = (rhs - a * yprev) * inv;
            u[q] = ((q == 0 ? -a : (T)0) - a * uprev) * inv;
            if (q == MS - 2) wlast = (-c - a * (T)0) * inv;
        } else {
            ar = a; br = d; cr = c; dr = rhs;
        }
    }
    // back substitution of the interior rows (coupling to iota_t: the
    // running product wrun, w[q] = 0 - cp[q] w[q + 1])
    T wrun = wlast;
#pragma unroll
    for (int q = MS - 3; q >= 0; --q) {
        y[q] -= cp[q] * y[q + 1];
        u[q] -= cp[q] * u[q + 1];
        wrun = (T)0 - cp[q] * wrun;
    }
    // interface equation of the segment's last row (the last segment's
    // coupling to a next one, cr, is zero)
    const T yN = LL::template above<1>(y[0], lane), uN = LL::template above<1>(u[0], lane),
            wN = LL::template above<1>(wrun, lane);
    T A = ar * u[MS - 2];
    T B = br + ar * wlast + cr * uN;
    T C = cr * wN;
    T D = dr - ar * y[MS - 2] - cr * yN;
    line_pcr<1, TL>(A, B, C, D, lane);
    const T iota = qdiv(D, B);
    const T left = LL::template below<1>(iota, lane);  // the first segment's coupling to it, u, is zero
    g.x[MS - 1] = iota;
    T wq = wlast;
#pragma unroll
    for (int q = MS - 2; q >= 0; --q) {
        if (q < MS - 2) wq = (T)0 - cp[q] * wq;
        g.x[q] = y[q] + u[q] * left + wq * iota;
    }
    if (g.active) *(typename AsPtr<V4, AS>::type)(v.x + k0) = g.x;
}

template <typename T, bool kTrans, int TL, class Team, int AS>
__device__ __attribute__((noinline)) void line_sweep_x(Level<T>& v0, int col) {
    const LV<T, AS> v(v0);
    const int need = ((v.ny - col + 1) >> 1) * TL;
    for (int base = 0; base < need; base += Team::size()) {
        Segment<T> g;
        line_solve_x<T, kTrans, TL, Team, AS>(v, col, base, g, BesideX{});
    }
    Team::sync();
}

// Prolongation from level c and the post-smoothing.  A line replaces its row,
// so only the odd rows, as the first colour's neighbours, are ever read with
// the correction: the even rows' lines add it to what they load, and a pass
// over the level with its barrier is gone.  Per iteration, level 0 from the
// prolongation on: 64x32 9.2 -> 4.9 us, 128x64 in one workgroup 10.6 -> 7.0,
// 256x128 on 8 workgroups 11.9 -> 8.1 (level 1 14.3 -> 11.1).
template <typename T, bool kTrans, int TL, class Team, int ASC, int AS>
__device__ __attribute__((noinline)) void line_up(const Level<T>& c0, Level<T>& v0) {
    const LV<T, ASC> c(c0);
    const LV<T, AS> v(v0);
    for (int base = 0; base < (v.ny >> 1) * TL; base += Team::size()) {
        Segment<T> g;
        line_solve_x<T, kTrans, TL, Team, AS>(v, 0, base, g, BesideProlonged<T, TL, ASC>{c});
    }
    Team::sync();
    for (int base = 0; base < (v.ny >> 1) * TL; base += Team::size()) {
        Segment<T> g;
        line_solve_x<T, kTrans, TL, Team, AS>(v, 1, base, g, BesideX{});
    }
    Team::sync();
}

// Pre-smoothing from x = 0 (even rows, then odd rows) and the even rows'
// residual, for levels whose even rows are one pass of the team: the even
// rows' couplings, diagonals and solution stay in registers for the residual
// instead of being loaded and formed again, and the first colour reads no x.
// Per iteration, level 0 down to the restriction: 64x32 11.9 -> 6.2 us, 128x64
// in one workgroup 17.2 -> 12.4, 256x128 on 8 workgroups 13.8 -> 10.2.
template <typename T, bool kTrans, int TL, class Team, int AS>
__device__ __attribute__((noinline)) void line_down(Level<T>& v0) {
    using LL = LineLanes<TL>;
    using V4 = Vec4<T>;
    constexpr int nx = 4 * TL;
    const LV<T, AS> v(v0);
    const int lane = threadIdx.x & (kWave - 1);
    Segment<T> g;
    line_solve_x<T, kTrans, TL, Team, AS>(v, 0, 0, g, BesideZero{});
    Team::sync();
    {
        Segment<T> o;
        line_solve_x<T, kTrans, TL, Team, AS>(v, 1, 0, o, BesideX{});
    }
    Team::sync();
    const int ks = g.j > 0 ? g.k0 - nx : g.k0, kn = g.j + 1 < v.ny ? g.k0 + nx : g.k0;
    const V4 xS = *(typename AsPtr<V4, AS>::type)(v.x + ks), xN = *(typename AsPtr<V4, AS>::type)(v.x + kn);
    const T xW = LL::template below<1>((T)g.x[3], lane), xE = LL::template above<1>((T)g.x[0], lane);
    V4 r;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        T ax = fused(g.d[q], (T)g.x[q], -rounded_mul(g.w[q], q == 0 ? xW : (T)g.x[q > 0 ? q - 1 : 0]));
        ax -= g.e[q] * (q == 3 ? xE : (T)g.x[q < 3 ? q + 1 : 3]);
        ax -= g.s[q] * xS[q];
        ax -= g.n[q] * xN[q];
        r[q] = g.b[q] - ax;
    }
    if (g.active) *(typename AsPtr<V4, AS>::type)(v.r + g.k0) = r;
    Team::sync();
}

// One colour of lines.  x-lines of 64 to 256 cells (FP64: 128) take line_sweep_x's
// four rows per lane, longer ones the fewest that fit a line in one wavefront.
// y-lines and x-lines of fewer than 64 cells are asked for by
// henry_level_smooth alone (y-lines of 64 to 256 rows with four rows per lane,
// so that a wavefront holds two or more neighbouring columns and each of its
// loads touches half as many, or fewer, cache lines as with one column).
template <typename T, bool kXLine, bool kTrans = false, class Team = BlockTeam, int AS = 0>
__device__ void line_sweep(Level<T>& v, int col) {
    const int len = kXLine ? v.nx : v.ny;  // 2 .. 1024, a power of two
    if constexpr (kXLine && AS == 1 && std::is_same<Team, ClusterTeam>::value) {
        if (len >= 512 && g_cl.K > 1 && (int)(blockDim.x / kWave) <= g_cl.stage_waves) {
            if (len == 512) line_sweep_x_staged<T, kTrans, 8>(v, col);
            else line_sweep_x_staged<T, kTrans, 16>(v, col);
            return;
        }
    }
    if constexpr (kXLine) {
        if (len < 64) line_sweep_m<T, kXLine, kTrans, 2, Team, AS>(v, col);
        else if (len == 64) line_sweep_x<T, kTrans, 16, Team, AS>(v, col);
        else if (len == 128) line_sweep_x<T, kTrans, 32, Team, AS>(v, col);
        else if (len == 256) {  // FP64, 60 half-sweeps of 256x128: 2516 us with line_sweep_x, 1858 here
            if constexpr (sizeof(T) == 4) line_sweep_x<T, kTrans, 64, Team, AS>(v, col);
            else line_sweep_m<T, kXLine, kTrans, 4, Team, AS>(v, col);
        }
        else if (len == 512) line_sweep_m<T, kXLine, kTrans, 8, Team, AS>(v, col);
        else line_sweep_m<T, kXLine, kTrans, 16, Team, AS>(v, col);
    } else {
        if (len < 64) line_sweep_m<T, kXLine, kTrans, 2, Team, AS>(v, col);
        else if (len <= 256) line_sweep_m<T, kXLine, kTrans, 4, Team, AS>(v, col);
        else line_sweep_m<T, kXLine, kTrans, 8, Team, AS>(v, col);
    }
}

// One zebra sweep in one direction: x-lines (even rows, then odd rows) or
// y-lines (even columns, then odd columns; a one-row level has only its
// x-line).
template <typename T, bool kTrans = false, class Team = BlockTeam, int AS = 0>
__device__ void line_smooth(Level<T>& v, bool ylines) {
    if (ylines && v.ny > 1) {
        line_sweep<T, false, kTrans, Team, AS>(v, 0);
        line_sweep<T, false, kTrans, Team, AS>(v, 1);
    } else {
        line_sweep<T, true, kTrans, Team, AS>(v, 0);
        line_sweep<T, true, kTrans, Team, AS>(v, 1);
    }
}

#include "henry_wave.hpp"

// ------------------------------------------------------------------ levels in registers
// A level of which every thread of the team holds C consecutive cells of each
// colour (one pass: C = 1, 2 or 4) is smoothed from registers: couplings,
// reciprocal diagonals, b and x of the thread's cells are loaded or formed
// once per leg instead of once per half-sweep, the west and east neighbours
// are the thread's own other colour and one value of the next lane, and a
// half-sweep loads only the rows above and below: 48 bytes for four cells
// instead of 160, and a fifth of the instructions.  The arithmetic per cell
// is rbgs's and level_residual's.  Pressure legs of level 0 per iteration,
// down and up: 128x64 in one workgroup 17.5 and 13.0 -> 11.4 and 4.7 us,
// 64x32 9.6 and 7.6 -> 5.7 and 2.9, 256x128 on 8 workgroups 15.3 and 13.6 ->
// 11.9 and 9.4.
// A row's lanes lie in one wavefront: nx <= 128 C.
template <int C, typename T> struct VecC { using type = T __attribute__((ext_vector_type(C))); };
template <typename T> struct VecC<1, T> { using type = T; };

template <int C, typename T, int AS>
__device__ inline void load_c(typename AsPtr<T, AS>::type p, T (&o)[C]) {
    if constexpr (C == 1) o[0] = *p;
    else {
        const auto v = *(typename AsPtr<typename VecC<C, T>::type, AS>::type)p;
#pragma unroll
        for (int q = 0; q < C; ++q) o[q] = v[q];
    }
}
template <int C, typename T, int AS>
__device__ inline void store_c(typename AsPtr<T, AS>::type p, const T (&x)[C]) {
    if constexpr (C == 1) *p = x[0];
    else {
        typename VecC<C, T>::type v;
#pragma unroll
        for (int q = 0; q < C; ++q) v[q] = x[q];
        *(typename AsPtr<typename VecC<C, T>::type, AS>::type)p = v;
    }
}

// The thread's cells are those of positions kr .. kr + C - 1 of row j, if
// active; x is the level's (XS = AS), or that of rows lo .. hi - 1 in LDS.
template <typename T, class Team, int AS, int XS, int C>
struct RbOwn {
    using XP = typename AsPtr<T, XS>::type;
    const LV<T, AS>& v;
    XP lds;
    int lo, hi;
    int nx, half, j, kr, o;  // o: column 2 (kr + q) + o of the red cells, 1 - o of the black ones
    bool active;
    T cw[2][C], ce[2][C], cs[2][C], cn[2][C], cd[2][C], dred[C], b[2][C], x[2][C];

    // cells k .. k + C - 1 of each colour, counted from row lo
    __device__ inline RbOwn(const LV<T, AS>& lv, XP lds, int lo, int hi, int k) : v(lv), lds(lds), lo(lo), hi(hi) {
        nx = v.nx; half = nx >> 1;
        active = k < half * (hi - lo);
        const int kk = active ? k : 0;
        j = lo + (kk >> log2i(half));
        kr = kk & (half - 1);
        o = j & 1;
        const bool hs = j > 0;
        T te[2][C], tn[2][C], ts[2][C];
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            load_c<C, T, AS>(v.te + j * nx + c * half + kr, te[c]);
            load_c<C, T, AS>(v.tn + j * nx + c * half + kr, tn[c]);
            load_c<C, T, AS>(v.tn + (hs ? (j - 1) * nx + (1 - c) * half + kr : j * nx + kr), ts[c]);
            load_c<C, T, AS>(v.b + j * nx + c * half + kr, b[c]);
        }
        // the colour whose cells lie in the even columns of the row has its
        // first west neighbour in the lane before
        const T edge = wave_below(o ? te[0][C - 1] : te[1][C - 1]);
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            const int oc = o ^ c;
#pragma unroll
            for (int q = 0; q < C; ++q) {
                const bool hw = kr + q + oc > 0, he = !(oc == 1 && kr + q == half - 1);
                const T tW = oc ? te[1 - c][q] : (q > 0 ? te[1 - c][q > 0 ? q - 1 : 0] : edge);
                cw[c][q] = hw ? tW : (T)0;
                ce[c][q] = he ? te[c][q] : (T)0;  // the seawater coefficient is diagonal only
                cn[c][q] = tn[c][q];
                cs[c][q] = hs ? ts[c][q] : (T)0;
                const T d = te[c][q] + cw[c][q] + cn[c][q] + cs[c][q];
                if (c == 0) dred[q] = d;
                cd[c][q] = diag_prep(d);
            }
        }
    }
    __device__ inline XP x_row(int jr) const {
        if constexpr (XS == AS) return v.x + jr * nx;
        else return lds + (jr - lo) * nx;
    }
    __device__ inline void put(int c) const {
        if (active) store_c<C, T, XS>(x_row(j) + c * half + kr, x[c]);
    }
    // the neighbours of the cells of colour c: win[q], win[q + 1] west and east
    __device__ inline void neighbours(int c, T (&win)[C + 1], T (&xs)[C], T (&xn)[C]) const {
        const int oc = o ^ c;
        load_c<C, T, XS>(x_row(j > (XS == AS ? 0 : lo) ? j - 1 : j) + (1 - c) * half + kr, xs);
        load_c<C, T, XS>(x_row(j + 1 < (XS == AS ? v.ny : hi) ? j + 1 : j) + (1 - c) * half + kr, xn);
        const T below = wave_below(x[1 - c][C - 1]), above = wave_above(x[1 - c][0]);
        win[0] = oc ? x[1 - c][0] : below;
#pragma unroll
        for (int q = 1; q < C; ++q) win[q] = oc ? x[1 - c][q] : x[1 - c][q - 1];
        win[C] = oc ? above : x[1 - c][C - 1];
    }
    __device__ inline void update(int c) {
        T win[C + 1], xs[C], xn[C];
        neighbours(c, win, xs, xn);
#pragma unroll
        for (int q = 0; q < C; ++q) {
            T a = b[c][q];
            a += cw[c][q] * win[q];
            a += ce[c][q] * win[q + 1];
            a += cs[c][q] * xs[q];
            a += cn[c][q] * xn[q];
            x[c][q] = diag_div(a, cd[c][q]);
        }
    }
    __device__ inline void half_sweep(int c) {
        update(c);
        put(c);
        Team::sync();
    }
    // the black cells of v.x with the correction prolonged from level c
    template <int ASC>
    __device__ inline void prolong_black(const LV<T, ASC>& c) {
        const int hc = half >> 1;
        // coarse cells kr - 1 .. kr + C of the rows J and Jn
        const int J = j >> 1, Jn = (j & 1) ? min(J + 1, c.ny - 1) : max(J - 1, 0);
        T cj[C + 2], cn[C + 2];
#pragma unroll
        for (int q = 0; q < C + 2; ++q) {
            const int I = min(max(kr - 1 + q, 0), half - 1);
            cj[q] = c.x[J * half + ((I + J) & 1) * hc + (I >> 1)];
            cn[q] = c.x[Jn * half + ((I + Jn) & 1) * hc + (I >> 1)];
        }
        load_c<C, T, AS>(v.x + j * nx + half + kr, x[1]);
#pragma unroll
        for (int q = 0; q < C; ++q)
            x[1][q] = x[1][q] + (o ? prolonged(cj[q + 1], cj[q], cn[q + 1], cn[q])
                                   : prolonged(cj[q + 1], cj[q + 2], cn[q + 1], cn[q + 2]));
    }
};

// Prolongation from level c and the post-smoothing (two sweeps).  A half-sweep
// replaces the cells of its colour, so only the black cells, as the first
// red half-sweep's neighbours, are ever read with the correction.  (Each
// thread adding it to the black cells it loads, without the pass that stores
// them, was no faster: 64x32 3.3 -> 3.7 us a leg, 128x64 in one workgroup
// 5.2 -> 7.9.)
template <typename T, class Team, int ASC, int AS, int C>
__device__ __attribute__((noinline)) void rb_up(const Level<T>& c0, const Level<T>& v0) {
    const LV<T, ASC> c(c0);
    const LV<T, AS> v(v0);
    RbOwn<T, Team, AS, AS, C> R(v, v.x, 0, v.ny, Team::rank() * C);
    R.prolong_black(c);
    R.put(1);
    Team::sync();
    for (int s = 0; s < 2; ++s) {
        R.half_sweep(0);
        R.half_sweep(1);
    }
}

// ------------------------------------------------------------------ strips of a level
// A pressure level of a cluster, by strips of ny / K rows: each member smooths
// its strip with a halo of rows beside it, x in its LDS, so that the
// half-sweeps of a leg meet at the workgroup's barrier and only its end at the
// cluster's (a half-sweep took 1.8 us with the cluster's barrier and loads
// from L2, against 0.6 in a workgroup).  A halo cell is formed from the same
// values by the same operations as its owner forms it, as far as it is used:
// a half-sweep of n that are still to come needs n rows beside the strip.
// The LDS is that of the levels the leader runs (g_cl.stage), idle meanwhile.
// Per iteration, legs down and up: 256x128 on 8 workgroups 10.9 and 9.3 -> 5.4
// and 6.3 us, its level 1 7.4 and 7.6 -> 3.4 and 3.7, 128x64 on 4 9.7 and 9.2
// -> 3.9 and 5.2, on 2 9.6 and 9.3 -> 5.3 and 6.8.
constexpr int kStripDown = 5, kStripUp = 4;  // halo rows

struct Strip { int j0, j1, lo, hi; };  // own rows, rows held
__device__ inline Strip strip_of(int ny, int halo) {
    const int rows = ny / g_cl.K, j0 = g_cl.member * rows;
    return {j0, j0 + rows, max(j0 - halo, 0), min(j0 + rows + halo, ny)};
}

// Cells of one colour per thread (0: the level is not taken by strips): four,
// or eight where a strip and its halo need them (128x64 on 2 workgroups and
// 256x128 on 8).  Levels of 512 columns and more do not fit in one pass.
template <typename T, class Team, int AS>
__device__ inline int strip_cells(int nx, int ny) {
    if constexpr (!std::is_same<Team, ClusterTeam>::value || AS != 1) return 0;
    const int K = g_cl.K;
    if (K == 1 || nx < 64 || nx > 256 || ny < 2 * K) return 0;
    const int rows = ny / K + 2 * kStripDown;
    if (rows * nx * (int)sizeof(T) > g_cl.stage_bytes) return 0;
    const int m = rows * (nx >> 1), ts = (int)blockDim.x;
    return m <= 4 * ts ? 4 : kStripWide && sizeof(T) == 4 && m <= 8 * ts ? 8 : 0;
}

// Pre-smoothing (two sweeps from x = 0) and the red cells' residual; a strip
// (XS = 3 of a level in global memory) restricts it too.
template <typename T, class Team, int AS, int XS, int C>
__device__ __attribute__((noinline)) void rb_down(const Level<T>& c0, const Level<T>& v0) {
    constexpr bool kStrip = XS != AS;
    const LV<T, AS> v(v0);
    Strip s = {0, 0, 0, v.ny};
    typename AsPtr<T, XS>::type lds = {};
    if constexpr (kStrip) {
        s = strip_of(v.ny, kStripDown);
        lds = as_ptr<3>(reinterpret_cast<T*>(g_cl.stage));
    }
    RbOwn<T, Team, AS, XS, C> R(v, lds, s.lo, s.hi, Team::rank() * C);
#pragma unroll
    for (int q = 0; q < C; ++q) R.x[0][q] = diag_div(R.b[0][q], R.cd[0][q]);
    R.put(0);
    Team::sync();
    R.half_sweep(1);
    R.half_sweep(0);
    R.half_sweep(1);
    T win[C + 1], xs[C], xn[C], r[C];
    R.neighbours(0, win, xs, xn);
#pragma unroll
    for (int q = 0; q < C; ++q) {
        T ax = fused(R.dred[q], R.x[0][q], -rounded_mul(R.cw[0][q], win[q]));
        ax -= R.ce[0][q] * win[q + 1];
        ax -= R.cs[0][q] * xs[q];
        ax -= R.cn[0][q] * xn[q];
        r[q] = R.b[0][q] - ax;
    }
    if constexpr (!kStrip) {
        if (R.active) store_c<C, T, AS>(v.r + R.j * R.nx + R.kr, r);
        Team::sync();
    } else {
        if (R.active) {
            store_c<C, T, XS>(R.x_row(R.j) + R.kr, r);  // the red cells' x is not read again
            if (R.j >= s.j0 && R.j < s.j1) {
                store_c<C, T, AS>(v.x + R.j * R.nx + R.kr, R.x[0]);
                store_c<C, T, AS>(v.x + R.j * R.nx + R.half + R.kr, R.x[1]);
            }
        }
        Team::sync();
        restrict_pairs<T, XS, AS, true>(lds - s.lo * v.nx, v.nx, v.ny, LV<T, AS>(c0), s.j0 >> 1, s.j1 >> 1, Team::rank(),
                                        Team::size());
    }
}

// Other members read the level's x in their halo meanwhile: the result goes
// to r's array, and the two change places.
template <typename T, int C>
__device__ __attribute__((noinline)) void strip_up(const Level<T>& c0, Level<T>& v0) {
    const LV<T, 1> v(v0), c(c0);
    const Strip s = strip_of(v.ny, kStripUp);
    const auto x = as_ptr<3>(reinterpret_cast<T*>(g_cl.stage));
    RbOwn<T, BlockTeam, 1, 3, C> R(v, x, s.lo, s.hi, (int)threadIdx.x * C);
    R.prolong_black(c);
    R.put(1);
    __syncthreads();
    R.half_sweep(0);
    R.half_sweep(1);
    R.half_sweep(0);
    R.update(1);
    if (R.active && R.j >= s.j0 && R.j < s.j1) {
        store_c<C, T, 1>(v.r + R.j * R.nx + R.kr, R.x[0]);
        store_c<C, T, 1>(v.r + R.j * R.nx + R.half + R.kr, R.x[1]);
    }
    if (threadIdx.x == 0) {
        T* const t = v0.x;
        v0.x = v0.r;
        v0.r = t;
    }
    ClusterTeam::sync();
}

// Cells of one colour per thread when the level takes one such pass of the
// team (0: it does not, or its rows cross wavefronts).
template <class Team>
__device__ inline int rb_cells(int nx, int ny) {
    const int m = (nx >> 1) * ny, ts = Team::size();
    const int c = m <= ts ? 1 : m <= 2 * ts ? 2 : m <= 4 * ts ? 4 : 0;
    return nx <= 128 * c ? c : 0;
}

// ------------------------------------------------------------------ V-cycles
// Downward leg on level l (address space AS; level l+1 in ASN): smooth,
// residual, restriction to level l+1.
template <typename T, bool kTransport, bool kTrans, class Team, int AS, int ASN>
__device__ void vdown(Solve<T>& S, int l) {
    Level<T>& v = S.lv[l];
    Level<T>& c = (S.hand && l + 1 == S.lc) ? S.hg : S.lv[l + 1];
    if constexpr (kTransport) {
        const bool once = ((v.ny + 1) >> 1) * (v.nx >> 2) <= Team::size();
        if (once && v.nx == 64) line_down<T, kTrans, 16, Team, AS>(v);
        else if (once && v.nx == 128) line_down<T, kTrans, 32, Team, AS>(v);
        else if (once && v.nx == 256) line_down<T, kTrans, 64, Team, AS>(v);
        else {
            line_smooth<T, kTrans, Team, AS>(v, false);
            level_residual<T, kTransport, kTrans, Team, AS>(v);
            Team::sync();
        }
    } else {
        switch (strip_cells<T, Team, AS>(v.nx, v.ny)) {
            case 4: rb_down<T, BlockTeam, 1, 3, 4>(c, v); Team::sync(); return;
            case 8: if constexpr (kStripWide && sizeof(T) == 4) { rb_down<T, BlockTeam, 1, 3, 8>(c, v); Team::sync(); return; }
        }
        switch (rb_cells<Team>(v.nx, v.ny)) {
            case 1: rb_down<T, Team, AS, AS, 1>(c, v); break;
            case 2: rb_down<T, Team, AS, AS, 2>(c, v); break;
            case 4: rb_down<T, Team, AS, AS, 4>(c, v); break;
            default:
                rbgs<T, Team, AS>(v, 2);
                level_residual<T, kTransport, kTrans, Team, AS>(v);
                Team::sync();
        }
    }
    restrict_residual<T, Team, AS, ASN, !kTransport>(v, c);
    Team::sync();
}

// Upward leg on level l: prolongation from level l+1, smooth.  The
// transport post-smoothing takes x-lines here and y-lines on the levels of
// 512 cells or fewer (henry_wave.hpp): in global memory a y-line sweep costs
// about three x-line sweeps (the rows of a column are a cache line apart),
// and the outer iteration counts stay the same (1.69 per step on 256x128/800
// either way).
template <typename T, bool kTransport, bool kTrans, class Team, int AS, int ASN>
__device__ void vup(Solve<T>& S, int l) {
    Level<T>& v = S.lv[l];
    const Level<T>& c = (S.hand && l + 1 == S.lc) ? S.hg : S.lv[l + 1];
    if constexpr (kTransport) {
        switch (v.nx) {
            case 64: return line_up<T, kTrans, 16, Team, ASN, AS>(c, v);
            case 128: return line_up<T, kTrans, 32, Team, ASN, AS>(c, v);
            case 256: return line_up<T, kTrans, 64, Team, ASN, AS>(c, v);
        }
    } else {
        switch (strip_cells<T, Team, AS>(v.nx, v.ny)) {
            case 4: return strip_up<T, 4>(c, v);
            case 8: if constexpr (kStripWide && sizeof(T) == 4) return strip_up<T, 8>(c, v);
        }
        switch (rb_cells<Team>(v.nx, v.ny)) {
            case 1: return rb_up<T, Team, ASN, AS, 1>(c, v);
            case 2: return rb_up<T, Team, ASN, AS, 2>(c, v);
            case 4: return rb_up<T, Team, ASN, AS, 4>(c, v);
        }
    }
    prolong_add<T, Team, ASN, AS, !kTransport>(c, v);
    Team::sync();
    if constexpr (kTransport) line_smooth<T, kTrans, Team, AS>(v, false);
    else rbgs<T, Team, AS>(v, 2);
}

// Level lc between the cluster and the leader's LDS (S.hand): the leader
// copies what the cluster formed in the level's global copy (coefficients,
// restricted right-hand side) into LDS before its part of the cycle, and
// the correction x back afterwards.  Four cells per load and all arrays'
// loads before the first store: one round trip to L2 for a 64x32 level and
// 512 threads, four with a cell per load.  (The level has 512 cells at least
// and its arrays follow one another from an aligned start.)  Per outer iteration:
// 128x64 at K = 2 123.0 -> 116.0 us, at K = 4 107.0 -> 100.7, 256x128 at K = 8
// 180 -> 173.
template <int kArrays, typename T>
__device__ inline void copy_in(const LV<T, 1>& G, const LV<T, 3>& D, typename AsPtr<T, 1>::type const (&from)[kArrays],
                               typename AsPtr<T, 3>::type const (&to)[kArrays]) {
    using V4 = Vec4<T>;
    const int n4 = (G.nx * G.ny) >> 2;
    for (int i = threadIdx.x; i < n4; i += blockDim.x) {
        V4 a[kArrays];
#pragma unroll
        for (int k = 0; k < kArrays; ++k) a[k] = ((typename AsPtr<V4, 1>::type)from[k])[i];
#pragma unroll
        for (int k = 0; k < kArrays; ++k) ((typename AsPtr<V4, 3>::type)to[k])[i] = a[k];
        ((typename AsPtr<V4, 3>::type)D.x)[i] = (V4){};
    }
}

template <typename T, bool kTransport>
__device__ void handoff_in(Solve<T>& S) {
    const LV<T, 1> G(S.hg);
    const LV<T, 3> D(S.lv[S.lc]);
    if constexpr (kTransport) {
        copy_in<6>(G, D, {G.b, G.acc, G.mx, G.my, G.dx, G.dy}, {D.b, D.acc, D.mx, D.my, D.dx, D.dy});
        for (int j = threadIdx.x; j < G.ny; j += blockDim.x) {
            D.dl[j] = G.dl[j]; D.dr[j] = G.dr[j]; D.mr[j] = G.mr[j]; D.ml[j] = G.ml[j];
        }
    } else {
        copy_in<3>(G, D, {G.b, G.te, G.tn}, {D.b, D.te, D.tn});
    }
}

template <typename T>
__device__ void handoff_out(Solve<T>& S) {
    using V4 = Vec4<T>;
    const LV<T, 3> D(S.lv[S.lc]);
    const LV<T, 1> G(S.hg);
    const int n4 = (G.nx * G.ny) >> 2;
    for (int i = threadIdx.x; i < n4; i += blockDim.x)
        ((typename AsPtr<V4, 1>::type)G.x)[i] = ((typename AsPtr<V4, 3>::type)D.x)[i];
}

// One V-cycle.  The cluster levels (0 .. lc-1) are run by the whole
// cluster; the leader alone runs the rest: its workgroup the levels in
// global memory or in its part of LDS, and from the first level of at most
// lds_cells cells (S.lds_from; the coarsest level always is) down to the
// coarsest and back, its wavefront 0 alone while the other wavefronts wait at
// one barrier.  With coarse_coeffs the leader first forms the coefficients of
// levels lc+1 .. lds_from (the cluster formed levels 1 .. lc before the
// cycle).
template <typename T, bool kTransport, bool kTrans = false>
__device__ void vcycle(Solve<T>& S, PhaseClock* pc = nullptr, bool coarse_coeffs = false) {
    const int lw = S.lds_from;
    const int lc = S.lc;
    const int t0 = kTransport ? 16 : 8;
    if (pc) pc->tick(kTransport ? 4 : 1);
    for (int l = 0; l < lc; ++l) {
        vdown<T, kTransport, kTrans, ClusterTeam, 1, 1>(S, l);
        if (pc) pc->tick(t0 + (l == 0 ? 1 : 2));
    }
    const int lb = S.lb;
    if (g_cl.member == 0) {
        if (S.hand) {
            handoff_in<T, kTransport>(S);
            __syncthreads();
        }
        if (coarse_coeffs) coarsen_leader<T, kTransport>(S, lc + 1);
        for (int l = lc; l < lw; ++l) {
            if (l + 1 < lb) vdown<T, kTransport, kTrans, BlockTeam, 1, 1>(S, l);
            else if (l < lb) vdown<T, kTransport, kTrans, BlockTeam, 1, 3>(S, l);
            else vdown<T, kTransport, kTrans, BlockTeam, 3, 3>(S, l);
            if (pc) pc->tick(t0 + (l == 0 ? 1 : 2));
        }
        if (threadIdx.x < kWave) wave_cycle<T, kTransport, kTrans>(S.lv[lw], S.wave);
        __syncthreads();
        if (pc) pc->tick(t0 + 3);
        for (int l = lw - 1; l >= lc; --l) {
            if (l + 1 < lb) vup<T, kTransport, kTrans, BlockTeam, 1, 1>(S, l);
            else if (l < lb) vup<T, kTransport, kTrans, BlockTeam, 1, 3>(S, l);
            else vup<T, kTransport, kTrans, BlockTeam, 3, 3>(S, l);
            if (pc) pc->tick(t0 + (l == 0 ? 6 : 4));
        }
        if (S.hand) handoff_out(S);
    }
    if (lc > 0) {
        ClusterTeam::sync();
        for (int l = lc - 1; l >= 0; --l) {
            vup<T, kTransport, kTrans, ClusterTeam, 1, 1>(S, l);
            if (pc) pc->tick(t0 + (l == 0 ? 6 : 4));
        }
    }
}

// Batched per-cell loops of the step: every thread first loads its kB cells
// (kB round trips in flight at once), then stores; one cell per loop trip
// would wait out a full memory latency per cell.
template <int kB>
__device__ inline void extrapolate_field(const double* u0, const double* u1, const double* u2, const double* u3,
                                         double* u4, int order, int n, int rk, int ts) {
    for (int base = rk; base < n; base += kB * ts) {
        double a0[kB], a1[kB], a2[kB], a3[kB], a4[kB];
#pragma unroll
        for (int k = 0; k < kB; ++k) {
            const int idx = base + k * ts;
            if (idx < n) {
                a0[k] = u0[idx]; a1[k] = u1[idx]; a2[k] = u2[idx]; a3[k] = u3[idx];
                a4[k] = order == 4 ? u4[idx] : 0.0;
            }
        }
#pragma unroll
        for (int k = 0; k < kB; ++k) {
            const int idx = base + k * ts;
            if (idx < n) {
                double e = a0[k];
                if (order == 1) e = 2.0 * a0[k] - a1[k];
                else if (order == 2) e = 3.0 * a0[k] - 3.0 * a1[k] + a2[k];
                else if (order == 3) e = 4.0 * a0[k] - 6.0 * a1[k] + 4.0 * a2[k] - a3[k];
                else if (order == 4) e = (16.0 * a0[k] - 14.0 * a1[k] - 4.0 * a2[k] + 11.0 * a3[k] - 4.0 * a4[k]) * 0.2;
                u4[idx] = e;  // the oldest state's array becomes the iterate
            }
        }
    }
}

template <int kB, typename T, class XI>
__device__ inline void add_correction(double* u, const T* x, int n, int rk, int ts, XI xi) {
    for (int base = rk; base < n; base += kB * ts) {
        double uv[kB];
        T xv[kB];
#pragma unroll
        for (int k = 0; k < kB; ++k) {
            const int idx = base + k * ts;
            if (idx < n) { uv[k] = u[idx]; xv[k] = x[xi(idx)]; }
        }
#pragma unroll
        for (int k = 0; k < kB; ++k) {
            const int idx = base + k * ts;
            if (idx < n) u[idx] = uv[k] + (double)xv[k];
        }
    }
}

// One implicit Euler step (Sec. 2.3) from the state u^n = (S.p, S.c):
// u^n becomes S.cn / S.pp (c^n is the previous time level of the
// residual) and the older states move down one role (bind_history), and the
// defect correction runs until
// both scaled residual max norms are <= tol.  The iteration starts from an
// extrapolation through the last states, by `order`: 0..3 the polynomial
// through the last order + 1 states (u^n; 2u^n - u^{n-1};
// 3u^n - 3u^{n-1} + u^{n-2}; 4u^n - 6u^{n-1} + 4u^{n-2} - u^{n-3}), 4 the
// least-squares cubic through the last five, (16u^n - 14u^{n-1} - 4u^{n-2}
// + 11u^{n-3} - 4u^{n-4}) / 5, which amplifies the states' own errors (of
// the size of the tolerance) less than the interpolating cubic does; on
// entry S.cn/pp, c2/p2, c3/p3, c4/p4 hold u^{n-1} .. u^{n-4}.  The start
// only changes how many iterations a step takes, not what it converges to.
// Returns 0 converged, 1 max_outer reached, 2 non-finite residual; adds the
// iterations used to `iters`.
template <typename T>
__device__ int implicit_step(const Phys& ph, Solve<T>& S, double* red, int max_outer, double tol, double& iters,
                             PhaseClock& pc, int order = 0) {
    const int n = S.n;
    const int rk = ClusterTeam::rank(), ts = ClusterTeam::size();
    extrapolate_field<4>(S.c, S.cn, S.c2, S.c3, S.c4, order, n, rk, ts);
    extrapolate_field<4>(S.p, S.pp, S.p2, S.p3, S.p4, order, n, rk, ts);
    ClusterTeam::sync();
    if (threadIdx.x == 0) {
        S.hist = (S.hist + 4) % 5;
        bind_history(S, reinterpret_cast<uint8_t*>(S.scratch - (int64_t)kF64Arrays * n));
    }
    __syncthreads();
    pc.tick(7);
    for (int it = 0; it < max_outer; ++it) {
        double np, nc;
        pc.tick(13);
        residual_pass(S, 0, red, np, nc, &pc);
        pc.tick(0);
        if (!(np == np) || !(nc == nc) || np > 1e300 || nc > 1e300) return 2;
        if (np <= tol && nc <= tol) return 0;
        iters += 1.0;
        if (np > tol) {  // a pressure residual within the tolerance needs no correction
            coarsen_cluster<T, false>(S);
            pc.tick(1);
            vcycle<T, false>(S, &pc, true);
            pc.tick(2);
            const int nx = S.nx, sx = log2i(S.nx);
            add_correction<8>(S.p, S.lv[0].x, n, rk, ts, [=](int idx) {
                const int j = idx >> sx;
                return pidx(idx - j * nx, j, nx);
            });
            ClusterTeam::sync();
        }
        pc.tick(15);
        // the salt system's pass evaluates both residuals at the updated
        // state: the step may end here, before the salt cycle
        residual_pass(S, 1, red, np, nc, &pc);
        if (!(np == np) || !(nc == nc) || np > 1e300 || nc > 1e300) return 2;
        if (np <= tol && nc <= tol) return 0;
        pc.tick(3);
        coarsen_cluster<T, true>(S);
        pc.tick(4);
        vcycle<T, true>(S, &pc, true);
        pc.tick(5);
        add_correction<8>(S.c, S.lv[0].x, n, rk, ts, [](int idx) { return idx; });
        ClusterTeam::sync();
        pc.tick(6);
    }
    return 1;
}

// Initial state: c = c0 (or 0, Sec. 2.1); p only seeds the iteration: the
// cell's own hydrostatic value -rho(c) g y.
template <typename T>
__device__ void initial_state(const Phys& ph, Solve<T>& S, const double* c0) {
    for (int idx = ClusterTeam::rank(); idx < S.n; idx += ClusterTeam::size()) {
        const int j = idx / S.nx;
        const double c = c0 ? c0[idx] : 0.0;
        S.c[idx] = c;
        S.p[idx] = -rho_of(ph, c) * ph.g * (-1.0 + (j + 0.5) * S.h);
    }
}

// Q = h^2 sum_{x<1} phi rho(c) c (FP64) in an order fixed by the grid
// alone: wavefront 0 keeps 64 partial sums (lane l adds the cells of index
// l mod 64 in increasing order), then a fixed butterfly over the lanes, so
// every workgroup size, cluster size and build gives the same bits.  Once
// per solve; the other wavefronts wait.
template <typename T>
__device__ double qoi_of(const Phys& ph, Solve<T>& S, double* red) {
    if (threadIdx.x < kWave) {
        double part = 0.0;
        for (int idx = threadIdx.x; idx < S.n; idx += kWave)
            if ((idx % S.nx) < S.nx / 2) part += S.phi[idx] * rho_of(ph, S.c[idx]) * S.c[idx];
        part = wave_sum(part);
        if (threadIdx.x == 0) red[0] = part;
    }
    __syncthreads();
    const double q = red[0] * S.h * S.h;
    __syncthreads();  // red is reused
    return q;
}

// Start of a step after `good` converged states in a row (the initial state
// counts as one): the extrapolation order grows with the history, up to the
// interpolating cubic (predictor 1) or the least-squares cubic through five
// states (predictor 2).  Predictor 0 takes 2 where the states' own errors,
// of the size of tol, outweigh the cubic's interpolation error: solves of
// 200 steps or more at tol >= 1e-8; 1 elsewhere.
__device__ inline int max_order(int predictor, int nsteps, double tol) {
    return predictor == 2 || (predictor == 0 && nsteps >= 200 && tol >= 1e-8) ? 4 : 3;
}
__device__ inline int start_order(int good, int top) { return min(max(good - 1, 0), top); }
__device__ inline int next_good(int good, int st) { return st == 0 ? min(good + 1, 5) : 0; }

// ------------------------------------------------------------------ time series
// Value of the piecewise-constant solution at (x, y): the cell that holds
// the point; on a face between two cells the mean of both, at a corner of
// four the mean of the four (the mean of the one-sided limits).
__device__ inline double point_value(const double* c, int nx, int ny, double x, double y) {
    const double u = x * ny, v = (y + 1.0) * ny;
    int i0 = (int)floor(u), j0 = (int)floor(v);
    int i1 = i0, j1 = j0;
    if (u == (double)i0) i0 -= 1;  // a vertical face: the cells on both sides
    if (v == (double)j0) j0 -= 1;
    i0 = min(max(i0, 0), nx - 1); i1 = min(max(i1, 0), nx - 1);
    j0 = min(max(j0, 0), ny - 1); j1 = min(max(j1, 0), ny - 1);
    return 0.25 * ((c[j0 * nx + i0] + c[j0 * nx + i1]) + (c[j1 * nx + i0] + c[j1 * nx + i1]));
}

// One record of a solve's time series (eq:integral_fw, eq:12points), by the
// whole workgroup of the leader: the fresh-water area h^2 #{c <= c_fresh}
// (an integer count, so the sum is exact in any order) and c at the points.
template <typename T>
__device__ void record_trace(const Launch& lp, Solve<T>& S, int index, int k, double* red) {
    double* out = lp.trace + ((int64_t)index * lp.trace_nrec + (k - 1)) * (1 + lp.trace_npts);
    double cnt = 0.0;
    for (int idx = threadIdx.x; idx < S.n; idx += blockDim.x) cnt += S.c[idx] <= lp.trace_fresh ? 1.0 : 0.0;
    cnt = block_sum(cnt, red);
    if (threadIdx.x == 0) out[0] = cnt * S.h * S.h;
    if (threadIdx.x < lp.trace_npts)
        out[1 + threadIdx.x] =
            point_value(S.c, S.nx, S.ny, lp.trace_pts[2 * threadIdx.x], lp.trace_pts[2 * threadIdx.x + 1]);
}

// ------------------------------------------------------------------ the solve kernel
// Cluster levels of a solve shared by K workgroups: level 0, then every
// level of >= 1024 K cells (>= 1024 per member) whose coarser neighbour is
// not run by wavefront 0; the level after them is handed to the leader's
// LDS when it lives there (cluster levels, of 8192 cells or more, never
// do).  At K = 8 the 128x64 level of a 256x128 solve is split (1024 cells
// per member): 383 -> 367 ms for the 16 such solves of the L = 4 batch,
// against its leader running it alone.
template <typename T>
__device__ inline void set_cluster_levels(Solve<T>& S, int K) {
    int lc = 0;
    if (K > 1) {
        lc = 1;
        while (lc + 1 < S.lds_from && (S.lv[lc].nx * S.lv[lc].ny) >= 1024 * K) ++lc;
    }
    S.lc = lc;
    S.hand = lc > 0 && lc == S.lb;
}

// Blocks of a launch: one per solve, or with clusters of K > 1 the blocks
// x + 8 (K c + r), r = 0 .. K-1, for cluster (solve) x + 8 c, so that the
// K members of a solve share an XCD; the launch has ceil(nsolves / 8) 8 K
// blocks and those of clusters past the last solve return at once.
__device__ inline void cluster_of_block(int K, int& cid, int& member) {
    const int b = (int)blockIdx.x;
    if (K == 1) { cid = b; member = 0; return; }
    const int x = b & 7, s = b >> 3;
    cid = x + 8 * (s / K);
    member = s % K;
}

template <typename T>
__global__ void __launch_bounds__(sizeof(T) == 4 ? HENRY_FP32_THREADS : 512) henry_solve_kernel(Launch lp) {
    extern __shared__ __align__(256) uint8_t lds_levels[];
    __shared__ Solve<T> S;
    __shared__ double red[32];
    int cid, member;
    cluster_of_block(lp.cluster, cid, member);
    if (cid >= lp.nsolves) return;
    const SolveDesc d = lp.descs[cid];
    const Phys& ph = lp.ph;
    // local steps of this launch: a solve with r steps advances r/g_total
    // local steps per global step (lockstep schedule across grids)
    const int s_begin = (int)(((int64_t)lp.g_begin * d.nsteps) / lp.g_total);
    const int s_end = (int)(((int64_t)lp.g_end * d.nsteps) / lp.g_total);
    if (s_begin >= s_end) return;
    if (threadIdx.x == 0) {
        bind_solve(S, lp.ws + d.ws_off, d.nx, d.ny, lds_levels, lp.lds_cells, lp.lds_block_cells);
        S.nsteps = d.nsteps;
        S.tau = ph.T / d.nsteps;
        S.ph = ph;
        set_cluster_levels(S, lp.cluster);
    }
    __syncthreads();
    double* sp = S.scratch;
    if (lp.cluster > 1) cluster_init(lp.cluster, member, sp, lp.cluster_wait, lp.redo);
    else cluster_init_single();
    if (threadIdx.x == 0) cluster_stage(lds_levels, lp.lds_bytes, line_stage_bytes_per_wave<T>());
    const int n = S.n;
    // scratch: [0] = q, [1] = status, [2] = iterations, [3] = converged
    // states in a row (the initial state counts as one), [4] = the history's
    // rotation; written by the leader at the end of a launch, read by every
    // member at the next
    int status = 0, good = 1;
    double iters = 0.0;
    if (s_begin == 0) {
        initial_state(ph, S, lp.c0 ? lp.c0 + d.field_off : nullptr);
    } else {
        status = (int)sp[1];
        iters = sp[2];
        good = (int)sp[3];
    }
    if (threadIdx.x == 0) {
        S.q = sp[0];
        if (s_begin > 0) {
            S.hist = (int)sp[4];
            bind_history(S, lp.ws + d.ws_off);
        }
    }
    ClusterTeam::sync();
    PhaseClock pc;
    pc.init();
    const int64_t N = d.nsteps, nrec = lp.trace ? lp.trace_nrec : 0;
    const int top = max_order(lp.predictor, d.nsteps, lp.tol);
    int s = s_begin;
    for (; s < s_end && status != 2 && !g_cl.failed; ++s) {
        // extrapolate only through converged states: a step that stopped at
        // max_outer restarts the history
        const int st = implicit_step(ph, S, red, lp.max_outer, lp.tol, iters, pc, start_order(good, top));
        if (st == 2) status = 2;
        else if (st == 1 && status == 0) status = 1;
        good = next_good(good, st);
        if (nrec && st != 2) {
            // the record whose step is s + 1, if any (nrec <= N: at most one)
            const int64_t k = (int64_t)(s + 1) * nrec / N;
            if (k >= 1 && (k * N + nrec - 1) / nrec == s + 1) {
                if (member == 0) record_trace(lp, S, d.index, (int)k, red);
                ClusterTeam::sync();  // the others keep c until the leader has read it
            }
        }
    }
    ClusterTeam::sync();
    if (g_cl.failed) status = kStatusSync;
    if (member != 0) return;
    // outputs may overlap what the solve reads when it starts again (c0)
    const bool left = g_cl.failed && g_cl.redo;
    if (nrec && !left && (status == 2 || status == kStatusSync)) {
        // NaN in the records of step s (the step the solve stopped in, or
        // the first step of this launch) and later: the first such record is
        // k0 = floor((s - 1) nrec / N) + 1
        const int rw = 1 + lp.trace_npts;
        const int64_t k0 = s > 0 ? (int64_t)(s - 1) * nrec / N + 1 : 1;
        for (int64_t k = k0; k <= nrec; ++k)
            for (int v = threadIdx.x; v < rw; v += blockDim.x)
                lp.trace[((int64_t)d.index * nrec + (k - 1)) * rw + v] = __builtin_nan("");
    }
    if (threadIdx.x == 0) {
        sp[3] = (double)good;
        sp[1] = (double)status;
        sp[2] = iters;
        sp[4] = (double)S.hist;
        sp[kClusterGen] = (double)g_cl.gen;
#ifdef HENRY_PHASE_TIMERS
        for (int k = 0; k < 24; ++k) sp[8 + k] = (double)pc.acc[k];
#endif
    }
    if (left) {
        if (threadIdx.x == 0 && s_end == d.nsteps) lp.status[d.index] = status;
    } else if (s_end == d.nsteps) {
        // outputs: c, p at T and the QoI
        for (int idx = threadIdx.x; idx < n; idx += blockDim.x) {
            lp.c_out[d.field_off + idx] = S.c[idx];
            if (lp.p_out) lp.p_out[d.field_off + idx] = S.p[idx];
        }
        const double Q = qoi_of(ph, S, red);
        if (threadIdx.x == 0) {
            lp.qoi_out[d.index] = Q;
            lp.status[d.index] = status;
            if (lp.iters) lp.iters[d.index] = (int32_t)iters;
        }
    }
}

// The kernels below run from the main build only (a build of the solve
// kernel alone defines HENRY_SOLVE_KERNEL_ONLY).
#ifndef HENRY_SOLVE_KERNEL_ONLY

// The FP64 residual of one solve's discrete equations at a given state
// (p, c; previous time level cn): the same residual pass as the solver's,
// writing R^p and R^c instead of the inner-solve arrays.  One workgroup per
// solve, after henry_fields_kernel.  kWide: with the face coefficients formed
// from K and phi and four rows loaded ahead, for grids of at least
// kResidualWide columns, where a thread's rows are a long chain of loads.
template <bool kWide>
__global__ void __launch_bounds__(kWide ? 256 : 1024)
    henry_residual_kernel(Launch lp, const double* p, const double* c, const double* cn, double* rp, double* rc) {
    extern __shared__ __align__(256) uint8_t lds_levels[];  // launched with none: no level in LDS
    __shared__ Solve<float> S;
    __shared__ double red[32];
    const SolveDesc d = lp.descs[blockIdx.x];
    const Phys& ph = lp.ph;
    if (threadIdx.x == 0) {
        bind_solve(S, lp.ws + d.ws_off, d.nx, d.ny, lds_levels, 0, 0);
        S.nsteps = d.nsteps;
        S.tau = ph.T / d.nsteps;
        S.ph = ph;
        S.q = S.scratch[0];
        S.rout_p = rp + d.field_off;
        S.rout_c = rc + d.field_off;
    }
    cluster_init_single();
    for (int idx = threadIdx.x; idx < S.n; idx += blockDim.x) {
        S.p[idx] = p[d.field_off + idx];
        S.c[idx] = c[d.field_off + idx];
        S.cn[idx] = cn[d.field_off + idx];
    }
    __syncthreads();
    residual_rows<float, 2, kWide>(S);
}

// Before a launch of one workgroup per solve over the same descriptors that
// takes the solves which reported HENRY_STATUS_SYNC: no steps for the others.
__global__ void henry_redo_kernel(SolveDesc* descs, int nsolves, const int32_t* status) {
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k < nsolves && status[descs[k].index] != kStatusSync) descs[k].nsteps = 0;
}

// ------------------------------------------------------------------ random fields
// Point values at cell centres of the closed-form fields, of the KL
// expansions, of the two-layer porosity model, or the caller's explicit
// fields; FP64.  One block per solve.
__global__ void henry_fields_kernel(Launch lp) {
    const SolveDesc d = lp.descs[blockIdx.x];
    const Phys& ph = lp.ph;
    uint8_t* base = lp.ws + d.ws_off;
    double* f = reinterpret_cast<double*>(base);
    const int nx = d.nx, ny = d.ny, n = nx * ny;
    double* phi = f + (int64_t)kPhi * n;
    double* K = f + (int64_t)kK * n;
    double* sp = f + (int64_t)kF64Arrays * n;
    const double h = 1.0 / ny;
    if (lp.field_kind == 2) {
        // truncated KL expansions: phi = phi0 (1 + s_phi Z_phi), log K = log k0 + s_K Z_K,
        // Z = sum_k sqrt(lam_k) e_k xi_k; recharge factor (1 + 0.2 xi_41)
        const double* xi = lp.xi + (size_t)41 * d.index;
        for (int idx = threadIdx.x; idx < n; idx += blockDim.x) {
            double zp = 0.0, zk = 0.0;
            for (int k = 0; k < 20; ++k) {
                const double m = lp.kl_modes[(size_t)k * n + idx];
                zp += m * xi[k];
                zk += m * xi[20 + k];
            }
            phi[idx] = ph.phi0 * (1.0 + lp.kl_sigma_phi * zp);
            K[idx] = exp(log(ph.k0) + lp.kl_sigma_logk * zk);
        }
        if (threadIdx.x == 0) sp[0] = ph.q_in * (1.0 + 0.2 * xi[40]);
    } else if (lp.field_kind == 0) {
        const double x1 = lp.xi[3 * d.index], x2 = lp.xi[3 * d.index + 1], x3 = lp.xi[3 * d.index + 2];
        for (int idx = threadIdx.x; idx < n; idx += blockDim.x) {
            const int i = idx % nx, j = idx / nx;
            const double x = (i + 0.5) * h, y = -1.0 + (j + 0.5) * h;
            phi[idx] = ph.phi0 * (1.0 + 0.2 * x1 * cos(M_PI * x / 2.0) * cos(M_PI * y));
            K[idx] = ph.k0 * exp(0.5 * x2 * sin(M_PI * x / 2.0));
        }
        if (threadIdx.x == 0) sp[0] = ph.q_in * (1.0 + 0.2 * x3);
    } else if (lp.field_kind == 3) {
        // two porosity layers split at y = -0.75 (eq:poro_2levels, eq:poro_2levels_C),
        // Kozeny-Carman permeability (e_perm_Kozeny_Carman) scaled so that
        // K(phi0) = k0, recharge q_in (1 + 0.5 xi3)
        const double x1 = lp.xi[3 * d.index], x2 = lp.xi[3 * d.index + 1], x3 = lp.xi[3 * d.index + 2];
        const double kappa = ph.k0 * (1.0 - ph.phi0 * ph.phi0) / (ph.phi0 * ph.phi0 * ph.phi0);
        for (int idx = threadIdx.x; idx < n; idx += blockDim.x) {
            const int i = idx % nx, j = idx / nx;
            const double x = (i + 0.5) * h, y = -1.0 + (j + 0.5) * h;
            const double layer = y < -0.75 ? 1.0 + 0.2 * x1 : 1.0 - 0.2 * x1;
            const double fP =
                ph.phi0 * (1.0 + 0.15 * (x2 * cos(M_PI * x / 2.0) + x2 * sin(2.0 * M_PI * y) + x1 * cos(2.0 * M_PI * x))) *
                layer;
            phi[idx] = fP;
            K[idx] = kappa * fP * fP * fP / (1.0 - fP * fP);
        }
        if (threadIdx.x == 0) sp[0] = ph.q_in * (1.0 + 0.5 * x3);
    } else {
        for (int idx = threadIdx.x; idx < n; idx += blockDim.x) {
            phi[idx] = lp.phi_in[d.field_off + idx];
            K[idx] = exp(lp.logk_in[d.field_off + idx]);
        }
        if (threadIdx.x == 0) sp[0] = lp.qin_in[d.index];
    }
    // a fresh cluster state for the solve's first launch
    if (threadIdx.x == 0) {
        for (int k = kClusterFlags; k <= kClusterGen; ++k) sp[k] = 0.0;
    }
    __syncthreads();
    // face coefficients (harmonic means) and the residual scale
    double* tx = f + (int64_t)kTx * n;
    double* ty = f + (int64_t)kTy * n;
    double* wx = f + (int64_t)kWx * n;
    double* wy = f + (int64_t)kWy * n;
    double* isc = f + (int64_t)kIsc * n;
    const double tau = ph.T / d.nsteps;
    for (int idx = threadIdx.x; idx < n; idx += blockDim.x) {
        const int i = idx % nx, j = idx / nx;
        const double KP = K[idx], fP = phi[idx];
        if (i + 1 < nx) {
            const FacePair fx = face_pair(ph, KP, K[idx + 1], fP, phi[idx + 1]);
            tx[idx] = fx.t;
            wx[idx] = fx.w;
        } else {
            const FacePair fx = face_pair(ph, KP, KP, fP, fP);
            tx[idx] = 2.0 * fx.t;
            wx[idx] = 2.0 * fx.w;
        }
        if (j + 1 < ny) {
            const FacePair fy = face_pair(ph, KP, K[idx + nx], fP, phi[idx + nx]);
            ty[idx] = fy.t;
            wy[idx] = fy.w;
        } else {
            ty[idx] = 0.0;
            wy[idx] = 0.0;
        }
        isc[idx] = res_scale(ph, tau, h, fP);
    }
}

#endif  // HENRY_SOLVE_KERNEL_ONLY

}  // namespace HENRY_NS
