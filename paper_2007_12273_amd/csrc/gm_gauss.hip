// gm_gauss.hip -- Gauss'-law weight correction after resampling (Sec. 2.4.1).
//
// Mesh: periodic, nx cells (dx = 1) or nx * ny cells (dx = 2, cell c at
// (c % nx, c / nx)), unit cells; cell i has centre X_i = i + 1/2 and a
// particle of cell c with cell-local position x sits at X = (cell) + x.
//
//   k_stencil   one wave per cell: the quadratic B-spline weights
//               S2(X_i - X_p) of its particles on the 3 (1D) or 9 (2D) mesh
//               cells around it, summed plain (the cell's column of the mass
//               matrix M_ij = sum_{p in j} S2(X_i - X_p), eq.
//               p-weight-correction with the top-hat S0) and weighted by w_p
//               (the cell's share of the deposit D_i = sum_p w_p S2(X_i -
//               X_p)); FP64, fixed-order sums
//   k_deposit   D_i or (M a)_i from the neighbouring cells' columns in a
//               fixed order (a gather: no atomics, deterministic)
//   solver      M dA = D_target - D(w) by BiCGSTAB with the Jacobi
//               preconditioner diag(M) applied on the right.  Every scalar
//               of the iteration stays in device memory: one-thread
//               epilogues fold the fixed-order block partials of the dot
//               products into rho, alpha, omega and a done flag, and every
//               vector kernel returns at once when the flag is set, so the
//               host enqueues iterations in chunks and reads the state once
//               per chunk.  A restart recomputes the true residual b - M dA,
//               which alone decides convergence (below tol |b|).  Meshes
//               of up to 131072 cells run the whole solve in one launch
//               (k_solve).
//   k_apply_dA  w_p += dA_{cell(p)} (eq. new-p-weight)
#include <atomic>
#include <cmath>

#include "gm_device.h"

namespace gm {

constexpr int kStencilThreads = 256;
constexpr int kVecThreads = 256;

__device__ __forceinline__ double bspline2(double s)
{
    const double a = fabs(s);
    if (a <= 0.5) return 0.75 - a * a;
    if (a <= 1.5) return 0.5 * (1.5 - a) * (1.5 - a);
    return 0.0;
}

// slot o of a cell's stencil: 1D o = ox + 1 (ox = -1, 0, 1); 2D o = 3 (oy +
// 1) + (ox + 1); the cell's own slot is 1 (1D) or 4 (2D)
template <int DX>
constexpr int kSlots = DX == 1 ? 3 : 9;
template <int DX>
constexpr int kCentre = DX == 1 ? 1 : 4;

// one wave per cell (kStencilThreads / 64 cells per workgroup): lanes stride
// over the cell's particles, then wave-wide sums of the slots (fixed order)
template <int DX>
__global__ __launch_bounds__(kStencilThreads) void k_stencil(const double* x, const double* w, const int64_t* off,
                                                             int64_t n_cells, double* colM, double* colW,
                                                             unsigned long long* tag, int ntag)
{
    constexpr int NS = kSlots<DX>;
    if (blockIdx.x == 0 && (int)threadIdx.x < ntag) tag[threadIdx.x] = 0;  // k_solve's tags
    const int lane = threadIdx.x & 63;
    const int64_t c = (int64_t)blockIdx.x * (kStencilThreads / 64) + (threadIdx.x >> 6);
    if (c >= n_cells) return;  // whole waves leave; no workgroup barrier follows
    const int64_t o0 = off[c], n = off[c + 1] - o0;
    double acc[2 * NS];
#pragma unroll
    for (int t = 0; t < 2 * NS; ++t) acc[t] = 0.0;
    for (int64_t i = lane; i < n; i += 64) {
        const double wp = w[o0 + i];
        double sx[3], sy[3] = {1.0, 0.0, 0.0};
        const double px = x[(o0 + i) * DX];
#pragma unroll
        for (int o = 0; o < 3; ++o) sx[o] = bspline2((o - 1) + 0.5 - px);
        if constexpr (DX == 2) {
            const double py = x[(o0 + i) * DX + 1];
#pragma unroll
            for (int o = 0; o < 3; ++o) sy[o] = bspline2((o - 1) + 0.5 - py);
        }
#pragma unroll
        for (int oy = 0; oy < (DX == 2 ? 3 : 1); ++oy)
#pragma unroll
            for (int ox = 0; ox < 3; ++ox) {
                const double s = DX == 2 ? sx[ox] * sy[oy] : sx[ox];
                acc[oy * 3 + ox] += s;
                acc[NS + oy * 3 + ox] += wp * s;
            }
    }
    // value v of the transposed sums ends in register v / 4 of every lane of
    // its row; the row's last lane stores it
    constexpr int NB = (2 * NS + 3) / 4;
    double b[NB];
    wave_sums_transposed<2 * NS>(acc, b);
    if ((lane & 15) == 15) {
        const int r = lane >> 4, first = 2 * (r & 1) + (r >> 1);
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            const int v = 4 * j + first;
            if (v < NS) {
                if (colM) colM[c * NS + v] = b[j];
            } else if (v < 2 * NS) {
                colW[c * NS + v - NS] = b[j];
            }
        }
    }
}

// sum over the stencil slots o of col[j(i, o)][o] * f(j), j = the cell whose
// slot o lands on mesh cell i
template <int DX, typename F>
__device__ __forceinline__ double gather(const double* col, int64_t i, int64_t n_cells, int nx, int ny, F f)
{
    constexpr int NS = kSlots<DX>;
    double t = 0.0;
    if constexpr (DX == 1) {
#pragma unroll
        for (int o = 0; o < 3; ++o) {
            int64_t j = i - (o - 1);
            j = j < 0 ? j + n_cells : (j >= n_cells ? j - n_cells : j);
            t += col[j * NS + o] * f(j);
        }
    } else {
        const int ix = (int)(i % nx), iy = (int)(i / nx);
#pragma unroll
        for (int oy = 0; oy < 3; ++oy) {
            int jy = iy - (oy - 1);
            jy = jy < 0 ? jy + ny : (jy >= ny ? jy - ny : jy);
#pragma unroll
            for (int ox = 0; ox < 3; ++ox) {
                int jx = ix - (ox - 1);
                jx = jx < 0 ? jx + nx : (jx >= nx ? jx - nx : jx);
                const int64_t j = (int64_t)jy * nx + jx;
                t += col[j * NS + oy * 3 + ox] * f(j);
            }
        }
    }
    return t;
}

// the deposit D_i from the weighted columns
template <int DX>
__global__ __launch_bounds__(kVecThreads) void k_deposit(const double* colW, int64_t n_cells, int nx, int ny,
                                                        double* out)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n_cells) return;
    out[i] = gather<DX>(colW, i, n_cells, nx, ny, [](int64_t) { return 1.0; });
}

// ---------------------------------------------------------------------------
// solver state (device): the scalars of the iteration and its flags
// ---------------------------------------------------------------------------
enum : int { S_RHO, S_ALPHA, S_OMEGA, S_BETA, S_TOL2B2, S_R2, S_DONE, S_ITERS, S_EMPTY, S_COUNT };
// S_DONE: 0 running, 1 converged, 2 stopped (a breakdown or a vanishing
// omega; the host restarts from the true residual); of k_solve 3: all
// iterations used, far from the tolerance

// Block partials of two dot products: every thread adds its own terms, the
// workgroup reduces them in a fixed order, thread 0 stores them.
__device__ __forceinline__ void store_partials(double a0, double a1, double* partial)
{
    __shared__ double red[2 * kMaxWaves * 2];
    int par = 0;
    double acc[2] = {a0, a1};
    block_sum<2>(acc, red, par, blockDim.x >> 6);
    if (threadIdx.x == 0) {
        partial[2 * blockIdx.x] = acc[0];
        partial[2 * blockIdx.x + 1] = acc[1];
    }
}

__device__ __forceinline__ bool halted(const double* st) { return st[S_DONE] != 0.0; }

enum : int { E_INIT, E_RESTART, E_ALPHA, E_OMEGA, E_RES_RHO };

// Folds the block partials (fixed order) and updates the state:
//   E_INIT     s0 = b.b, s1 = number of empty cells
//   E_RESTART  s0 = r.r of the true residual (rh = r, p = v = 0): converged
//              when s0 <= tol^2 b.b, else a fresh start with rho = rh.r = s0
//   E_ALPHA    s0 = rh.v: alpha = rho / s0
//   E_OMEGA    s0 = t.s, s1 = t.t: omega = s0 / s1
//   E_RES_RHO  s0 = r.r, s1 = rh.r of the new residual: one more iteration;
//              done, or beta = (s1 / rho) (alpha / omega) and rho = s1
__global__ __launch_bounds__(kVecThreads) void k_fold(const double* partial, int nblocks, double* st, int mode,
                                                      double tol)
{
    __shared__ double red[2 * kMaxWaves * 2];
    int par = 0;
    double acc[2] = {0.0, 0.0};
    for (int b = threadIdx.x; b < nblocks; b += blockDim.x) {
        acc[0] += partial[2 * b];
        acc[1] += partial[2 * b + 1];
    }
    block_sum<2>(acc, red, par, blockDim.x >> 6);
    if (threadIdx.x != 0) return;
    const double s0 = acc[0], s1 = acc[1];
    switch (mode) {
        case E_INIT:
            st[S_TOL2B2] = tol * tol * s0;
            st[S_EMPTY] = s1;
            st[S_R2] = s0;
            st[S_ITERS] = 0.0;
            st[S_DONE] = s0 == 0.0 ? 1.0 : 0.0;
            break;
        case E_RESTART:
            st[S_R2] = s0;
            st[S_ALPHA] = 1.0;
            st[S_OMEGA] = 1.0;
            st[S_RHO] = s0;
            st[S_BETA] = 0.0;
            st[S_DONE] = s0 <= st[S_TOL2B2] ? 1.0 : (isfinite(s0) ? 0.0 : 2.0);
            break;
        case E_ALPHA:
            if (st[S_DONE] != 0.0) break;
            if (s0 == 0.0 || !isfinite(s0))
                st[S_DONE] = 2.0;
            else
                st[S_ALPHA] = st[S_RHO] / s0;
            break;
        case E_OMEGA:
            if (st[S_DONE] != 0.0) break;
            st[S_OMEGA] = s1 > 0.0 ? s0 / s1 : 0.0;
            break;
        case E_RES_RHO:
            if (st[S_DONE] != 0.0) break;
            st[S_ITERS] += 1.0;
            st[S_R2] = s0;
            if (s0 <= st[S_TOL2B2]) {
                st[S_DONE] = 1.0;
            } else if (st[S_OMEGA] == 0.0 || s1 == 0.0 || !isfinite(s0) || !isfinite(s1)) {
                st[S_DONE] = 2.0;
            } else {
                st[S_BETA] = (s1 / st[S_RHO]) * (st[S_ALPHA] / st[S_OMEGA]);
                st[S_RHO] = s1;
            }
            break;
    }
}

// dinv_j = 1 / M_jj (a cell with particles has M_jj >= n_j / 4 > 0), b =
// target - D(w), dA = 0; partials of (b.b, number of empty cells)
template <int DX>
__global__ __launch_bounds__(kVecThreads) void k_setup(const double* colM, const double* colW,
                                                       const double* target, const int64_t* off, int64_t n_cells,
                                                       int nx, int ny, double* dinv, double* b, double* x,
                                                       double* partial)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    double bb = 0.0, e = 0.0;
    if (i < n_cells) {
        const bool empty = off[i + 1] <= off[i];
        dinv[i] = empty ? 0.0 : 1.0 / colM[i * kSlots<DX> + kCentre<DX>];
        const double bi = target[i] - gather<DX>(colW, i, n_cells, nx, ny, [](int64_t) { return 1.0; });
        b[i] = bi;
        x[i] = 0.0;
        bb = bi * bi;
        e = empty ? 1.0 : 0.0;
    }
    store_partials(bb, e, partial);
}

// restart: r = rh = b - M dA, p = v = 0; partials of (r.r, r.r)
template <int DX>
__global__ __launch_bounds__(kVecThreads) void k_restart(const double* colM, const double* b, const double* x,
                                                         int64_t n_cells, int nx, int ny, double* r, double* rh,
                                                         double* p, double* v, double* partial)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    double rr = 0.0;
    if (i < n_cells) {
        const double ri = b[i] - gather<DX>(colM, i, n_cells, nx, ny, [&](int64_t j) { return x[j]; });
        r[i] = ri;
        rh[i] = ri;
        p[i] = 0.0;
        v[i] = 0.0;
        rr = ri * ri;
    }
    store_partials(rr, rr, partial);
}

// p = r + beta (p - omega v)
__global__ __launch_bounds__(kVecThreads) void k_update_p(const double* st, const double* r, const double* v,
                                                          double* p, int64_t n)
{
    if (halted(st)) return;
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = r[i] + st[S_BETA] * (p[i] - st[S_OMEGA] * v[i]);
}

// y = M diag(dinv) a; partials of (rh.y, 0), or (y.a, y.y) when TS
template <int DX, bool TS>
__global__ __launch_bounds__(kVecThreads) void k_spmv(const double* st, const double* colM, const double* dinv,
                                                      const double* a, const double* rh, int64_t n_cells, int nx,
                                                      int ny, double* y, double* partial)
{
    if (halted(st)) return;
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    double q0 = 0.0, q1 = 0.0;
    if (i < n_cells) {
        const double yi = gather<DX>(colM, i, n_cells, nx, ny, [&](int64_t j) { return dinv[j] * a[j]; });
        y[i] = yi;
        if constexpr (TS) {
            q0 = yi * a[i];
            q1 = yi * yi;
        } else {
            q0 = rh[i] * yi;
        }
    }
    store_partials(q0, q1, partial);
}

// s = r - alpha v
__global__ __launch_bounds__(kVecThreads) void k_update_s(const double* st, const double* r, const double* v,
                                                          double* s, int64_t n)
{
    if (halted(st)) return;
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) s[i] = r[i] - st[S_ALPHA] * v[i];
}

// dA += dinv (alpha p + omega s), r = s - omega t; partials of (r.r, rh.r)
__global__ __launch_bounds__(kVecThreads) void k_update_xr(const double* st, const double* dinv, const double* p,
                                                           const double* s, const double* t, const double* rh,
                                                           double* x, double* r, int64_t n, double* partial)
{
    if (halted(st)) return;
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    double q0 = 0.0, q1 = 0.0;
    if (i < n) {
        const double al = st[S_ALPHA], om = st[S_OMEGA];
        x[i] += dinv[i] * (al * p[i] + om * s[i]);
        const double ri = s[i] - om * t[i];
        r[i] = ri;
        q0 = ri * ri;
        q1 = rh[i] * ri;
    }
    store_partials(q0, q1, partial);
}

// ---------------------------------------------------------------------------
// The whole solve in one launch, for meshes whose rows fit a workgroup.
//
// Workgroup g owns a block of whole rows (dx = 2) or of cells (dx = 1), up to
// kSolveOwn cells, two per thread; a thread keeps its cells' mass-matrix rows
// and vectors in registers and the workgroup the scaled vector it multiplies
// in LDS, with one row (one cell) of halo on either side.  An iteration needs
// two exchanges: after v = M dinv p the workgroups publish v and their parts
// of rh.v and of the |r|^2 that the iteration before left, after t = M dinv s
// they publish t and their parts of t.s, t.t, rh.s and rh.t; omega and the new
// rho = rh.s - omega rh.t follow from those.  That difference cancels (in one
// part it lost up to four times what a dot product with r rounds off), so its
// two sums and the difference are carried in two parts; it then holds more than
// the dot product would.  Every workgroup
// updates p, r and s of its halo itself from the neighbours' v and t.  The
// restarts from the true residual b - M dA, which alone decides convergence,
// run inside as well.  Launched one kernel per step the solve was bound by
// its eight launches and a host round trip per eight iterations: 23 us an
// iteration.  Solve on the 65536-cell grid (64 workgroups, 27 iterations)
// 0.27 ms against 0.74 ms and four host round trips, on 4096 cells in 1D (4
// workgroups) 0.10 ms against 0.36 ms; what is left is the two exchanges, 4.6 us
// each.
//
// An exchange: each workgroup stores its halo-visible values and partial
// sums, then, once they are out, a tag with the exchange's number; every
// workgroup waits for all tags and adds the partials in workgroup order, so
// all take the same decisions.  Buffers alternate by the parity of the
// exchange: a workgroup two exchanges ahead would need every tag of the one
// between.  The exchanges need the whole grid (at most kSolveMaxGroups
// workgroups, one per CU) resident.  The host launches it only where the device
// has that many CUs that no other such solve of the process holds (SolvePlaces);
// where another process or a long kernel keeps some of its workgroups out all
// the same, a wait gives up after kSolveWaitUs and marks its tags, on which
// every other workgroup leaves too, those that start later at their first
// exchange.
//
// A solve that used up max_iter without a restart, still kSolveFar above its
// tolerance, is the answer: launch by launch the same iterations end there too
// (five of them on the 65536-cell grid: 0.27 ms, 0.54 with that).  Any
// other that did not converge (an abandoned wait, a breakdown, iterations that
// ended near the tolerance, where another order of the sums may save one)
// leaves the weights alone, and the host solves launch by launch.
// ---------------------------------------------------------------------------
constexpr int kSolveThreads = 512;
constexpr int kSolveOwn = 2 * kSolveThreads;   // cells a workgroup owns
constexpr int kSolveHalo = kSolveThreads;      // cells of one halo row
constexpr int kSolveMaxGroups = 128;
constexpr int kSolvePart = 8;                  // doubles per workgroup and exchange: two sums, two in two parts (2 3, 6 7)
constexpr int kSolveMaxPolls = 1 << 20;        // bounds a wait whatever the clock says
// A wait is some microseconds where the grid is resident.  The limit is about
// the launch-per-step solve's time on the largest mesh taken here: giving up
// later would cost more than that solve, giving up earlier would leave grids
// whose start another stream's kernels delay.
constexpr int kSolveWaitUs = 2000;
constexpr double kSolveFar = 1e3;
constexpr unsigned long long kSolveGone = ~0ull;  // tag of a workgroup that gave up

struct SolveArgs {
    const double* colM;
    const double* colW;
    const double* target;
    const int64_t* off;
    int64_t n;
    int nx, ny;
    int per;              // rows (dx = 2) or cells (dx = 1) per workgroup
    double tol;
    int max_iter, max_restarts;
    long long wait;       // longest wait in ticks of the wall clock; 0: gives up at once
    double* x;            // [n] the corrections dA
    double* halo[2];      // [n] v or t (or dA, r at a restart), alternating
    double* part;         // [2][groups][kSolvePart]
    unsigned long long* tag;  // [2][groups], zero at the start
    double* st;
};

__device__ __forceinline__ void agent_store(double* p, double v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ double agent_load(const double* p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// the exchange's sums, in one part or two
__device__ __forceinline__ void agent_store(double* p, const Sum2& v)
{
    agent_store(p, v.hi);
    agent_store(p + 4, v.lo);
}
__device__ __forceinline__ void agent_load(const double* p, double& v) { v = agent_load(p); }
__device__ __forceinline__ void agent_load(const double* p, Sum2& v) { v = Sum2{agent_load(p), agent_load(p + 4)}; }
__device__ __forceinline__ void add2(double& a, double b) { a += b; }
struct NoSums {};

// Waits until this wave's stores have reached the point of coherence.  All
// that the workgroups share goes through agent-scope atomics, which pass the
// XCD's L2 by; a release fence would write the L2's other lines back as well,
// in every wave and exchange (18 us per exchange of 64 workgroups against 4.5).
__device__ __forceinline__ void stores_done() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

template <int DX>
__global__ __launch_bounds__(kSolveThreads) void k_solve(SolveArgs A)
{
    constexpr int NS = kSlots<DX>;
    constexpr int NC = 2;                       // own cells per thread, and halo cells per thread
    __shared__ double vec[kSolveOwn + 2 * kSolveHalo];
    constexpr int NW = kSolveThreads / 64;
    __shared__ double red[4][NW], tot[2];       // of the sums in one part
    __shared__ Sum2 red2[4][NW], tot2[2];       // of those in two
    const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
    const int G = gridDim.x, g = blockIdx.x;
    const int H = DX == 1 ? 1 : A.nx;           // cells of one halo row
    const int64_t c0 = (int64_t)g * A.per * (DX == 1 ? 1 : A.nx);
    const int64_t c1 = c0 + (int64_t)A.per * (DX == 1 ? 1 : A.nx) < A.n ? c0 + (int64_t)A.per * (DX == 1 ? 1 : A.nx) : A.n;
    const int own = (int)(c1 - c0);

    // local layout of `vec`: [0, H) the row before, [H, H + own) own, then the row after
    int64_t gi[NC], hi[NC];                     // global indices of own and halo cells
    int li[NC], lh[NC], nb[NC][NS];             // their places in vec; the stencil's places
    double m[NC][NS], dinv[NC], hdinv[NC], b[NC];
    double x[NC], p[NC], r[NC], rh[NC], v[NC], sv[NC], t[NC];
    double hp[NC], hr[NC], hv[NC], hs[NC];
    auto column = [&](int64_t j, int o) { return A.colM[j * NS + o]; };
#pragma unroll
    for (int k = 0; k < NC; ++k) {
        const int q = tid + k * kSolveThreads;
        const bool in = q < own;
        gi[k] = in ? c0 + q : -1;
        li[k] = H + q;
        dinv[k] = b[k] = x[k] = p[k] = r[k] = rh[k] = v[k] = sv[k] = t[k] = 0.0;
#pragma unroll
        for (int o = 0; o < NS; ++o) {
            m[k][o] = 0.0;
            nb[k][o] = 0;
        }
        if (in) {
            const int64_t i = gi[k];
            const bool empty = A.off[i + 1] <= A.off[i];
            dinv[k] = empty ? 0.0 : 1.0 / column(i, kCentre<DX>);
            b[k] = A.target[i] - gather<DX>(A.colW, i, A.n, A.nx, A.ny, [](int64_t) { return 1.0; });
            if constexpr (DX == 1) {
#pragma unroll
                for (int o = 0; o < 3; ++o) {
                    int64_t j = i - (o - 1);
                    j = j < 0 ? j + A.n : (j >= A.n ? j - A.n : j);
                    m[k][o] = column(j, o);
                    nb[k][o] = li[k] - (o - 1);
                }
            } else {
                const int ix = (int)(i % A.nx), iy = (int)(i / A.nx);
#pragma unroll
                for (int oy = 0; oy < 3; ++oy) {
                    int jy = iy - (oy - 1);
                    jy = jy < 0 ? jy + A.ny : (jy >= A.ny ? jy - A.ny : jy);
#pragma unroll
                    for (int ox = 0; ox < 3; ++ox) {
                        int jx = ix - (ox - 1);
                        jx = jx < 0 ? jx + A.nx : (jx >= A.nx ? jx - A.nx : jx);
                        m[k][oy * 3 + ox] = column((int64_t)jy * A.nx + jx, oy * 3 + ox);
                        nb[k][oy * 3 + ox] = li[k] - ix - (oy - 1) * A.nx + jx;
                    }
                }
            }
        }
        // halo cell q of 2 H: the row before the first own one, then the row after the last
        const bool hin = q < 2 * H;
        const int64_t j = q < H ? c0 - H + q : c1 + (q - H);
        hi[k] = hin ? (j < 0 ? j + A.n : (j >= A.n ? j - A.n : j)) : -1;
        lh[k] = q < H ? q : own + q;            // own + H + (q - H)
        hdinv[k] = hp[k] = hr[k] = hv[k] = hs[k] = 0.0;
        if (hin) hdinv[k] = A.off[hi[k] + 1] <= A.off[hi[k]] ? 0.0 : 1.0 / column(hi[k], kCentre<DX>);
    }

    unsigned long long epoch = 0;
    // publish val of the own cells, add up q over the grid (into tot), and
    // return the neighbours' val on the halo; false when a wait gave up
    auto exchange = [&](const double (&val)[NC], const double (&q)[2], const auto& q2, double (&hval)[NC]) -> bool {
        constexpr bool TWO = !std::is_same<std::remove_cv_t<std::remove_reference_t<decltype(q2)>>, NoSums>::value;
        ++epoch;
        const int par = (int)(epoch & 1);
        double* halo = A.halo[par];
#pragma unroll
        for (int k = 0; k < NC; ++k)
            if (gi[k] >= 0) agent_store(halo + gi[k], val[k]);
        // sum u ends in every lane of row tv_row(u)
        double w[1];
        wave_sums_transposed<2>(q, w);
        const int row = lane >> 4, sum = 2 * (row & 1) + (row >> 1);
        if ((lane & 15) == 15) red[sum][wid] = w[0];
        if constexpr (TWO) {
            Sum2 w2[1];
            wave_sums_transposed<2>(q2, w2);
            if ((lane & 15) == 15) red2[sum][wid] = w2[0];
        }
        stores_done();  // this wave's part is out before the tag below
        __syncthreads();
        double* part = A.part + (size_t)par * G * kSolvePart;
        if (wid == 0) {
            // sum u of the waves in the lanes 8 u .. 8 u + 7
            static_assert(NW == 8, "eight lanes hold a sum's waves");
            const int u = (lane >> 3) & 3;
            double* mine = part + (size_t)g * kSolvePart + u;
            const bool first = (lane & 7) == 0 && lane < 16;
            double a = red[u][lane & 7];
            dpp_add<0xB1>(a);
            dpp_add<0x4E>(a);
            dpp_add<0x141>(a);
            if (first) agent_store(mine, a);
            if constexpr (TWO) {
                Sum2 a2 = red2[u][lane & 7];
                dpp_add<0xB1>(a2);
                dpp_add<0x4E>(a2);
                dpp_add<0x141>(a2);
                if (first) agent_store(mine + 2, a2);
            }
            stores_done();
            if (lane == 0)
                __hip_atomic_store(A.tag + (size_t)par * G + g, epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        // lane l of wave w waits for workgroup 64 w + l
        bool ok = true;
        if (tid < G) {
            ok = false;
            long long t0 = 0;  // the clock is read in long waits only
            for (int poll = 0; A.wait > 0 && poll < kSolveMaxPolls; ++poll) {
                const unsigned long long seen =
                    __hip_atomic_load(A.tag + (size_t)par * G + tid, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                ok = seen == epoch;
                if (ok || seen == kSolveGone) break;
                if (poll == 32) t0 = wall_clock64();
                if (poll > 32 && wall_clock64() - t0 >= A.wait) break;
                __builtin_amdgcn_s_sleep(1);
            }
        }
        const bool all = __syncthreads_and(ok);
        if (!all) {
            if (tid < 2)
                __hip_atomic_store(A.tag + (size_t)tid * G + g, kSolveGone, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return false;
        }
        // wave u adds sum u over the workgroups: a lane its two, then the wave
        auto total = [&](auto zero, int u) {
            decltype(zero) a[1] = {zero}, b[1];
            const double* at = part + (size_t)lane * kSolvePart + u;
            if (lane < G) agent_load(at, a[0]);
            if (lane + 64 < G) {
                agent_load(at + 64 * kSolvePart, b[0]);
                add2(a[0], b[0]);
            }
            wave_sums_transposed<1>(a, b);
            return b[0];  // in lane 15
        };
        if (wid < 2) {
            const double a = total(0.0, wid);
            if (lane == 15) tot[wid] = a;
        } else if (TWO && wid < 4) {
            const Sum2 a = total(Sum2{0.0, 0.0}, wid);
            if (lane == 15) tot2[wid - 2] = a;
        }
#pragma unroll
        for (int k = 0; k < NC; ++k) hval[k] = hi[k] >= 0 ? agent_load(halo + hi[k]) : 0.0;
        __syncthreads();
        return true;
    };
    // y = M a over the own cells, a given on own and halo cells
    auto product = [&](const double (&a)[NC], const double (&ha)[NC], double (&y)[NC]) {
        __syncthreads();  // the last product's reads are done
#pragma unroll
        for (int k = 0; k < NC; ++k) {
            if (gi[k] >= 0) vec[li[k]] = a[k];
            if (hi[k] >= 0) vec[lh[k]] = ha[k];
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < NC; ++k) {
            double acc = 0.0;
#pragma unroll
            for (int o = 0; o < NS; ++o) acc += m[k][o] * vec[nb[k][o]];
            y[k] = gi[k] >= 0 ? acc : 0.0;
        }
    };

    double hx[NC], a_[NC], ha_[NC];
    int done = 0, iters = 0;
    double b2 = 0.0, r2 = 0.0, true_r2 = 0.0, empty = 0.0;
    // b.b and the number of empty cells
    double qb[2] = {0.0, 0.0};
#pragma unroll
    for (int k = 0; k < NC; ++k) {
        qb[0] += b[k] * b[k];
        if (gi[k] >= 0 && A.off[gi[k] + 1] <= A.off[gi[k]]) qb[1] += 1.0;
    }
    bool ok = exchange(x, qb, NoSums{}, hx);
    if (ok) {
        b2 = true_r2 = tot[0];
        empty = tot[1];
    }
    const double tol2b2 = A.tol * A.tol * b2;
    if (empty != 0.0 || b2 == 0.0) done = 1;
    for (int rs = 0; ok && done == 0 && rs <= A.max_restarts; ++rs) {
        // the true residual of the current dA (zero at first), and r on the halo
        product(x, hx, a_);
        double rho = 0.0, alpha = 1.0, omega = 1.0, beta = 0.0;
        double q[2] = {0.0, 0.0};
#pragma unroll
        for (int k = 0; k < NC; ++k) {
            r[k] = rh[k] = b[k] - a_[k];
            p[k] = v[k] = 0.0;
            hp[k] = hv[k] = 0.0;
            q[0] += r[k] * r[k];
        }
        ok = exchange(r, q, NoSums{}, hr);
        if (!ok) break;
        r2 = true_r2 = rho = tot[0];
        if (r2 <= tol2b2) {
            done = 1;
            break;
        }
        if (!isfinite(r2) || iters >= A.max_iter) {
            done = rs == 1 && isfinite(r2) && r2 > kSolveFar * kSolveFar * tol2b2 ? 3 : 2;
            break;
        }
        bool stop = false;
        while (!stop && iters < A.max_iter) {
#pragma unroll
            for (int k = 0; k < NC; ++k) {
                p[k] = r[k] + beta * (p[k] - omega * v[k]);
                hp[k] = hr[k] + beta * (hp[k] - omega * hv[k]);
                a_[k] = dinv[k] * p[k];
                ha_[k] = hdinv[k] * hp[k];
            }
            product(a_, ha_, v);
            q[0] = q[1] = 0.0;
#pragma unroll
            for (int k = 0; k < NC; ++k) {
                q[0] += rh[k] * v[k];
                q[1] += r[k] * r[k];
            }
            ok = exchange(v, q, NoSums{}, hv);
            if (!ok) break;
            // converged by the recurrence: checked against the true residual
            if (tot[1] <= tol2b2) break;
            const double rv = tot[0];
            if (rv == 0.0 || !isfinite(rv) || !isfinite(tot[1])) break;  // breakdown: restart
            alpha = rho / rv;
#pragma unroll
            for (int k = 0; k < NC; ++k) {
                sv[k] = r[k] - alpha * v[k];
                hs[k] = hr[k] - alpha * hv[k];
                a_[k] = dinv[k] * sv[k];
                ha_[k] = hdinv[k] * hs[k];
            }
            product(a_, ha_, t);
            q[0] = q[1] = 0.0;
            Sum2 q2[2] = {};
#pragma unroll
            for (int k = 0; k < NC; ++k) {
                q[0] += t[k] * sv[k];
                q[1] += t[k] * t[k];
                mul_add2(q2[0], rh[k], sv[k]);
                mul_add2(q2[1], rh[k], t[k]);
            }
            double ht[NC];
            ok = exchange(t, q, q2, ht);
            if (!ok) break;
            omega = tot[1] > 0.0 ? tot[0] / tot[1] : 0.0;
#pragma unroll
            for (int k = 0; k < NC; ++k) {
                x[k] += dinv[k] * (alpha * p[k] + omega * sv[k]);
                r[k] = sv[k] - omega * t[k];
                hr[k] = hs[k] - omega * ht[k];
            }
            ++iters;
            const double rho1 = value2(sub_scaled2(tot2[0], omega, tot2[1]));
            if (omega == 0.0 || rho1 == 0.0 || !isfinite(rho1)) stop = true;
            else {
                beta = (rho1 / rho) * (alpha / omega);
                rho = rho1;
            }
        }
        if (!ok) break;
        // dA on the halo for the next true residual
        q[0] = q[1] = 0.0;
        ok = exchange(x, q, NoSums{}, hx);
    }
#pragma unroll
    for (int k = 0; k < NC; ++k)
        if (gi[k] >= 0) A.x[gi[k]] = x[k];
    if (g == 0 && tid == 0) {
        A.st[S_TOL2B2] = b2;  // the host divides by b.b
        A.st[S_R2] = true_r2;
        A.st[S_EMPTY] = empty;
        A.st[S_ITERS] = (double)iters;
        A.st[S_DONE] = ok && done != 0 ? (double)done : 2.0;
    }
}

// w_p += dA of its cell; nothing when st says that the solve is not the answer
__global__ void k_apply_dA(double* w, const int64_t* off, const double* dA, const double* st)
{
    if (st && (st[S_EMPTY] != 0.0 || st[S_DONE] == 2.0)) return;
    const int c = blockIdx.x;
    const int64_t o0 = off[c], n = off[c + 1] - o0;
    const double d = dA[c];
    for (int64_t i = threadIdx.x; i < n; i += blockDim.x) w[o0 + i] += d;
}

}  // namespace gm

namespace {

constexpr size_t al256(size_t x) { return (x + 255) & ~(size_t)255; }

struct GaussWs {
    double *colM, *colW, *dinv, *b, *x, *r, *rh, *p, *v, *s, *t, *partial, *st;
    size_t total;
};

int64_t vec_blocks(int64_t n_cells) { return (n_cells + gm::kVecThreads - 1) / gm::kVecThreads; }

unsigned stencil_blocks(int64_t n_cells)
{
    const int64_t per = gm::kStencilThreads / 64;
    return (unsigned)((n_cells + per - 1) / per);
}

GaussWs gauss_layout(int64_t n_cells, int dx, char* base)
{
    GaussWs g;
    const size_t n = (size_t)n_cells, ns = dx == 1 ? 3 : 9;
    size_t o = 0;
    auto take = [&](size_t bytes) {
        double* ptr = base ? (double*)(base + o) : nullptr;
        o += al256(bytes);
        return ptr;
    };
    g.colM = take(n * ns * 8);
    g.colW = take(n * ns * 8);
    g.dinv = take(n * 8);
    g.b = take(n * 8);
    g.x = take(n * 8);
    g.r = take(n * 8);
    g.rh = take(n * 8);
    g.p = take(n * 8);
    g.v = take(n * 8);
    g.s = take(n * 8);
    g.t = take(n * 8);
    g.partial = take((size_t)vec_blocks(n_cells) * 2 * 8);
    g.st = take(gm::S_COUNT * 8);
    g.total = o;
    return g;
}

bool mesh_ok(int64_t n_cells, int dx, int nx)
{
    if (n_cells < 1 || n_cells > 0x7fffffff) return false;
    if (dx == 1) return nx == n_cells || nx <= 0;
    if (dx == 2) return nx >= 1 && n_cells % nx == 0;
    return false;
}

// iterations enqueued between two reads of the solver state
constexpr int kChunk = 8;
// restarts from the true residual before the solve gives up
constexpr int kMaxRestarts = 8;

// The one-launch solves of the process at once, per device: their workgroups
// together take at most a CU each, so none keeps part of another's grid out.
// A call holds its places until its solve has ended.
constexpr int kMaxDevices = 64;
std::atomic<int> g_solve_held[kMaxDevices];

// a device attribute, looked up once per device; 0 if it cannot be had
int device_attribute(std::atomic<int> (&known)[kMaxDevices], hipDeviceAttribute_t which, int dev)
{
    int x = known[dev].load(std::memory_order_relaxed);
    if (x == 0 && hipDeviceGetAttribute(&x, which, dev) == hipSuccess) known[dev].store(x, std::memory_order_relaxed);
    return x;
}
std::atomic<int> g_cus[kMaxDevices], g_clock_khz[kMaxDevices];

struct SolvePlaces {
    int dev = -1, held = 0, khz = 0;  // khz: of the device's wall clock
    // `groups` places of the device's CUs, or of `places` where that is not
    // negative; false if they are not free
    bool take(int groups, int places)
    {
        if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return false;
        int cus = device_attribute(g_cus, hipDeviceAttributeMultiprocessorCount, dev);
        khz = device_attribute(g_clock_khz, hipDeviceAttributeWallClockRate, dev);
        if (khz <= 0) return false;
        if (places >= 0 && places < cus) cus = places;
        held = groups;
        if (g_solve_held[dev].fetch_add(groups) + groups <= cus) return true;
        release();
        return false;
    }
    void release()
    {
        if (held) g_solve_held[dev].fetch_sub(held);
        held = 0;
    }
    ~SolvePlaces() { release(); }
};

template <int DX>
int gauss_correct_impl(const double* x, double* w, const int64_t* off, int64_t n, int nx, int ny,
                       const double* target, double tol, int max_iter, const GaussWs& g, hipStream_t st,
                       int32_t* iters_out, double* resid_out, gm_gauss_diag* diag)
{
    using namespace gm;
    int ignored = 0;
    int32_t& path = diag ? diag->path : ignored;
    path = 0;
    const unsigned nb = (unsigned)vec_blocks(n);
    const dim3 vb(kVecThreads);
    double hs[S_COUNT];
    auto read_state = [&]() -> bool {
        if (hipGetLastError() != hipSuccess) return false;
        if (hipMemcpyAsync(hs, g.st, sizeof(hs), hipMemcpyDeviceToHost, st) != hipSuccess) return false;
        return hipStreamSynchronize(st) == hipSuccess;
    };
    auto fold = [&](int mode) {
        hipLaunchKernelGGL(k_fold, dim3(1), vb, 0, st, g.partial, (int)nb, g.st, mode, tol);
    };
    // The one-launch solve: rows that fit a workgroup with their halo, and a
    // mesh that a resident grid covers (131072 cells; at 65536, half of that,
    // it takes 0.36 of the other path's time, and at one workgroup a quarter).
    // Longer rows and larger meshes are launched step by step.
    const int per = DX == 1 ? kSolveOwn : (nx <= kSolveHalo ? kSolveOwn / nx : 0);
    const int64_t ngroups = per > 0 ? ((DX == 1 ? n : (int64_t)ny) + per - 1) / per : 0;
    SolvePlaces place;
    const bool one_launch =
        per > 0 && ngroups <= kSolveMaxGroups && place.take((int)ngroups, diag ? diag->places : -1);
    const int groups = one_launch ? (int)ngroups : 0;
    hipLaunchKernelGGL(k_stencil<DX>, dim3(stencil_blocks(n)), dim3(kStencilThreads), 0, st, x, w, off, n, g.colM,
                       g.colW, (unsigned long long*)g.t, one_launch ? 2 * groups : 0);
    if (one_launch) {
        SolveArgs a;
        a.colM = g.colM;
        a.colW = g.colW;
        a.target = target;
        a.off = off;
        a.n = n;
        a.nx = nx;
        a.ny = ny;
        a.per = per;
        a.tol = tol;
        a.max_iter = max_iter;
        a.max_restarts = kMaxRestarts;
        a.wait = (long long)place.khz * (diag && diag->wait_us >= 0 ? diag->wait_us : kSolveWaitUs) / 1000;
        a.x = g.x;
        a.halo[0] = g.p;
        a.halo[1] = g.v;
        a.part = g.s;  // 128 B per group: the vector holds 8 B per cell, at least 256 in all
        a.tag = (unsigned long long*)g.t;
        a.st = g.st;
        hipLaunchKernelGGL(k_solve<DX>, dim3(groups), dim3(kSolveThreads), 0, st, a);
        hipLaunchKernelGGL(k_apply_dA, dim3((unsigned)n), dim3(256), 0, st, w, off, g.x, g.st);
        path = 1;
        if (!read_state()) return GM_EHIP;
        place.release();
        if (hs[S_EMPTY] != 0.0) return GM_EINVAL;  // a cell without particles: M is singular
        const double rel = hs[S_TOL2B2] > 0.0 ? std::sqrt(hs[S_R2] / hs[S_TOL2B2]) : 0.0;
        if ((hs[S_DONE] == 1.0 || hs[S_DONE] == 3.0) && std::isfinite(rel)) {
            if (iters_out) *iters_out = (int)hs[S_ITERS];
            if (resid_out) *resid_out = rel;
            return hs[S_DONE] == 1.0 ? GM_OK : GM_ENOCONV;
        }
        path = 2;
    }
    hipLaunchKernelGGL(k_setup<DX>, dim3(nb), vb, 0, st, g.colM, g.colW, target, off, n, nx, ny, g.dinv, g.b, g.x,
                       g.partial);
    fold(E_INIT);
    if (!read_state()) return GM_EHIP;
    if (hs[S_EMPTY] != 0.0) return GM_EINVAL;  // a cell without particles: M is singular
    const double b2 = hs[S_R2];
    bool converged = hs[S_DONE] == 1.0;
    int iters = 0;
    double r2 = b2;
    for (int rs = 0; !converged && rs <= kMaxRestarts; ++rs) {
        // the true residual of the current dA decides convergence
        hipLaunchKernelGGL(k_restart<DX>, dim3(nb), vb, 0, st, g.colM, g.b, g.x, n, nx, ny, g.r, g.rh, g.p, g.v,
                           g.partial);
        fold(E_RESTART);
        if (!read_state()) return GM_EHIP;
        r2 = hs[S_R2];
        if (hs[S_DONE] == 1.0) {
            converged = true;
            break;
        }
        if (hs[S_DONE] != 0.0 || iters >= max_iter) break;
        while (iters < max_iter) {
            const int k = max_iter - iters < kChunk ? max_iter - iters : kChunk;
            for (int it = 0; it < k; ++it) {
                hipLaunchKernelGGL(k_update_p, dim3(nb), vb, 0, st, g.st, g.r, g.v, g.p, n);
                hipLaunchKernelGGL((k_spmv<DX, false>), dim3(nb), vb, 0, st, g.st, g.colM, g.dinv, g.p, g.rh, n, nx,
                                   ny, g.v, g.partial);
                fold(E_ALPHA);
                hipLaunchKernelGGL(k_update_s, dim3(nb), vb, 0, st, g.st, g.r, g.v, g.s, n);
                hipLaunchKernelGGL((k_spmv<DX, true>), dim3(nb), vb, 0, st, g.st, g.colM, g.dinv, g.s, g.rh, n, nx,
                                   ny, g.t, g.partial);
                fold(E_OMEGA);
                hipLaunchKernelGGL(k_update_xr, dim3(nb), vb, 0, st, g.st, g.dinv, g.p, g.s, g.t, g.rh, g.x, g.r, n,
                                   g.partial);
                fold(E_RES_RHO);
            }
            if (!read_state()) return GM_EHIP;
            iters = (int)hs[S_ITERS];  // iterations since the start, over every restart
            if (hs[S_DONE] != 0.0) break;
        }
    }
    hipLaunchKernelGGL(k_apply_dA, dim3((unsigned)n), dim3(256), 0, st, w, off, g.x, (const double*)nullptr);
    if (hipGetLastError() != hipSuccess) return GM_EHIP;
    const double rel = b2 > 0.0 ? std::sqrt(r2 / b2) : 0.0;
    if (iters_out) *iters_out = iters;
    if (resid_out) *resid_out = rel;
    return converged && std::isfinite(rel) ? GM_OK : GM_ENOCONV;
}

}  // namespace

extern "C" {

size_t gm_gauss_workspace(int64_t n_cells, int32_t dx)
{
    if (!mesh_ok(n_cells, dx, dx == 1 ? (int)n_cells : 1)) return 0;
    return gauss_layout(n_cells, dx, nullptr).total;
}

int gm_deposit(const double* x, const double* w, const int64_t* cell_off, int64_t n_cells, int32_t dx, int32_t nx,
               double* dep, void* ws, size_t ws_bytes, void* stream)
{
    using namespace gm;
    if (!mesh_ok(n_cells, dx, nx)) return GM_EINVAL;
    if (!x || !w || !cell_off || !dep) return GM_EINVAL;
    GaussWs g = gauss_layout(n_cells, dx, (char*)ws);
    if (!ws || ws_bytes < g.total) return GM_ENOMEM;
    hipStream_t st = (hipStream_t)stream;
    const int NX = dx == 1 ? (int)n_cells : nx, NY = dx == 1 ? 1 : (int)(n_cells / nx);
    const unsigned nb = (unsigned)vec_blocks(n_cells);
    if (dx == 1) {
        hipLaunchKernelGGL(k_stencil<1>, dim3(stencil_blocks(n_cells)), dim3(kStencilThreads), 0, st, x, w,
                           cell_off, n_cells, nullptr, g.colW, (unsigned long long*)nullptr, 0);
        hipLaunchKernelGGL(k_deposit<1>, dim3(nb), dim3(kVecThreads), 0, st, g.colW, n_cells, NX, NY, dep);
    } else {
        hipLaunchKernelGGL(k_stencil<2>, dim3(stencil_blocks(n_cells)), dim3(kStencilThreads), 0, st, x, w,
                           cell_off, n_cells, nullptr, g.colW, (unsigned long long*)nullptr, 0);
        hipLaunchKernelGGL(k_deposit<2>, dim3(nb), dim3(kVecThreads), 0, st, g.colW, n_cells, NX, NY, dep);
    }
    return hipGetLastError() == hipSuccess ? GM_OK : GM_EHIP;
}

int gm_gauss_correct_diag(const double* x, double* w, const int64_t* cell_off, int64_t n_cells, int32_t dx,
                          int32_t nx, const double* dep_target, double tol, int32_t max_iter, void* ws,
                          size_t ws_bytes, void* stream, int32_t* iters_out, double* resid_out, gm_gauss_diag* diag)
{
    if (!mesh_ok(n_cells, dx, nx) || !(tol > 0.0) || !(tol < 1.0) || max_iter < 1) return GM_EINVAL;
    if (!x || !w || !cell_off || !dep_target) return GM_EINVAL;
    GaussWs g = gauss_layout(n_cells, dx, (char*)ws);
    if (!ws || ws_bytes < g.total) return GM_ENOMEM;
    hipStream_t st = (hipStream_t)stream;
    const int NX = dx == 1 ? (int)n_cells : nx, NY = dx == 1 ? 1 : (int)(n_cells / nx);
    if (dx == 1)
        return gauss_correct_impl<1>(x, w, cell_off, n_cells, NX, NY, dep_target, tol, max_iter, g, st, iters_out,
                                     resid_out, diag);
    return gauss_correct_impl<2>(x, w, cell_off, n_cells, NX, NY, dep_target, tol, max_iter, g, st, iters_out,
                                 resid_out, diag);
}

int gm_gauss_correct(const double* x, double* w, const int64_t* cell_off, int64_t n_cells, int32_t dx, int32_t nx,
                     const double* dep_target, double tol, int32_t max_iter, void* ws, size_t ws_bytes, void* stream,
                     int32_t* iters_out, double* resid_out)
{
    return gm_gauss_correct_diag(x, w, cell_off, n_cells, dx, nx, dep_target, tol, max_iter, ws, ws_bytes, stream,
                                 iters_out, resid_out, nullptr);
}

}  // extern "C"
