// Pressure Poisson solver: preconditioned conjugate gradients on the
// singular, symmetric operator L = -A, A P = sum_d delta_1 delta_1 P (the
// discrete continuity constraint Eq 3.24 with the face flux of Eq 3.23;
// zero flux through non-periodic sides, section 3.3). The preconditioner is
// one symmetric geometric multigrid V-cycle: red-black Gauss-Seidel
// (red-black down, black-red up), 2^d-cell averaging restriction,
// piecewise-constant prolongation, rediscretised coarse operators and an
// exact pseudo-inverse on the coarsest grid, so the zero-mean solution is
// obtained as with the augmented-matrix method the paper uses. The V-cycle
// runs in FP64, or in FP32 (mixed modes) with FP64 residuals, operator,
// updates and dot products.
//
// CG. Single-reduction CG (Chronopoulos-Gear: one global reduction per
// iteration) in FP64 and in the default mixed mode. On 2D tiles the V-cycle
// stores w = A u on the finest level and s = A p is carried by recurrence;
// elsewhere neither is stored and the update forms A p from p. Flexible CG
// (Polak-Ribiere beta, q = A p stored) in the flexible mixed mode. Scalars
// never leave the device. A reduction kernel writes one
// partial sum per block; the next kernel that needs the total has every
// block sum those partials in the same fixed order (no atomics, no grid-wide
// fences, bitwise reproducible). The convergence test runs on the device and
// raises a flag that turns every later kernel into an immediate return; the
// host queues the expected iterations and reads the flag while the device
// goes on with the work behind the solve, gated on its outcome.
//
// Levels. 2D levels that a tile fits run one LDS tile
// kernel per level and direction with temporal blocking (nu red-black sweeps
// from a zero guess, residual and restriction on the way down; prolongation
// and nu black-red sweeps on the way up; on the finest level also the CG
// update, w = A u and the CG partial sums). Periodic 3D levels with beta = 1
// run the z-marching equivalent (lm_mg3d.h). Levels of at most kCoarseCells
// cells are solved by one workgroup (lm_coarse.h); the remaining levels run
// one kernel per half-sweep.
#include <hip/hip_ext.h>

#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "lm_device.h"

namespace lm {

constexpr int kRedBlocks = 1024;   // grid of the grid-stride reduction kernels
// 2D tiles of the fused multigrid kernels: 64 x 16 preferred on the finest
// level (bandwidth), 32 x 8 below it (latency bound: shorter phases), 16 x 16
// for sizes that neither divides.
constexpr int TX = 64, TY = 16;
constexpr int TXS = 32, TYS = 8;

Lay make_layout(int ndim, const int n[3], int elem_bytes) {
  Lay L;
  L.ndim = ndim;
  const int align = 128 / elem_bytes;  // elements per 128-byte line
  for (int d = 0; d < 3; ++d) L.n[d] = d < ndim ? n[d] : 1;
  const long px = ((long)(L.n[0] + 2) + align - 1) / align * align;
  const long py = L.n[1] + 2;
  L.s[0] = 1;
  L.s[1] = px;
  L.s[2] = ndim == 3 ? px * py : 0;
  const long planes = ndim == 3 ? L.n[2] + 2 : 1;
  long b0 = 1 + px + (ndim == 3 ? L.s[2] : 0);
  const long shift = (align - (b0 % align)) % align;
  L.base = b0 + shift;
  L.total = shift + px * py * planes + align;
  return L;
}

// ---------------------------------------------------------------------------
// Small device helpers
// ---------------------------------------------------------------------------

// v plus the value a DPP control moves to this lane (0 where it moves none).
template <int CTRL, int ROWS>
__device__ inline double dpp_add(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(b & 0xffffffffLL), CTRL, ROWS, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, ROWS, 0xf, true);
  return v + __longlong_as_double(((long long)hi << 32) | (long long)(unsigned)lo);
}
__device__ inline double lane_value(double v, int lane) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)(unsigned)(b & 0xffffffffLL), lane);
  const int hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
  return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned)lo);
}
// Sum over the first 16 lanes / the whole wavefront, in every lane: row
// shifts, then row broadcasts, in the vector unit (a shuffle goes through
// LDS: six dependent round trips per sum). All lanes active.
__device__ inline double row_sum16(double v) {
  v = dpp_add<0x111, 0xf>(v);
  v = dpp_add<0x112, 0xf>(v);
  v = dpp_add<0x114, 0xf>(v);
  v = dpp_add<0x118, 0xf>(v);
  return v;  // lane 15 of each row holds the row's sum
}
__device__ inline double wave_sum(double v) {
  v = row_sum16(v);
  v = dpp_add<0x142, 0xa>(v);  // row_bcast:15 into rows 1 and 3
  v = dpp_add<0x143, 0xc>(v);  // row_bcast:31 into rows 2 and 3
  return lane_value(v, 63);
}

// Block-wide sums of NV values (at most 1024 threads, whole wavefronts),
// identical in every thread: wavefront sums, one exchange through LDS, then
// every wavefront adds the per-wavefront sums in the same order.
template <int NV>
__device__ inline void block_allsum_n(double (&v)[NV]) {
  __shared__ double shn[NV][16];
#pragma unroll
  for (int q = 0; q < NV; ++q) v[q] = wave_sum(v[q]);
  const int t = linear_tid();
  const int nw = (blockDim.x * blockDim.y * blockDim.z + 63) / 64;
  __syncthreads();  // an earlier call may still be reading shn
  if ((t & 63) == 0) {
#pragma unroll
    for (int q = 0; q < NV; ++q) shn[q][t >> 6] = v[q];
  }
  __syncthreads();
  if (nw <= 4) {
#pragma unroll
    for (int q = 0; q < NV; ++q) {
      double s = 0.0;
      for (int w = 0; w < nw; ++w) s += shn[q][w];
      v[q] = s;
    }
  } else {
    const int lane = t & 15;
#pragma unroll
    for (int q = 0; q < NV; ++q) v[q] = lane_value(row_sum16(lane < nw ? shn[q][lane] : 0.0), 15);
  }
}

// This thread's share of the sum of np partials: loads issued four at a
// time so their latencies overlap.
__device__ inline double partial_share(const double *part, int np) {
  const int t = linear_tid();
  const int nt = blockDim.x * blockDim.y * blockDim.z;
  double s = 0.0;
  for (int q0 = 0; q0 < np; q0 += 4 * nt) {
    double v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int q = q0 + u * nt + t;
      v[u] = part[q < np ? q : 0];
      if (q >= np) v[u] = 0.0;
    }
    s += (v[0] + v[1]) + (v[2] + v[3]);
  }
  return s;
}

// Sum of np partials, identical in every block and thread.
__device__ inline double sum_all(const double *part, int np, double *) {
  double v[1] = {partial_share(part, np)};
  block_allsum_n<1>(v);
  return v[0];
}

// Sums of three partial arrays of np entries each (one combined pass).
__device__ inline void sum_all3(const double *p0, const double *p1, const double *p2, int np, double *,
                                double &s0, double &s1, double &s2) {
  double v[3] = {partial_share(p0, np), partial_share(p1, np), p2 ? partial_share(p2, np) : 0.0};
  block_allsum_n<3>(v);
  s0 = v[0];
  s1 = v[1];
  s2 = v[2];
}

// ||c||^2 (the partials of the solve's right-hand side on the first
// iteration, the value stored by block 0 afterwards) together with the
// three sums of sum_all3, in one pass.
__device__ inline void sum_cc3(int k, const double *part_cc, int np_cc, const SolverScalars *sc, const double *p0,
                               const double *p1, const double *p2, int np, double &cc, double &s0, double &s1,
                               double &s2) {
  if (k == 1) {
    double v[4] = {partial_share(part_cc, np_cc), partial_share(p0, np), partial_share(p1, np),
                   p2 ? partial_share(p2, np) : 0.0};
    block_allsum_n<4>(v);
    cc = v[0];
    s0 = v[1];
    s1 = v[2];
    s2 = v[3];
  } else {
    cc = sc->cc;
    double v[3] = {partial_share(p0, np), partial_share(p1, np), p2 ? partial_share(p2, np) : 0.0};
    block_allsum_n<3>(v);
    s0 = v[0];
    s1 = v[1];
    s2 = v[2];
  }
}

template <int DIM>
__device__ inline void decode(const Lay &L, long t, int &i, int &j, int &k);

// Grid-stride loops run over 64 x 4 tiles of cells (one wavefront per row):
// one 32-bit division per tile instead of per cell.
__device__ inline int ntiles_of(const Lay &L) { return ((L.n[0] + 63) >> 6) * ((L.n[1] + 3) >> 2) * L.n[2]; }

__device__ inline bool tile_cell(const Lay &L, int tile, int &i, int &j, int &k) {
  const int tx = (L.n[0] + 63) >> 6, ty = (L.n[1] + 3) >> 2;
  const int txy = tx * ty;
  k = tile / txy;
  const int rem = tile - k * txy;
  const int y = rem / tx;
  const int x = rem - y * tx;
  i = (x << 6) + (threadIdx.x & 63);
  j = (y << 2) + (threadIdx.x >> 6);
  return i < L.n[0] && j < L.n[1];
}

template <int DIM>
__device__ inline void decode(const Lay &L, long t, int &i, int &j, int &k) {
  i = (int)(t % L.n[0]);
  j = (int)((t / L.n[0]) % L.n[1]);
  k = DIM == 3 ? (int)(t / ((long)L.n[0] * L.n[1])) : 0;
}

// Neighbour sum and diagonal of L = -A at one cell (periodic wrap, zero
// flux through non-periodic sides).
template <int DIM, typename A, typename T>
__device__ inline void op_parts(const Lay &L, const Bnd &B, const A ih2[3], const T *x, int i, int j, int k,
                                long c, A &nbsum, A &diag) {
  nbsum = A(0);
  diag = A(0);
  const int q[3] = {i, j, k};
#pragma unroll
  for (int d = 0; d < DIM; ++d) {
    A s = A(0);
    int cnt = 0;
    const long lo = (q[d] > 0) ? c - L.s[d] : (B.periodic[d] ? c + (long)(L.n[d] - 1) * L.s[d] : -1);
    const long hi = (q[d] + 1 < L.n[d]) ? c + L.s[d] : (B.periodic[d] ? c - (long)(L.n[d] - 1) * L.s[d] : -1);
    if (lo >= 0) {
      s += (A)x[lo];
      ++cnt;
    }
    if (hi >= 0) {
      s += (A)x[hi];
      ++cnt;
    }
    nbsum += ih2[d] * s;
    diag += ih2[d] * (A)cnt;
  }
}

template <typename T>
struct Ih2 {
  T v[3];
};

// Face coefficient of the variable-coefficient operator: beta = 1/rho_f
// with rho_f = (rho_a + rho_b)/2 the two-point face average (Eq 3.20,
// n = 1). Symmetric in its arguments bit for bit.
template <typename T>
__device__ inline T face_beta(T ra, T rb) {
  return T(2) / (ra + rb);
}

// Face coefficient along direction d. On a stretched 2D grid (met) the
// volume-weighted operator dV A has, on an x-face, dy / (distance between
// the two centres) = 2 / (dx_a/dy + dx_b/dy), i.e. face_beta of the cell
// ratio dx/dy, and on a y-face face_beta of dy/dx: the cell array holds
// dx/dy and y-faces take its reciprocals.
template <typename T>
__device__ inline T face_coef(T ra, T rb, int d, int met) {
  if (met && d == 1) return face_beta<T>(T(1) / ra, T(1) / rb);
  return face_beta<T>(ra, rb);
}

// Neighbour sum and diagonal of L = -A_beta at one cell, beta = 1/rho_f
// (same neighbour rules as op_parts).
template <int DIM, typename A, typename T, typename R>
__device__ inline void op_parts_vc(const Lay &L, const Bnd &B, const A ih2[3], const R *rho, const T *x, int i, int j,
                                   int k, long c, A &nbsum, A &diag, int met = 0) {
#pragma clang fp contract(off)
  nbsum = A(0);
  diag = A(0);
  const int q[3] = {i, j, k};
  const A rc = (A)rho[c];
#pragma unroll
  for (int d = 0; d < DIM; ++d) {
    A s = A(0), sb = A(0);
    const long lo = (q[d] > 0) ? c - L.s[d] : (B.periodic[d] ? c + (long)(L.n[d] - 1) * L.s[d] : -1);
    const long hi = (q[d] + 1 < L.n[d]) ? c + L.s[d] : (B.periodic[d] ? c - (long)(L.n[d] - 1) * L.s[d] : -1);
    if (lo >= 0) {
      const A bt = face_coef<A>(rc, (A)rho[lo], d, met);
      s += bt * (A)x[lo];
      sb += bt;
    }
    if (hi >= 0) {
      const A bt = face_coef<A>(rc, (A)rho[hi], d, met);
      s += bt * (A)x[hi];
      sb += bt;
    }
    nbsum += ih2[d] * s;
    diag += ih2[d] * sb;
  }
}


// ---------------------------------------------------------------------------
// CG kernels (FP64 vectors on the fine layout, grid-stride over cells)
// ---------------------------------------------------------------------------
struct CGArgs {
  Lay L;
  Bnd B;
  double ih2[3], ih[3];
  const double *b, *x0;
  double *x;
  double *rold, *rnew;    // r_{k-1}, r_k
  double *pold, *pnew;    // p_{k-1}, p_k
  double *q;
  const void *z, *zold;   // z_{k-1}, z_{k-2} (flexible)
  double *part_cc, *part_pq, *part_rz;  // part_rz: [rz | rr | rzo] x np_rz
  int np_rz, np_pq;
  SolverScalars *sc;
  double tol2;
  int k;
  int flexible;
  const double *rho;      // density of beta = 1/rho_f; NULL: beta = 1
  int met = 0;                   // stretched 2D grid: rho holds dx/dy (face_coef)
  const double *vol = nullptr;   // stretched: cell volumes (the right-hand side is dV b)
};

// x = x0; r_0 = c - L x0 with c = -(b - mean(b) - outflow shift); ||c||^2
// partials, one per block (one thread per cell: the stencil of x0 reads
// planes a patch plane apart, still in L2).
template <int DIM>
__global__ void __launch_bounds__(kBlock) k_cg_init(CGArgs a, double *partials) {
  __shared__ double sh[kBlock / 64];
  SolverScalars *sc = a.sc;
  if (a.rho && sc->rho_bad) {  // invalid density: the solve ends at once
    if (linear_block() == 0 && linear_tid() == 0) {
      sc->done = 1;
      sc->nonconv = 1;
    }
    return;
  }
  double cc = 0.0;
  CellPos p;
  if (cell_of_thread(a.L, p)) {
    const int i = p.i, j = p.j, k = p.k;
    const long c = p.c;
    const double mb = sc->mean_b, oc = sc->outflow_c;
    const double xv = a.x0 ? a.x0[c] : 0.0;
    a.x[c] = xv;
    double bb = a.b[c] - mb;
    const int q[3] = {i, j, k};
#pragma unroll
    for (int d = 0; d < DIM; ++d) {
      if (a.B.kind[d][0] == LM_SIDE_OUTFLOW && q[d] == 0) bb -= oc * a.ih[d];
      if (a.B.kind[d][1] == LM_SIDE_OUTFLOW && q[d] == a.L.n[d] - 1) bb -= oc * a.ih[d];
    }
    const double cv = a.vol ? -(bb * a.vol[c]) : -bb;  // stretched: dV (b - mean)
    double Lx = 0.0;
    if (a.x0) {
      double nbs, dg;
      if (a.rho)
        op_parts_vc<DIM, double, double, double>(a.L, a.B, a.ih2, a.rho, a.x0, i, j, k, c, nbs, dg, a.met);
      else
        op_parts<DIM, double, double>(a.L, a.B, a.ih2, a.x0, i, j, k, c, nbs, dg);
      Lx = dg * xv - nbs;
    }
    a.rnew[c] = cv - Lx;
    cc = cv * cv;
  }
  const double s = block_sum(cc, sh);
  if (linear_tid() == 0) partials[linear_block()] = s;
}

// Folds nb per-block partials into gridDim.x partials, each the fixed-order
// sum of a contiguous run.
__global__ void __launch_bounds__(kBlock) k_fold_partials(const double *in, long nb, double *out) {
  __shared__ double sh[kBlock / 64];
  const long per = (nb + gridDim.x - 1) / gridDim.x;
  const long q0 = (long)blockIdx.x * per, q1 = q0 + per < nb ? q0 + per : nb;
  double s = 0.0;
  for (long q = q0 + threadIdx.x; q < q1; q += blockDim.x) s += in[q];
  const double t = block_sum(s, sh);
  if (threadIdx.x == 0) out[blockIdx.x] = t;
}

// Whether the solve ended before the kernel that makes the test of step k.
// Its block 0 sets sc->done while other blocks are starting, so done is
// k + 1, not merely nonzero: a block that starts late still makes the test
// itself, with every wavefront. (With a plain flag the wavefronts of one
// block can read it on either side of the store, and those that go on would
// add up the partials without the others' shares.)
__device__ inline bool ended_before(const SolverScalars *sc, int k) {
  const int done = sc->done;
  return done && done != k + 1;
}

// Convergence test on r_{k-1}; beta_k; p_k = z_{k-1} + beta_k p_{k-1};
// q = L p_k; partials of p_k.q.
template <int DIM, typename TZ>
__global__ void __launch_bounds__(kBlock) k_cg_pq(CGArgs a, int np_cc) {
  __shared__ double sh[kBlock / 64];
  SolverScalars *sc = a.sc;
  const int k = a.k;
  if (ended_before(sc, k)) return;
  double cc, rz, rr, rzo;
  sum_cc3(k, a.part_cc, np_cc, sc, a.part_rz, a.part_rz + a.np_rz, a.flexible ? a.part_rz + 2 * a.np_rz : nullptr,
          a.np_rz, cc, rz, rr, rzo);
  const bool converged = (cc == 0.0) || (rr <= a.tol2 * cc);
  const bool broken = !isfinite(rr) || !isfinite(rz);
  double beta = 0.0;
  if (k > 1) beta = (a.flexible ? rz - rzo : rz) / sc->rzh[(k - 2) & 1];
  if (linear_block() == 0 && linear_tid() == 0) {
    sc->rzh[(k - 1) & 1] = rz;
    sc->rr = rr;
    sc->cc = cc;
    sc->iters = k - 1;
    if (converged || broken) {
      sc->zero = (cc == 0.0);
      sc->nonconv = broken && !converged;
      sc->done = k + 1;
    }
  }
  if (converged || broken) return;
  const TZ *z = (const TZ *)a.z;
  double pq = 0.0;
  for (int tile = blockIdx.x; tile < ntiles_of(a.L); tile += gridDim.x) {
    int i, j, kk;
    if (!tile_cell(a.L, tile, i, j, kk)) continue;
    const long c = a.L.at(i, j, kk);
    auto pv = [&](long m) -> double { return k > 1 ? (double)z[m] + beta * a.pold[m] : (double)z[m]; };
    const double pc = pv(c);
    double nbs = 0.0, dg = 0.0;
    const int q[3] = {i, j, kk};
#pragma unroll
    for (int d = 0; d < DIM; ++d) {
      double s = 0.0, sb = 0.0;
      const long lo = (q[d] > 0) ? c - a.L.s[d] : (a.B.periodic[d] ? c + (long)(a.L.n[d] - 1) * a.L.s[d] : -1);
      const long hi = (q[d] + 1 < a.L.n[d]) ? c + a.L.s[d]
                                            : (a.B.periodic[d] ? c - (long)(a.L.n[d] - 1) * a.L.s[d] : -1);
      if (lo >= 0) {
        const double bt = a.rho ? face_coef<double>(a.rho[c], a.rho[lo], d, a.met) : 1.0;
        s += bt * pv(lo);
        sb += bt;
      }
      if (hi >= 0) {
        const double bt = a.rho ? face_coef<double>(a.rho[c], a.rho[hi], d, a.met) : 1.0;
        s += bt * pv(hi);
        sb += bt;
      }
      nbs += a.ih2[d] * s;
      dg += a.ih2[d] * sb;
    }
    const double qv = dg * pc - nbs;
    a.pnew[c] = pc;
    a.q[c] = qv;
    pq += pc * qv;
  }
  const double s = block_sum(pq, sh);
  if (linear_tid() == 0) a.part_pq[blockIdx.x] = s;
}

// alpha_k = rho_{k-1}/(p_k.q); x += alpha p_k; r_k = r_{k-1} - alpha q.
template <int DIM>
__global__ void __launch_bounds__(kBlock) k_cg_update(CGArgs a) {
  __shared__ double sh[kBlock / 64];
  SolverScalars *sc = a.sc;
  if (sc->done) return;
  const double pq = sum_all(a.part_pq, a.np_pq, sh);
  const double alpha = sc->rzh[(a.k - 1) & 1] / pq;
  for (int tile = blockIdx.x; tile < ntiles_of(a.L); tile += gridDim.x) {
    int i, j, k;
    if (!tile_cell(a.L, tile, i, j, k)) continue;
    const long c = a.L.at(i, j, k);
    a.x[c] += alpha * a.pnew[c];
    a.rnew[c] = a.rold[c] - alpha * a.q[c];
  }
}

// Partials of r.z, r.r (and r.z_old) for the unfused finest level.
template <int DIM, typename TZ>
__global__ void __launch_bounds__(kBlock) k_cg_rz(CGArgs a) {
  SolverScalars *sc = a.sc;
  if (sc->done) return;
  const TZ *z = (const TZ *)a.z;
  const TZ *zo = (const TZ *)a.zold;
  double rz = 0.0, rr = 0.0, rzo = 0.0;
  for (int tile = blockIdx.x; tile < ntiles_of(a.L); tile += gridDim.x) {
    int i, j, k;
    if (!tile_cell(a.L, tile, i, j, k)) continue;
    const long c = a.L.at(i, j, k);
    const double rv = a.rnew[c];
    rz += rv * (double)z[c];
    rr += rv * rv;
    if (zo) rzo += rv * (double)zo[c];
  }
  double v3[3] = {rz, rr, rzo};  // rzo stays 0 without z_old
  block_allsum_n<3>(v3);
  if (linear_tid() == 0) {
    a.part_rz[blockIdx.x] = v3[0];
    a.part_rz[a.np_rz + blockIdx.x] = v3[1];
    a.part_rz[2 * a.np_rz + blockIdx.x] = v3[2];
  }
}

// Single-reduction CG (Chronopoulos-Gear) on a finest level without 2D
// tiles. Step k: convergence test on r_{k-1}; beta = g_{k-1}/g_{k-2},
// alpha = g_{k-1} / (d_{k-1} - beta g_{k-1}/alpha_{k-2}) with g = r.u and
// d = (A u).u; p = u + beta p; r -= alpha A p; x += alpha p.
//
// Bound by HBM: A p is formed again from p (its neighbours come from LDS or
// L2) instead of carried as s = A u + beta s, which with A u were three more
// arrays to move; and x takes its update every second step, both directions
// at once, when the old p is read anyway (x += alpha_{k-1} p_{k-1} +
// alpha_k p_k on even steps, the pending one when the solve ends on an odd
// one). 48 B per cell and step instead of 80: 256^3 FP64 166 - 170 us in step
// (4.7 - 4.8 TB/s) instead of 257 us.
struct CgScalars {
  double alpha, beta, alpha_old;
  bool end, pending;  // the solve ends with this test; x lacks alpha_{k-1} p_{k-1}
};
// False: the solve was done before this kernel.
__device__ inline bool cgcg_scalars(const CGArgs &a, int np_cc, CgScalars &q) {
  SolverScalars *sc = a.sc;
  const int k = a.k;
  if (ended_before(sc, k)) return false;
  double cc, g, d, rr;
  sum_cc3(k, a.part_cc, np_cc, sc, a.part_rz, a.part_rz + a.np_rz, a.part_rz + 2 * a.np_rz, a.np_rz, cc, g, d, rr);
  const bool conv = (cc == 0.0) || (rr <= a.tol2 * cc);
  q.beta = q.alpha_old = 0.0;
  if (k == 1) {
    q.alpha = g / d;
  } else {
    q.alpha_old = sc->alh[(k - 2) & 1];
    q.beta = g / sc->rzh[(k - 2) & 1];
    q.alpha = g / (d - q.beta * g / q.alpha_old);
  }
  const bool broken = !isfinite(rr) || !isfinite(q.alpha) || !isfinite(q.beta);
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    sc->rzh[(k - 1) & 1] = g;
    sc->alh[(k - 1) & 1] = q.alpha;
    sc->rr = rr;
    sc->cc = cc;
    sc->iters = k - 1;
    if (conv || broken) {
      sc->zero = (cc == 0.0);
      sc->nonconv = broken && !conv;
      sc->done = k + 1;
    }
  }
  q.end = conv || broken;
  q.pending = k >= 2 && (k & 1) == 0 && !(broken && !conv);
  return true;
}

// 2D: one thread per cell of a grid-stride loop.
template <typename TZ>
__global__ void __launch_bounds__(kBlock) k_cgcg_update(CGArgs a, int np_cc) {
  CgScalars q;
  if (!cgcg_scalars(a, np_cc, q) || (q.end && !q.pending)) return;
  const TZ *u = (const TZ *)a.z;
  const bool old = a.k >= 2;
  for (int tile = blockIdx.x; tile < ntiles_of(a.L); tile += gridDim.x) {
    int i, j, kk;
    if (!tile_cell(a.L, tile, i, j, kk)) continue;
    const long c = a.L.at(i, j, kk);
    if (q.end) {
      a.x[c] += q.alpha_old * a.pold[c];
      continue;
    }
    auto pv = [&](long m) -> double { return old ? (double)u[m] + q.beta * a.pold[m] : (double)u[m]; };
    const double pc = pv(c);
    double nbs = 0.0, dg = 0.0;
    const int x[2] = {i, j};
#pragma unroll
    for (int d = 0; d < 2; ++d) {
      const long lo = nbr(a.L, a.B, c, x[d], d, -1), hi = nbr(a.L, a.B, c, x[d], d, +1);
      double s = 0.0, sb = 0.0;
      if (lo >= 0) {
        const double bt = a.rho ? face_coef<double>(a.rho[c], a.rho[lo], d, a.met) : 1.0;
        s += bt * pv(lo);
        sb += bt;
      }
      if (hi >= 0) {
        const double bt = a.rho ? face_coef<double>(a.rho[c], a.rho[hi], d, a.met) : 1.0;
        s += bt * pv(hi);
        sb += bt;
      }
      nbs += a.ih2[d] * s;
      dg += a.ih2[d] * sb;
    }
    a.pnew[c] = pc;
    a.rnew[c] = a.rold[c] - q.alpha * (dg * pc - nbs);
    if (q.pending) a.x[c] += q.alpha_old * a.pold[c] + q.alpha * pc;
  }
}

// 3D: a block owns a 64 x 8 column of cells and marches up a run of planes.
// Each thread keeps its column's p of three planes in registers; the x and y
// neighbours come from an LDS plane (with a one-cell ring) filled one plane
// ahead; the loads run two planes ahead. Every array is read once but for
// the rings (28 % of u and p, from L2). Positions past the far sides are
// copies of the cells they wrap to, and not written.
// FORM 0: periodic, beta = 1; 1: any sides, beta = 1; 2: any sides, beta =
// 1/rho_f (the density goes the way of p, 8 B per cell more). A face of a
// side that is not periodic has the coefficient 0. 256^3, walls, mean over a
// solve's iterations: 152 us (FP64), 135 us (mixed), with a density 190 us;
// the same update with one thread per cell of a grid-stride loop, its
// neighbours read from L2: 339, 442 and 499 us; with s = A p carried, 231 us.
constexpr int kUX = 64, kUY = 8, kUW = kUX + 2;
constexpr int kURing = 2 * kUX + 2 * kUY;  // ring cells: two rows, two columns (no corners)
template <typename TZ, int FORM>
__global__ void __launch_bounds__(kUX *kUY, 4) k_cgcg_march(CGArgs a, int np_cc, int tiles_x, int tiles_y, int tz) {
  constexpr bool VC = FORM == 2;
  __shared__ double P[2][(kUY + 2) * kUW];
  __shared__ double Q[VC ? 2 : 1][VC ? (kUY + 2) * kUW : 1];
  CgScalars q;
  if (!cgcg_scalars(a, np_cc, q) || (q.end && !q.pending)) return;
  const Lay &L = a.L;
  const int nx = L.n[0], ny = L.n[1], nz = L.n[2];
  const int lb = xcd_remap(blockIdx.x, gridDim.x);
  const int tile = lb % (tiles_x * tiles_y), chunk = lb / (tiles_x * tiles_y);
  const int x0 = (tile % tiles_x) * kUX, y0 = (tile / tiles_x) * kUY;
  const int z0 = chunk * tz, z1 = min(z0 + tz, nz);
  const int tid = threadIdx.x, lx = tid & (kUX - 1), ly = tid / kUX;
  const bool own = x0 + lx < nx && y0 + ly < ny;
  const long s2 = L.s[2];
  const TZ *u = (const TZ *)a.z;
  const long col = L.base + (x0 + lx) % nx + (long)((y0 + ly) % ny) * L.s[1];
  if (q.end) {  // only the pending update of x
    if (own)
      for (int z = z0; z < z1; ++z) a.x[col + z * s2] += q.alpha_old * a.pold[col + z * s2];
    return;
  }
  const bool old = a.k >= 2;
  // this thread's ring cell: rows below and above, columns left and right
  const bool ring = tid < kURing;
  int rx, ry;
  if (tid < 2 * kUX) {
    rx = tid & (kUX - 1);
    ry = tid < kUX ? -1 : kUY;
  } else {
    rx = tid < 2 * kUX + kUY ? -1 : kUX;
    ry = (tid - 2 * kUX) & (kUY - 1);
  }
  const long rcol = ring ? L.base + (x0 + rx + nx) % nx + (long)((y0 + ry + ny) % ny) * L.s[1] : col;
  const int me = (ly + 1) * kUW + lx + 1, mr = (ry + 1) * kUW + rx + 1;
  const double ihx = a.ih2[0], ihy = a.ih2[1], ihz = a.ih2[2], dg = 2.0 * (ihx + ihy + ihz);
  // FORM > 0: 1/h^2 of the cell's low and high faces along x and y, 0
  // through a side
  double fx0 = ihx, fx1 = ihx, fy0 = ihy, fy1 = ihy;
  if constexpr (FORM != 0) {
    if (!a.B.periodic[0] && x0 + lx == 0) fx0 = 0.0;
    if (!a.B.periodic[0] && x0 + lx + 1 >= nx) fx1 = 0.0;
    if (!a.B.periodic[1] && y0 + ly == 0) fy0 = 0.0;
    if (!a.B.periodic[1] && y0 + ly + 1 >= ny) fy1 = 0.0;
  }
  auto plane = [&](int z) __attribute__((always_inline)) { return (long)(z < 0 ? z + nz : (z >= nz ? z - nz : z)) * s2; };
  auto pv = [&](TZ uv, double po) __attribute__((always_inline)) { return (double)uv + (old ? q.beta * po : 0.0); };
  // p below, at and above the first plane; its ring; the old p of the centre
  const long gm = plane(z0 - 1), g0 = plane(z0), g1 = plane(z0 + 1);
  double pom = old ? a.pold[col + gm] : 0.0, po = old ? a.pold[col + g0] : 0.0;
  double pm = pv(u[col + gm], pom), pc = pv(u[col + g0], po);
  TZ un = u[col + g1];
  double pn = old ? a.pold[col + g1] : 0.0;
  double rv = a.rold[col + g0], xv = q.pending ? a.x[col + g0] : 0.0;
  TZ ur = TZ(0);
  double pr = 0.0;
  // densities likewise: below, at and above the plane; the next plane's ring
  double dm = 0.0, dc = 0.0, dn = 0.0, dr = 0.0;
  if constexpr (VC) {
    dm = a.rho[col + gm];
    dc = a.rho[col + g0];
    dn = a.rho[col + g1];
    Q[z0 & 1][me] = dc;
  }
  P[z0 & 1][me] = pc;
  if (ring) {
    P[z0 & 1][mr] = pv(u[rcol + g0], old ? a.pold[rcol + g0] : 0.0);
    ur = u[rcol + g1];
    pr = old ? a.pold[rcol + g1] : 0.0;
    if constexpr (VC) {
      Q[z0 & 1][mr] = a.rho[rcol + g0];
      dr = a.rho[rcol + g1];
    }
  }
  __syncthreads();
  for (int z = z0; z < z1; ++z) {
    // values of plane z + 1 in hand; those of z + 2 (and r, x of z + 1) in flight
    const double pp = pv(un, pn), pon = pn, pring = pv(ur, pr);
    const double rc = rv, xc = xv, dp = dn, dring = dr;
    const long g2 = plane(z + 2), gn = plane(z + 1), gz = (long)z * s2;
    if (z + 1 < z1) {
      un = u[col + g2];
      pn = old ? a.pold[col + g2] : 0.0;
      rv = a.rold[col + gn];
      xv = q.pending ? a.x[col + gn] : 0.0;
      if constexpr (VC) dn = a.rho[col + g2];
      if (ring) {
        ur = u[rcol + g2];
        pr = old ? a.pold[rcol + g2] : 0.0;
        if constexpr (VC) dr = a.rho[rcol + g2];
      }
    }
    const double *S = P[z & 1];
    double Ap;
    if constexpr (FORM == 0) {
      const double nbs = ihx * (S[me - 1] + S[me + 1]) + ihy * (S[me - kUW] + S[me + kUW]) + ihz * (pm + pp);
      Ap = dg * pc - nbs;
    } else {
      double cx0 = fx0, cx1 = fx1, cy0 = fy0, cy1 = fy1;
      double cz0 = a.B.periodic[2] || z > 0 ? ihz : 0.0, cz1 = a.B.periodic[2] || z + 1 < nz ? ihz : 0.0;
      if constexpr (VC) {
        const double *D = Q[z & 1];
        cx0 *= face_beta<double>(dc, D[me - 1]);
        cx1 *= face_beta<double>(dc, D[me + 1]);
        cy0 *= face_beta<double>(dc, D[me - kUW]);
        cy1 *= face_beta<double>(dc, D[me + kUW]);
        cz0 *= face_beta<double>(dc, dm);
        cz1 *= face_beta<double>(dc, dp);
      }
      const double nbs = (cx0 * S[me - 1] + cx1 * S[me + 1]) + (cy0 * S[me - kUW] + cy1 * S[me + kUW]) + (cz0 * pm + cz1 * pp);
      Ap = ((cx0 + cx1) + (cy0 + cy1) + (cz0 + cz1)) * pc - nbs;
    }
    if (own) {
      a.pnew[col + gz] = pc;
      a.rnew[col + gz] = rc - q.alpha * Ap;
      if (q.pending) a.x[col + gz] = xc + (q.alpha_old * po + q.alpha * pc);
    }
    P[(z + 1) & 1][me] = pp;
    if (ring) P[(z + 1) & 1][mr] = pring;
    if constexpr (VC) {
      Q[(z + 1) & 1][me] = dp;
      if (ring) Q[(z + 1) & 1][mr] = dring;
      dm = dc;
      dc = dp;
    }
    __syncthreads();
    pm = pc;
    pc = pp;
    po = pon;
  }
}

// Partials of r.u, w.u, r.r with w = A u (u = M r) for the unfused finest
// level.
template <int DIM, typename TZ>
__global__ void __launch_bounds__(kBlock) k_cgcg_w(CGArgs a) {
  if (a.sc->done) return;
  const TZ *u = (const TZ *)a.z;
  double ru = 0.0, wu = 0.0, rr = 0.0;
  for (int tile = blockIdx.x; tile < ntiles_of(a.L); tile += gridDim.x) {
    int i, j, k;
    if (!tile_cell(a.L, tile, i, j, k)) continue;
    const long c = a.L.at(i, j, k);
    double nbs, dg;
    if (a.rho)
      op_parts_vc<DIM, double, TZ, double>(a.L, a.B, a.ih2, a.rho, u, i, j, k, c, nbs, dg, a.met);
    else
      op_parts<DIM, double, TZ>(a.L, a.B, a.ih2, u, i, j, k, c, nbs, dg);
    const double uc = (double)u[c];
    const double wv = dg * uc - nbs;
    const double rv = a.rnew[c];
    ru += rv * uc;
    wu += wv * uc;
    rr += rv * rv;
  }
  double v3[3] = {ru, wu, rr};
  block_allsum_n<3>(v3);
  if (linear_tid() == 0) {
    a.part_rz[blockIdx.x] = v3[0];
    a.part_rz[a.np_rz + blockIdx.x] = v3[1];
    a.part_rz[2 * a.np_rz + blockIdx.x] = v3[2];
  }
}

// Sum of x into partials (mean of the final solution).
template <int DIM>
__global__ void __launch_bounds__(kBlock) k_sum_x(Lay L, const double *x, double *part, const double *vol,
                                                  const SolverScalars *sc) {
  __shared__ double sh[kBlock / 64];
  if (!sc->done) return;
  // four tiles' loads in flight per trip, four running sums combined in a
  // fixed order
  double s[4] = {0.0, 0.0, 0.0, 0.0};
  const int nt = ntiles_of(L);
  for (int t0 = blockIdx.x; t0 < nt; t0 += 4 * gridDim.x) {
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int tile = t0 + u * gridDim.x;
      int i, j, k;
      if (tile < nt && tile_cell(L, tile, i, j, k)) {
        const long c = L.at(i, j, k);
        s[u] += vol ? x[c] * vol[c] : x[c];   // stretched: the integral of x
      }
    }
  }
  const double r = block_sum((s[0] + s[1]) + (s[2] + s[3]), sh);
  if (linear_tid() == 0) part[blockIdx.x] = r;
}

// The scalars of a solve into the host's pinned memory, then their number.
__device__ inline void host_write(HostSolve *host, const SolverScalars *sc, unsigned seq) {
  host->sc = *sc;
  __threadfence_system();
  __hip_atomic_store(&host->seq, seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// Mean of the solution of an ended solve; the scalars to the host's pinned
// memory, if it waits there.
__global__ void __launch_bounds__(kBlock) k_fin_mean_x(const double *part, int np, double ncells, SolverScalars *sc,
                                                       HostSolve *host, unsigned seq) {
  __shared__ double sh[kBlock / 64];
  if (sc->done) {
    const double s = sum_all(part, np, sh);
    if (threadIdx.x == 0) sc->mean_x = s / ncells;
  }
  if (host && threadIdx.x == 0) host_write(host, sc, seq);
}

// ---------------------------------------------------------------------------
// Unfused multigrid kernels (any dimension, ragged sizes)
// ---------------------------------------------------------------------------

// One red (color 0) or black (color 1) half-sweep of Gauss-Seidel on
// L x = b. With zero_init the previous iterate is zero (first half-sweep
// of the pre-smoother): red cells take b/diag without reading x.
template <int DIM, typename TX, typename TB>
__global__ void __launch_bounds__(kBlock) k_mg_smooth(Lay L, Bnd B, Ih2<TX> ih2, TX *x, const TB *b, int color,
                                                      int zero_init, const SolverScalars *sc, const TX *rho,
                                                      int met) {
  if (sc->done) return;
  CellPos p;
  if (!cell_of_thread(L, p)) return;
  if (((p.i + p.j + p.k) & 1) != color) return;
  TX nbs, dg;
  if (rho)
    op_parts_vc<DIM, TX, TX, TX>(L, B, ih2.v, rho, x, p.i, p.j, p.k, p.c, nbs, dg, met);
  else
    op_parts<DIM, TX, TX>(L, B, ih2.v, x, p.i, p.j, p.k, p.c, nbs, dg);
  if (zero_init && color == 0) nbs = TX(0);
  x[p.c] = ((TX)b[p.c] + nbs) / dg;
}

// Coarse right-hand side: average over the 2^DIM children of b - L x.
template <int DIM, typename TX, typename TB>
__global__ void __launch_bounds__(kBlock) k_mg_restrict(Lay Lf, Lay Lc, Bnd B, Ih2<TX> ih2, const TX *x,
                                                        const TB *b, TX *bc, const SolverScalars *sc, const TX *rho,
                                                        int met) {
  if (sc->done) return;
  CellPos p;
  if (!cell_of_thread(Lc, p)) return;
  TX acc = TX(0);
#pragma unroll
  for (int dz = 0; dz < (DIM == 3 ? 2 : 1); ++dz)
#pragma unroll
    for (int dy = 0; dy < 2; ++dy)
#pragma unroll
      for (int dx = 0; dx < 2; ++dx) {
        const int i = 2 * p.i + dx, j = 2 * p.j + dy, k = DIM == 3 ? 2 * p.k + dz : 0;
        const long c = Lf.at(i, j, k);
        TX nbs, dg;
        if (rho)
          op_parts_vc<DIM, TX, TX, TX>(Lf, B, ih2.v, rho, x, i, j, k, c, nbs, dg, met);
        else
          op_parts<DIM, TX, TX>(Lf, B, ih2.v, x, i, j, k, c, nbs, dg);
        acc += ((TX)b[c] - (dg * x[c] - nbs));
      }
  bc[p.c] = acc * (DIM == 3 ? TX(0.125) : TX(0.25));
}

// x_fine += x_coarse(parent) (piecewise-constant prolongation).
template <int DIM, typename TX>
__global__ void __launch_bounds__(kBlock) k_mg_prolong(Lay Lf, Lay Lc, TX *xf, const TX *xc,
                                                       const SolverScalars *sc) {
  if (sc->done) return;
  CellPos p;
  if (!cell_of_thread(Lf, p)) return;
  xf[p.c] += xc[Lc.at(p.i >> 1, p.j >> 1, DIM == 3 ? (p.k >> 1) : 0)];
}

// ---------------------------------------------------------------------------
// Variable-coefficient set-up (once per solve with beta = 1/rho_f)
// ---------------------------------------------------------------------------

// Flags a density that is not positive and finite; converts the finest
// density to the multigrid precision (rt NULL: used as is).
template <int DIM, typename T>
__global__ void __launch_bounds__(kBlock) k_vc_rho0(Lay L, const double *r64, T *rt, SolverScalars *sc) {
  CellPos p;
  if (!cell_of_thread(L, p)) return;
  const double r = r64[p.c];
  if (!(r > 0.0) || !isfinite(r)) sc->rho_bad = 1;
  if (rt) rt[p.c] = (T)r;
}

// Density of the next coarser level: mean of the 2^DIM children.
template <int DIM, typename TS, typename TD>
__global__ void __launch_bounds__(kBlock) k_vc_rho_down(Lay Lf, Lay Lc, const TS *rf, TD *rc) {
  CellPos p;
  if (!cell_of_thread(Lc, p)) return;
  double acc = 0.0;
#pragma unroll
  for (int dz = 0; dz < (DIM == 3 ? 2 : 1); ++dz)
#pragma unroll
    for (int dy = 0; dy < 2; ++dy)
#pragma unroll
      for (int dx = 0; dx < 2; ++dx)
        acc += (double)rf[Lf.at(2 * p.i + dx, 2 * p.j + dy, DIM == 3 ? 2 * p.k + dz : 0)];
  rc[p.c] = (TD)(acc * (DIM == 3 ? 0.125 : 0.25));
}

// Face coefficients of a tiled 2D level: beta of each cell's west and south
// faces (0 through a non-periodic side) and 1/diagonal of L (the same
// operations as op_parts_vc, so the same bits).
template <typename T>
__global__ void __launch_bounds__(kBlock) k_vc_coef2d(Lay L, Bnd B, T ihx, T ihy, const T *rho, T *fx, T *fy,
                                                      T *ig, int met) {
#pragma clang fp contract(off)
  CellPos p;
  if (!cell_of_thread(L, p)) return;
  const int nx = L.n[0], ny = L.n[1];
  const long c = p.c, sy = L.s[1];
  const T rc = rho[c];
  T bw = T(0), be = T(0), bs = T(0), bn = T(0);
  if (B.periodic[0] || p.i > 0) bw = face_coef<T>(rc, rho[p.i > 0 ? c - 1 : c + (nx - 1)], 0, met);
  if (B.periodic[0] || p.i + 1 < nx) be = face_coef<T>(rc, rho[p.i + 1 < nx ? c + 1 : c - (nx - 1)], 0, met);
  if (B.periodic[1] || p.j > 0) bs = face_coef<T>(rc, rho[p.j > 0 ? c - sy : c + (long)(ny - 1) * sy], 1, met);
  if (B.periodic[1] || p.j + 1 < ny) bn = face_coef<T>(rc, rho[p.j + 1 < ny ? c + sy : c - (long)(ny - 1) * sy], 1, met);
  fx[c] = bw;
  fy[c] = bs;
  ig[c] = T(1) / (ihx * (bw + be) + ihy * (bs + bn));
}

}  // namespace lm

#include "lm_mg_kernels.h"
#include "lm_mg3d.h"
#include "lm_coarse.h"

namespace lm {

// Pseudo-inverse of the coarsest variable-coefficient operator,
// (L + J/N)^{-1} - J/N with J the all-ones matrix: L + J/N is symmetric
// positive definite (L is singular with the constants as null space), so
// Gauss-Jordan elimination without pivoting inverts it. UNIT: beta = 1 on
// every face (no densities read).
// The N steps are a serial chain, one barrier each; the matrix stays in
// registers (column t % NP, every R-th row) and only the next pivot row and
// column pass through LDS. 64 cells: 55 us; with the matrix in LDS, 256
// threads and two barriers per step 130 us.
constexpr int kPinvThreads = 1024;
template <int DIM, typename T, bool UNIT, int NP>
__global__ void __launch_bounds__(kPinvThreads) k_vc_pinv(Lay L, Bnd B, Ih2<double> ih2v, int met, const T *rho,
                                                          T *pinv) {
  constexpr int R = kPinvThreads / NP, ROWS = NP / R;
  __shared__ double M[NP * NP];
  __shared__ double rk[2][NP], ck[2][NP];
  const int *n = L.n;
  const int N = n[0] * n[1] * n[2];
  const int t = threadIdx.x;
  const double jn = 1.0 / (double)N;
  for (int e = t; e < NP * NP; e += kPinvThreads) M[e] = (e / NP < N && e % NP < N) ? jn : 0.0;
  __syncthreads();
  if (t < N) {
    int i, j, k;
    c_decode<DIM>(n, t, i, j, k);
    const int q[3] = {i, j, k};
    const int st[3] = {1, n[0], n[0] * n[1]};
    const long g = L.at(i, j, k);
    const double rc = UNIT ? 1.0 : (double)rho[g];
    for (int d = 0; d < DIM; ++d) {
      const bool per = B.periodic[d] != 0;
      const double ih2 = (double)(T)ih2v.v[d];
      for (int side = 0; side < 2; ++side) {
        const bool in = side == 0 ? q[d] > 0 : q[d] + 1 < n[d];
        if (!in && !per) continue;
        const int m = side == 0 ? (in ? t - st[d] : t + (n[d] - 1) * st[d]) : (in ? t + st[d] : t - (n[d] - 1) * st[d]);
        const long gm = nbr(L, B, g, q[d], d, side ? 1 : -1);
        const double w = UNIT ? ih2 : ih2 * face_coef<double>(rc, (double)rho[gm], d, met);
        M[t * NP + t] += w;
        M[t * NP + m] -= w;
      }
    }
  }
  __syncthreads();
  const int j = t % NP, i0 = t / NP;
  double m[ROWS];
#pragma unroll
  for (int p = 0; p < ROWS; ++p) m[p] = M[(i0 + R * p) * NP + j];
  if (t < NP) {
    rk[0][t] = M[t];
    ck[0][t] = M[t * NP];
  }
  for (int kk = 0; kk < N; ++kk) {
    const int cur = kk & 1;
    __syncthreads();
    const double ip = 1.0 / rk[cur][kk];
    const double rj = rk[cur][j] * ip;
#pragma unroll
    for (int p = 0; p < ROWS; ++p) {
      const int i = i0 + R * p;
      const double c = ck[cur][i];
      double v = m[p] - c * rj;
      if (j == kk) v = -c * ip;
      if (i == kk) v = j == kk ? ip : rj;
      m[p] = v;
      if (i == kk + 1) rk[cur ^ 1][j] = v;
      if (j == kk + 1) ck[cur ^ 1][i] = v;
    }
  }
#pragma unroll
  for (int p = 0; p < ROWS; ++p) {
    const int i = i0 + R * p;
    if (i < N && j < N) pinv[i * N + j] = (T)(m[p] - jn);
  }
}
static_assert(kVcCoarsest == 128, "the larger of the two inverse kernels");
static_assert(kBlkGeo * sizeof(BlkGeo) == kGeoBytes, "size of the block geometry table");
}  // namespace lm

namespace lm {

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------

static int tile_x(const PoissonWS &ws, int l) { return ws.vc ? ws.vtx[l] : ws.tx[l]; }
static int tile_y(const PoissonWS &ws, int l) { return ws.vc ? ws.vty[l] : ws.ty[l]; }

// Tiles of a level along each direction / in all (the last ones may reach
// beyond the grid).
static int tiles_along(int n, int t) { return (n + t - 1) / t; }
static int tiles2d(const Lay &L, int tx, int ty) { return tiles_along(L.n[0], tx) * tiles_along(L.n[1], ty); }

// Tile of 2D level l (< lc) among the candidates, or 0 x 0 when none fits:
// the first that divides the level, else the one with the fewest cells in
// its frames (the halos included, which is what an edge tile costs: 120 x 88
// by 16 x 16 is 48 frames of 676 cells against 44 of 756 by 32 x 8). A frame
// may reach past the far side by less than a period only (wrap_or_out wraps
// once); smaller levels run the unfused kernels. Measured: a level of 96^2
// (stretched, FP64) or 120 x 88 (FP32) takes ten unfused launches of 3.3 - 5
// us per cycle, two tiled ones of 5 us: 8 steps of the 96^2 cavity 14.3 ->
// 6.4 ms, of 240 x 176 11.5 -> 7.0 ms.
static void fit_tile(const Lay &L, int nu, const int (*cand)[2], int nc, int &tx, int &ty) {
  tx = ty = 0;
  for (int q = 0; q < nc; ++q)
    if (L.n[0] % cand[q][0] == 0 && L.n[1] % cand[q][1] == 0) {
      tx = cand[q][0];
      ty = cand[q][1];
      return;
    }
  const int H = 2 * nu + 1;
  long best = 0;
  for (int q = 0; q < nc; ++q) {
    const int cx = cand[q][0], cy = cand[q][1];
    if (L.n[0] < cx + H || L.n[1] < cy + H) continue;
    const long cost = (long)tiles2d(L, cx, cy) * (cx + 2 * H) * (cy + 2 * H);
    if (tx == 0 || cost < best) {
      tx = cx;
      ty = cy;
      best = cost;
    }
  }
}

// The finest level takes the large tile, whose frame is 1.9 times its cells
// (the small one's 2.9), once the chip has one and a half per unit; below
// that the small one puts more wavefronts on a unit. FP64 solve, large and
// small: 256^2 478 and 404 us, 512^2 599 and 529, 768 x 512 1268 and 1186,
// 1024 x 512 2313 and 2308, 1024 x 768 1109 and 1216, 1024^2 840 and 1018.
// Up to the line also in the other forms: mixed, 256^2 441 and 379, 512^2
// 532 and 490, 768 x 512 785 and 774; with walls, FP64, 677 and 566, 833 and
// 757, 1147 and 1063; mixed-flexible with walls 714 and 611, 874 and 788,
// 1210 and 1115.
constexpr int kLargeTiles = 384;

static void choose_tile(PoissonWS &ws, int l) {
  const Lay &L = ws.lev[l].lay;
  ws.tx[l] = ws.ty[l] = 0;
  if (ws.met || L.ndim != 2 || ws.nu < 1 || ws.nu > 3 || l >= ws.lc) return;
  const int cand[3][2] = {{TX, TY}, {TXS, TYS}, {16, 16}};
  const int q = l == 0 && tiles2d(L, TX, TY) > kLargeTiles ? 0 : 1;
  fit_tile(L, ws.nu, cand + q, 3 - q, ws.tx[l], ws.ty[l]);
}

// Tile of 2D level l (< lc) for the variable-coefficient kernels (stretched
// grids too), whose frames carry three more LDS arrays (face coefficients,
// 1/diagonal): the small tiles only.
static void choose_tile_vc(PoissonWS &ws, int l) {
  const Lay &L = ws.lev[l].lay;
  ws.vtx[l] = ws.vty[l] = 0;
  if (!ws.vc_cap || L.ndim != 2 || ws.nu < 1 || ws.nu > 3 || l >= ws.lc) return;
  const int cand[2][2] = {{TXS, TYS}, {16, 16}};
  fit_tile(L, ws.nu, cand, 2, ws.vtx[l], ws.vty[l]);
}

// Fused 3D level kernels: the owned tile edge is the 32-cell frame less
// twice the x-y halo (down leg 2 nu; up leg 2 nu, plus one on the finest
// level of the single-reduction CG, which also forms w = A u; rounded up to
// even).
static int ti3(int nu, bool down, bool extra) {
  const int h = 2 * nu + ((!down && extra) ? 1 : 0);
  return kF3 - 2 * ((h + 1) & ~1);
}
static int tiles3(const Lay &L, int ti, int d) { return (L.n[d] + ti - 1) / ti; }

// Depth of the z chunk (a multiple of 4: the chunks start on the kernels'
// LDS buffer order): as many chunks as keep about one block per block slot
// of the chip (256 CUs, two 512-thread blocks each). Every chunk marches
// through 2H halo planes beyond its own, so a level that cannot fill the
// chip takes the shallowest chunks: its time is that of one block's march
// (about 0.55 us a plane step), whatever their number. 32^3 level: chunks of
// 4 planes 7.7 us per leg, of 16 planes 13.3 us.
static int tz3_of(const Lay &L, int ti) {
  const long tiles = (long)tiles3(L, ti, 0) * tiles3(L, ti, 1);
  const long nchunk = std::max(1L, 512L / tiles);
  const int tz = (int)((L.n[2] + nchunk - 1) / nchunk);
  return (tz + 3) & ~3;
}

// Blocks of one fused 3D launch on layout L with owned tile edge ti.
static long blocks3d(const Lay &L, int ti) {
  const int tz = tz3_of(L, ti);
  return (long)tiles3(L, ti, 0) * tiles3(L, ti, 1) * ((L.n[2] + tz - 1) / tz);
}

// Level l runs the fused 3D kernels (fully periodic grids, even sizes, every
// level above the one-workgroup cycle: 40 x 24 x 28, FP32, two launches of 8
// us against ten of 4.6 us; the march's plane index wraps once, so at least
// 16 planes).
static bool fused3d(const PoissonWS &ws, int l) {
  const Lay &L = ws.lev[l].lay;
  return !ws.vc && L.ndim == 3 && ws.bnd.all_periodic && ws.nu >= 1 && ws.nu <= 2 && l < ws.lc &&
         L.n[0] % 2 == 0 && L.n[1] % 2 == 0 && L.n[2] % 2 == 0 &&
         L.n[2] >= 16;
}

// Blocks of the finest level's up kernel with w = A u (its partials).
static long blocks3d_w(const PoissonWS &ws) { return blocks3d(ws.lev[0].lay, ti3(ws.nu, false, true)); }

static bool fused_level(const PoissonWS &ws, int l) { return tile_x(ws, l) > 0; }

// Offset of level l's coefficient sets in those of the coarse-kernel levels
// (every level but the last is even in all directions: 2^DIM-cell blocks).
static long coarse_coef_offset(const PoissonWS &ws, int l) {
  const bool three = ws.lay.ndim == 3;
  long off = 0;
  for (int q = ws.lc; q < l && q < ws.nlev - 1; ++q)
    off += (three ? kBlkSlots<3> * (ws.lev[q].lay.ncells() / 8) : kBlkSlots<2> * (ws.lev[q].lay.ncells() / 4));
  return off;
}

bool poisson_plan(PoissonWS &ws, Carver &cv, const Lay &fine, const Bnd &B, const double h[3], int mixed, int flexible,
                  int nu, int vc_cap, std::string *err) {
  ws.lay = fine;
  ws.bnd = B;
  ws.mixed = mixed;
  ws.nu = nu;
  ws.vc_cap = vc_cap;
  ws.vc = 0;
  const int ndim = fine.ndim;
  const int eb = mixed ? 4 : 8;
  int n[3] = {fine.n[0], fine.n[1], fine.n[2]};
  double hh[3] = {h[0], h[1], h[2]};
  int nl = 0;
  while (true) {
    MGLevel &m = ws.lev[nl];
    m.lay = nl == 0 ? fine : make_layout(ndim, n, eb);
    for (int d = 0; d < 3; ++d) m.ih2[d] = d < ndim ? 1.0 / (hh[d] * hh[d]) : 0.0;
    ++nl;
    long N = (long)n[0] * n[1] * n[2];
    bool even = true;
    for (int d = 0; d < ndim; ++d) even = even && (n[d] % 2 == 0) && (n[d] / 2 >= 2);
    if (!even || N <= 64 || nl == kMaxLev) break;
    for (int d = 0; d < ndim; ++d) {
      n[d] /= 2;
      hh[d] *= 2.0;
    }
  }
  ws.nlev = nl;
  if (ws.met) {
    // volume-weighted operator: unit coefficients on the finest level, a
    // quarter per coarser level (the restriction averages the 4 children
    // of a residual whose coarse operator sums them)
    for (int l = 0; l < nl; ++l)
      for (int d = 0; d < 3; ++d) ws.lev[l].ih2[d] = d < ndim ? std::ldexp(1.0, -2 * l) : 0.0;
  }
  const long ncoarsest = ws.lev[nl - 1].lay.ncells();
  if (ncoarsest > kMaxCoarsest) {
    if (err) *err = "grid does not coarsen to <= 1024 cells (need even sizes down to the coarse grid)";
    return false;
  }
  ws.lc = 0;
  while (ws.lc < nl - 1 && ws.lev[ws.lc].lay.ncells() > kCoarseCells) ++ws.lc;
  long lds = 0;
  for (int l = ws.lc; l < nl; ++l) lds += ws.lev[l].lay.ncells();
  if (lds > kCoarseLds || nl - ws.lc > kCoarseLev) {
    if (err) *err = "coarse grid too large for the one-block coarse solver";
    return false;
  }
  if (vc_cap && ncoarsest > kVcCoarsest) {
    if (err) *err = "the variable-coefficient solve needs a grid that coarsens to <= 128 cells";
    return false;
  }
  const size_t fbytes = (size_t)fine.total * 8;
  ws.x = (double *)cv.take(fbytes);
  ws.r[0] = (double *)cv.take(fbytes);
  ws.r[1] = (double *)cv.take(fbytes);
  ws.p[0] = (double *)cv.take(fbytes);
  ws.p[1] = (double *)cv.take(fbytes);
  ws.cgcg = !flexible;
  // 2D tiles
  for (int l = 0; l < kMaxLev; ++l) {
    ws.tx[l] = ws.ty[l] = 0;
    ws.vtx[l] = ws.vty[l] = 0;
    if (l < nl) {
      choose_tile(ws, l);
      choose_tile_vc(ws, l);
    }
  }
  // only flexible CG stores q = A p, and only the single-reduction form on 2D
  // tiles w = A u and s = A p
  const bool tiled = ws.tx[0] > 0 || ws.vtx[0] > 0;
  ws.q = flexible || ws.fixed ? (double *)cv.take(fbytes) : nullptr;
  ws.w = ws.s[0] = ws.s[1] = nullptr;
  if ((ws.cgcg && tiled) || ws.fixed)
    for (double **v : {&ws.w, &ws.s[0], &ws.s[1]}) *v = (double *)cv.take(fbytes);
  // grids the one-block V-cycle covers from the finest level: the whole
  // single-reduction solve in one workgroup (LM_BLOCK_PCG=0 turns it off)
  {
    const char *env = std::getenv("LM_BLOCK_PCG");
    const bool off = env && env[0] == '0';
    ws.block_pcg = !off && ws.cgcg && ws.lc == 0 && fine.ncells() <= kCoarseCells;
  }
  ws.z[0] = cv.take((size_t)fine.total * eb);
  ws.z[1] = (mixed && !ws.cgcg) ? cv.take((size_t)fine.total * eb) : ws.z[0];  // z_old: flexible CG only
  ws.zpre = cv.take((size_t)fine.total * eb);
  ws.lev[0].x = nullptr;
  ws.lev[0].xpost = nullptr;
  ws.lev[0].b = nullptr;
  for (int l = 1; l < nl; ++l) {
    const size_t lb = (size_t)ws.lev[l].lay.total * eb;
    ws.lev[l].x = cv.take(lb);
    ws.lev[l].xpost = cv.take(lb);
    ws.lev[l].b = cv.take(lb);
  }
  ws.pinv = cv.take((size_t)ncoarsest * ncoarsest * eb);
  if (!ws.fixed) ws.geo = cv.take(kGeoBytes);
  ws.rho64 = nullptr;
  ws.ccf = ws.pinv_vc = nullptr;
  ws.ccd = nullptr;
  for (int l = 0; l < kMaxLev; ++l) ws.rho[l] = nullptr;
  if (vc_cap) {
    ws.rho64 = (double *)cv.take(fbytes);
    ws.rho[0] = mixed ? cv.take((size_t)fine.total * eb) : (void *)ws.rho64;
    for (int l = 1; l < nl; ++l) ws.rho[l] = cv.take((size_t)ws.lev[l].lay.total * eb);
    ws.ccf = cv.take((size_t)coarse_coef_offset(ws, nl - 1) * eb);
    if (ws.block_pcg && mixed) ws.ccd = (double *)cv.take((size_t)coarse_coef_offset(ws, 1) * 8);
    ws.pinv_vc = cv.take((size_t)ncoarsest * ncoarsest * eb);
  }
  for (int l = 0; l < kMaxLev; ++l)
    for (int q = 0; q < 3; ++q) ws.cf[l][q] = nullptr;
  for (int l = 0; l < nl; ++l)
    if (ws.vtx[l] > 0)
      for (int q = 0; q < 3; ++q) ws.cf[l][q] = cv.take((size_t)ws.lev[l].lay.total * eb);
  long npmax = kRedBlocks;
  if (ws.tx[0] > 0) npmax = std::max(npmax, (long)tiles2d(fine, ws.tx[0], ws.ty[0]) + 1);
  if (ws.vtx[0] > 0) npmax = std::max(npmax, (long)tiles2d(fine, ws.vtx[0], ws.vty[0]) + 1);
  if (fused3d(ws, 0) && blocks3d_w(ws) > npmax) npmax = blocks3d_w(ws);
  ws.np_max = npmax;
  ws.part_cc = (double *)cv.take((size_t)npmax * 8);
  ws.part_pq = (double *)cv.take((size_t)npmax * 8);
  ws.part_rz = (double *)cv.take((size_t)3 * npmax * 8);
  ws.partials = (double *)cv.take((size_t)(nblocks_for(fine) + kRedBlocks) * 8 + 64);
  ws.sc = (SolverScalars *)cv.take(sizeof(SolverScalars));
  ws.vol = nullptr;
  ws.met_w = nullptr;
  if (ws.met) {
    long nw = 0;
    for (int l = 0; l < nl; ++l) nw += ws.lev[l].lay.n[0] + ws.lev[l].lay.n[1];
    ws.vol = (double *)cv.take(fbytes);
    ws.met_w = (double *)cv.take((size_t)nw * 8);
  }
  return true;
}

template <typename T>
static Ih2<T> ih2_of(const PoissonWS &ws, int l) {
  Ih2<T> v;
  for (int d = 0; d < 3; ++d) v.v[d] = (T)ws.lev[l].ih2[d];
  return v;
}

// Arrays of level l: input (pre-smoothed) and output (post-smoothed)
// corrections. Unfused levels smooth in place.
template <typename T>
static T *lev_xin(PoissonWS &ws, int l, void *z) {
  if (l == 0) return (fused_level(ws, 0) || fused3d(ws, 0)) ? (T *)ws.zpre : (T *)z;
  return (T *)ws.lev[l].x;
}
template <typename T>
static T *lev_xout(PoissonWS &ws, int l, void *z) {
  if (l == 0) return (T *)z;
  if (l >= ws.lc) return (T *)ws.lev[l].x;
  return ((fused_level(ws, l) || fused3d(ws, l)) ? (T *)ws.lev[l].xpost : (T *)ws.lev[l].x);
}

template <typename T>
static Fused3DArgs<T> f3_args(PoissonWS &ws, int l, const void *b, int b_double) {
  Fused3DArgs<T> a;
  const Lay &L = ws.lev[l].lay;
  a.Lf = L;
  a.Lc = ws.lev[l + 1].lay;
  a.ihx = (T)ws.lev[l].ih2[0];
  a.ihy = (T)ws.lev[l].ih2[1];
  a.ihz = (T)ws.lev[l].ih2[2];
  a.dihx = ws.lev[l].ih2[0];
  a.dihy = ws.lev[l].ih2[1];
  a.dihz = ws.lev[l].ih2[2];
  a.idg = (T)(1.0 / (2.0 * (ws.lev[l].ih2[0] + ws.lev[l].ih2[1] + ws.lev[l].ih2[2])));
  a.tiles_x = a.tiles_y = a.tz = 0;  // set by launch_3d for the leg
  a.b = b;
  a.b_double = b_double;
  a.xpre = nullptr;
  a.xc = nullptr;
  a.xout = nullptr;
  a.bc = (T *)ws.lev[l + 1].b;
  a.sc = ws.sc;
  return a;
}

// Launch with optional start/stop events bound to the dispatch itself: they
// bracket the kernel's execution, not the queueing gap before it.
template <typename K, typename A>
static void launch_ev(K kern, dim3 g, hipStream_t st, hipEvent_t e0, hipEvent_t e1, const A &a) {
  if (e0)
    hipExtLaunchKernelGGL(kern, g, dim3(kBlock), 0, st, e0, e1, 0, a);
  else
    hipLaunchKernelGGL(kern, g, dim3(kBlock), 0, st, a);
}

template <typename T>
static void launch_3d(int nu, bool down, Fused3DArgs<T> &a, hipStream_t st, bool extra = false,
                      hipEvent_t e0 = nullptr, hipEvent_t e1 = nullptr) {
  const int ti = ti3(nu, down, extra);
  a.tiles_x = tiles3(a.Lf, ti, 0);
  a.tiles_y = tiles3(a.Lf, ti, 1);
  a.tz = tz3_of(a.Lf, ti);
  const dim3 g((unsigned)blocks3d(a.Lf, ti));
  const dim3 bl(kF3Threads);
  // FP64 right-hand side in FP32 kernels only on the finest level
  const bool bd = a.b_double && sizeof(T) == 4;
  if (down) {
    auto k = nu == 1 ? (bd ? &k_mg_down3d<T, 1, true> : &k_mg_down3d<T, 1, false>)
                     : (bd ? &k_mg_down3d<T, 2, true> : &k_mg_down3d<T, 2, false>);
    if (e0)
      hipExtLaunchKernelGGL(k, g, bl, 0, st, e0, e1, 0, a);
    else
      hipLaunchKernelGGL(k, g, bl, 0, st, a);
  } else {
    auto k = extra ? (nu == 1 ? (bd ? &k_mg_up3d<T, 1, 1, true> : &k_mg_up3d<T, 1, 1, false>)
                              : (bd ? &k_mg_up3d<T, 2, 1, true> : &k_mg_up3d<T, 2, 1, false>))
                   : (nu == 1 ? (bd ? &k_mg_up3d<T, 1, 0, true> : &k_mg_up3d<T, 1, 0, false>)
                              : (bd ? &k_mg_up3d<T, 2, 0, true> : &k_mg_up3d<T, 2, 0, false>));
    if (e0)
      hipExtLaunchKernelGGL(k, g, bl, 0, st, e0, e1, 0, a);
    else
      hipLaunchKernelGGL(k, g, bl, 0, st, a);
  }
}

// The finest 3D up kernel forms w = A u and the single-reduction CG partials.
static bool w_in_up3d(const PoissonWS &ws) { return ws.cgcg && fused3d(ws, 0); }

template <typename T, int TXT, int TYT>
static void launch_nu_t(int nu, Down2DArgs<T> &a, dim3 g, hipStream_t st, hipEvent_t e0, hipEvent_t e1) {
  if (nu == 1) launch_ev(&k_mg_down2d<T, 1, TXT, TYT>, g, st, e0, e1, a);
  else if (nu == 2) launch_ev(&k_mg_down2d<T, 2, TXT, TYT>, g, st, e0, e1, a);
  else launch_ev(&k_mg_down2d<T, 3, TXT, TYT>, g, st, e0, e1, a);
}
template <typename T, int TXT, int TYT>
static void launch_nu_t(int nu, Up2DArgs<T> &a, dim3 g, hipStream_t st, bool extra) {
  if (extra) {
    if (nu == 1) hipLaunchKernelGGL((k_mg_up2d<T, 1, 1, TXT, TYT>), g, dim3(kBlock), 0, st, a);
    else if (nu == 2) hipLaunchKernelGGL((k_mg_up2d<T, 2, 1, TXT, TYT>), g, dim3(kBlock), 0, st, a);
    else hipLaunchKernelGGL((k_mg_up2d<T, 3, 1, TXT, TYT>), g, dim3(kBlock), 0, st, a);
    return;
  }
  if (nu == 1) hipLaunchKernelGGL((k_mg_up2d<T, 1, 0, TXT, TYT>), g, dim3(kBlock), 0, st, a);
  else if (nu == 2) hipLaunchKernelGGL((k_mg_up2d<T, 2, 0, TXT, TYT>), g, dim3(kBlock), 0, st, a);
  else hipLaunchKernelGGL((k_mg_up2d<T, 3, 0, TXT, TYT>), g, dim3(kBlock), 0, st, a);
}
template <typename T, int TXT, int TYT>
static void launch_nu_vc(int nu, Down2DArgs<T> &a, dim3 g, hipStream_t st, hipEvent_t e0, hipEvent_t e1) {
  if (nu == 1) launch_ev(&k_mg_down2d<T, 1, TXT, TYT, true>, g, st, e0, e1, a);
  else if (nu == 2) launch_ev(&k_mg_down2d<T, 2, TXT, TYT, true>, g, st, e0, e1, a);
  else launch_ev(&k_mg_down2d<T, 3, TXT, TYT, true>, g, st, e0, e1, a);
}
template <typename T, int TXT, int TYT>
static void launch_nu_vc(int nu, Up2DArgs<T> &a, dim3 g, hipStream_t st, bool extra) {
  if (extra) {
    if (nu == 1) hipLaunchKernelGGL((k_mg_up2d<T, 1, 1, TXT, TYT, true>), g, dim3(kBlock), 0, st, a);
    else if (nu == 2) hipLaunchKernelGGL((k_mg_up2d<T, 2, 1, TXT, TYT, true>), g, dim3(kBlock), 0, st, a);
    else hipLaunchKernelGGL((k_mg_up2d<T, 3, 1, TXT, TYT, true>), g, dim3(kBlock), 0, st, a);
    return;
  }
  if (nu == 1) hipLaunchKernelGGL((k_mg_up2d<T, 1, 0, TXT, TYT, true>), g, dim3(kBlock), 0, st, a);
  else if (nu == 2) hipLaunchKernelGGL((k_mg_up2d<T, 2, 0, TXT, TYT, true>), g, dim3(kBlock), 0, st, a);
  else hipLaunchKernelGGL((k_mg_up2d<T, 3, 0, TXT, TYT, true>), g, dim3(kBlock), 0, st, a);
}
// Level 0 runs the large tile where it has enough of them, other levels the
// small one; the variable-coefficient kernels run the small tiles only.
template <typename T>
static void launch_nu(const PoissonWS &ws, int l, int nu, Down2DArgs<T> &a, hipStream_t st, hipEvent_t e0 = nullptr,
                      hipEvent_t e1 = nullptr) {
  const int tx = tile_x(ws, l), ty = tile_y(ws, l);
  const dim3 g(tiles2d(a.Lf, tx, ty));
  if (ws.vc) {
    if (tx == TXS && ty == TYS)
      launch_nu_vc<T, TXS, TYS>(nu, a, g, st, e0, e1);
    else
      launch_nu_vc<T, 16, 16>(nu, a, g, st, e0, e1);
    return;
  }
  if (tx == TX && ty == TY)
    launch_nu_t<T, TX, TY>(nu, a, g, st, e0, e1);
  else if (tx == TXS && ty == TYS)
    launch_nu_t<T, TXS, TYS>(nu, a, g, st, e0, e1);
  else
    launch_nu_t<T, 16, 16>(nu, a, g, st, e0, e1);
}
template <typename T>
static void launch_nu(const PoissonWS &ws, int l, int nu, Up2DArgs<T> &a, hipStream_t st, bool extra) {
  const int tx = tile_x(ws, l), ty = tile_y(ws, l);
  const dim3 g(tiles2d(a.Lf, tx, ty));
  if (ws.vc) {
    if (tx == TXS && ty == TYS)
      launch_nu_vc<T, TXS, TYS>(nu, a, g, st, extra);
    else
      launch_nu_vc<T, 16, 16>(nu, a, g, st, extra);
    return;
  }
  if (tx == TX && ty == TY)
    launch_nu_t<T, TX, TY>(nu, a, g, st, extra);
  else if (tx == TXS && ty == TYS)
    launch_nu_t<T, TXS, TYS>(nu, a, g, st, extra);
  else
    launch_nu_t<T, 16, 16>(nu, a, g, st, extra);
}

template <typename T>
static Down2DArgs<T> down_args(PoissonWS &ws, int l, int k, const void *b, T *xpre, double *x, const double *p,
                               const double *q, double *rnew) {
  Down2DArgs<T> a;
  const Lay &L = ws.lev[l].lay;
  a.Lf = L;
  a.Lc = ws.lev[l + 1].lay;
  a.B = ws.bnd;
  a.ihx = (T)ws.lev[l].ih2[0];
  a.ihy = (T)ws.lev[l].ih2[1];
  a.idg = (T)(1.0 / (2.0 * ws.lev[l].ih2[0] + 2.0 * ws.lev[l].ih2[1]));
  a.finest = (l == 0);
  a.k = k;
  a.b = b;
  a.xpre = xpre;
  a.bc = (T *)ws.lev[l + 1].b;
  a.x = x;
  a.p = p;
  a.q = q;
  a.rnew = rnew;
  a.part_pq = ws.part_pq;
  a.np_pq = kRedBlocks;
  a.sc = ws.sc;
  a.tiles_x = tiles_along(L.n[0], tile_x(ws, l));
  // single-reduction CG (finest level, FP64)
  a.cgcg = ws.cgcg && l == 0;
  a.u = (const T *)ws.z[0];
  a.w = ws.w;
  a.s_old = ws.s[k & 1];
  a.s_new = ws.s[(k + 1) & 1];
  a.p_io = ws.p[0];
  a.part_g = ws.part_rz;
  a.part_cc = ws.part_cc;
  a.np_g = fused_level(ws, 0) ? tiles2d(ws.lay, tile_x(ws, 0), tile_y(ws, 0)) : 0;
  a.np_cc = kRedBlocks;
  a.tol2 = ws.tol2;
  a.cfx = ws.vc ? (const T *)ws.cf[l][0] : nullptr;
  a.cfy = ws.vc ? (const T *)ws.cf[l][1] : nullptr;
  a.cig = ws.vc ? (const T *)ws.cf[l][2] : nullptr;
  return a;
}

template <typename T>
static Up2DArgs<T> up_args(PoissonWS &ws, int l, const T *xpre, const T *xc, const void *b, T *xout,
                           const T *zold) {
  Up2DArgs<T> a;
  const Lay &L = ws.lev[l].lay;
  a.Lf = L;
  a.Lc = ws.lev[l + 1].lay;
  a.B = ws.bnd;
  a.ihx = (T)ws.lev[l].ih2[0];
  a.ihy = (T)ws.lev[l].ih2[1];
  a.dihx = ws.lev[l].ih2[0];
  a.dihy = ws.lev[l].ih2[1];
  a.idg = (T)(1.0 / (2.0 * ws.lev[l].ih2[0] + 2.0 * ws.lev[l].ih2[1]));
  a.xpre = xpre;
  a.xc = xc;
  a.b = b;
  a.xout = xout;
  a.finest = (l == 0);
  a.zold = zold;
  a.part_rz = ws.part_rz;
  a.np = tiles2d(L, tile_x(ws, l), tile_y(ws, l));
  a.sc = ws.sc;
  a.tiles_x = tiles_along(L.n[0], tile_x(ws, l));
  a.w = ws.w;
  a.cfx = ws.vc ? (const T *)ws.cf[l][0] : nullptr;
  a.cfy = ws.vc ? (const T *)ws.cf[l][1] : nullptr;
  a.cig = ws.vc ? (const T *)ws.cf[l][2] : nullptr;
  a.rho64 = ws.vc ? ws.rho64 : nullptr;
  a.met = ws.met;
  return a;
}

template <typename T>
static CoarseArgs<T> coarse_args(PoissonWS &ws, void *z, const double *r) {
  CoarseArgs<T> ca;
  memset((void *)&ca, 0, sizeof(ca));
  const int nd = ws.lay.ndim, lc = ws.lc;
  ca.nq = ws.nlev - lc;
  ca.nu = ws.nu;
  for (int d = 0; d < 3; ++d) ca.per[d] = ws.bnd.periodic[d];
  ca.walls = !ws.bnd.all_periodic;
  int xo = 0, bo = 0;
  for (int q = 0; q < ca.nq; ++q) {
    const MGLevel &m = ws.lev[lc + q];
    BlkLevel<T> &L = ca.lev[q];
    const bool last = q + 1 == ca.nq;
    for (int d = 0; d < 3; ++d) {
      ca.nb[q][d] = last ? 0 : (d < nd ? m.lay.n[d] / 2 : 1);
      L.ih2[d] = (T)m.ih2[d];
    }
    L.nblk = ca.nb[q][0] * ca.nb[q][1] * ca.nb[q][2];
    L.xo = xo;
    L.bo = bo;
    L.go = ca.ngeo;
    L.co = (int)coarse_coef_offset(ws, lc + q);
    xo += last ? (int)m.lay.ncells() : (L.nblk + 1) << nd;
    if (q > 0) bo += last ? (int)m.lay.ncells() : (L.nblk + 1) << nd;
    ca.ngeo += L.nblk;
    L.xn = xo;
    L.bn = bo;
    for (int code = 0; code < 8; ++code) {
      double dg = 0.0;
      for (int d = 0; d < nd; ++d) dg += m.ih2[d] * (((code >> d) & 1) ? 2.0 : 1.0);
      ca.idg[q][code] = (T)(1.0 / dg);
    }
    L.idg = ca.idg[q][7];
    L.dg = (T)(2.0 * (m.ih2[0] + m.ih2[1] + (nd == 3 ? m.ih2[2] : 0.0)));
  }
  const Lay &Ll = ws.lev[ws.nlev - 1].lay;
  for (int d = 0; d < 3; ++d) ca.n_last[d] = Ll.n[d];
  ca.N_last = (int)Ll.ncells();
  ca.wave_q = ca.nq;
  if (ca.N_last <= kBlkPinv)  // then at least the level above the last has at most 64 blocks
    for (int q = ca.nq - 2; q >= 0 && ca.lev[q].nblk <= 64; --q) ca.wave_q = q;
  ca.L0 = ws.lev[lc].lay;
  ca.b0 = lc == 0 ? (const void *)r : ws.lev[lc].b;
  ca.b0_double = (lc == 0);
  ca.x0 = lc == 0 ? (T *)z : (T *)ws.lev[lc].x;
  ca.pinv = (const T *)(ws.vc ? ws.pinv_vc : ws.pinv);
  ca.cf = ws.vc ? (const T *)ws.ccf : nullptr;
  ca.geo = (BlkGeo *)ws.geo;
  return ca;
}

static hipError_t launch_geo(hipStream_t st, PoissonWS &ws) {
  const CoarseArgs<double> ca = coarse_args<double>(ws, nullptr, nullptr);
  if (ca.nq > 1) {
    const dim3 g(ceil_div(ca.lev[0].nblk, kBlock), ca.nq - 1);
    if (ws.lay.ndim == 3)
      hipLaunchKernelGGL((k_blk_geo<3, double>), g, dim3(kBlock), 0, st, ca);
    else
      hipLaunchKernelGGL((k_blk_geo<2, double>), g, dim3(kBlock), 0, st, ca);
  }
  return hipGetLastError();
}

// Pseudo-inverse of the coarsest operator: (L + J/N)^{-1} - J/N, where J is
// the all-ones matrix (L is singular with the constants as null space).
hipError_t poisson_setup(hipStream_t st, PoissonWS &ws, const double h0[3]) {
  (void)h0;
  const MGLevel &m = ws.lev[ws.nlev - 1];
  const Lay &L = m.lay;
  const long N = L.ncells();
  std::vector<double> A((size_t)N * N, 0.0), I((size_t)N * N, 0.0);
  auto idx = [&](int i, int j, int k) { return (long)i + (long)L.n[0] * (j + (long)L.n[1] * k); };
  for (int k = 0; k < L.n[2]; ++k)
    for (int j = 0; j < L.n[1]; ++j)
      for (int i = 0; i < L.n[0]; ++i) {
        const long r = idx(i, j, k);
        const int q[3] = {i, j, k};
        for (int d = 0; d < L.ndim; ++d) {
          for (int dir = -1; dir <= 1; dir += 2) {
            int qq[3] = {q[0], q[1], q[2]};
            qq[d] += dir;
            if (qq[d] < 0 || qq[d] >= L.n[d]) {
              if (!ws.bnd.periodic[d]) continue;
              qq[d] = (qq[d] + L.n[d]) % L.n[d];
            }
            const long cidx = idx(qq[0], qq[1], qq[2]);
            A[r * N + r] += m.ih2[d];
            A[r * N + cidx] -= m.ih2[d];
          }
        }
      }
  for (long a = 0; a < N * N; ++a) A[a] += 1.0 / (double)N;
  for (long a = 0; a < N; ++a) I[a * N + a] = 1.0;
  for (long col = 0; col < N; ++col) {  // Gauss-Jordan, partial pivoting
    long piv = col;
    for (long r = col + 1; r < N; ++r)
      if (std::fabs(A[r * N + col]) > std::fabs(A[piv * N + col])) piv = r;
    if (piv != col)
      for (long c = 0; c < N; ++c) {
        std::swap(A[col * N + c], A[piv * N + c]);
        std::swap(I[col * N + c], I[piv * N + c]);
      }
    const double d = A[col * N + col];
    for (long c = 0; c < N; ++c) {
      A[col * N + c] /= d;
      I[col * N + c] /= d;
    }
    for (long r = 0; r < N; ++r) {
      if (r == col) continue;
      const double f = A[r * N + col];
      if (f == 0.0) continue;
      for (long c = 0; c < N; ++c) {
        A[r * N + c] -= f * A[col * N + c];
        I[r * N + c] -= f * I[col * N + c];
      }
    }
  }
  for (long a = 0; a < N * N; ++a) I[a] -= 1.0 / (double)N;
  hipError_t e = launch_geo(st, ws);
  if (e != hipSuccess) return e;
  if (ws.mixed) {
    std::vector<float> f(I.begin(), I.end());
    e = hipMemcpyAsync(ws.pinv, f.data(), f.size() * 4, hipMemcpyHostToDevice, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
  } else {
    e = hipMemcpyAsync(ws.pinv, I.data(), I.size() * 8, hipMemcpyHostToDevice, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
  }
  return e;
}

template <int DIM, typename T>
static void launch_coarse(hipStream_t st, PoissonWS &ws, void *z, const double *r) {
  const dim3 g(1), b(kBlkThreads<DIM>);
  if (ws.vc)
    hipLaunchKernelGGL((k_mg_coarse<DIM, T, true>), g, b, 0, st, coarse_args<T>(ws, z, r), (const SolverScalars *)ws.sc);
  else
    hipLaunchKernelGGL((k_mg_coarse<DIM, T, false>), g, b, 0, st, coarse_args<T>(ws, z, r), (const SolverScalars *)ws.sc);
}

// Coefficient sets of the coarse-kernel levels lc .. lc + nq - 1 from the
// densities (or cell ratios) of the levels, into out.
template <int DIM, typename R>
static void launch_blk_coef(hipStream_t st, PoissonWS &ws, int nq, const R *const rho[], R *out) {
  BlkCoefArgs<R> a;
  memset((void *)&a, 0, sizeof(a));
  a.nq = nq;
  a.B = ws.bnd;
  a.met = ws.met;
  long most = 0;
  for (int q = 0; q < nq; ++q) {
    const MGLevel &m = ws.lev[ws.lc + q];
    a.L[q] = m.lay;
    a.rho[q] = rho[q];
    for (int d = 0; d < 3; ++d) a.ih2[q][d] = m.ih2[d];
    a.co[q] = (int)coarse_coef_offset(ws, ws.lc + q);
    most = std::max(most, m.lay.ncells() >> DIM);
  }
  if (nq > 0)
    hipLaunchKernelGGL((k_blk_coef<DIM, R>), dim3(ceil_div(most, kBlock), nq), dim3(kBlock), 0, st, a, out);
}

template <int DIM, typename T, bool UNIT>
static void launch_pinv(hipStream_t st, PoissonWS &ws, const T *rho, T *pinv) {
  const Lay &L = ws.lev[ws.nlev - 1].lay;
  auto k = L.ncells() <= 64 ? &k_vc_pinv<DIM, T, UNIT, 64> : &k_vc_pinv<DIM, T, UNIT, kVcCoarsest>;
  hipLaunchKernelGGL(k, dim3(1), dim3(kPinvThreads), 0, st, L, ws.bnd, ih2_of<double>(ws, ws.nlev - 1),
                     UNIT ? 0 : ws.met, rho, pinv);
}

// Face coefficients and coarsest pseudo-inverse of the variable-coefficient
// cycle, from the levels' densities (or cell ratios).
template <int DIM, typename T>
static void launch_coarse_setup(hipStream_t st, PoissonWS &ws) {
  const T *rho[kCoarseLev];
  const int nq = ws.nlev - 1 - ws.lc;
  for (int q = 0; q < nq; ++q) rho[q] = (const T *)ws.rho[ws.lc + q];
  launch_blk_coef<DIM, T>(st, ws, nq, rho, (T *)ws.ccf);
  if (ws.ccd && nq > 0) {
    const double *r64[1] = {ws.rho64};
    launch_blk_coef<DIM, double>(st, ws, 1, r64, ws.ccd);
  }
  launch_pinv<DIM, T, false>(st, ws, (const T *)ws.rho[ws.nlev - 1], (T *)ws.pinv_vc);
}

// In-step timing: events for this launch when it is the next timed launch
// of the selected kernel class (0 finest down, 1 finest up, 2 CG update);
// the caller records the iteration after launching.
static bool timed_launch(const PoissonWS &ws, int which, hipEvent_t &e0, hipEvent_t &e1) {
  e0 = e1 = nullptr;
  if (ws.twhich != which || ws.tcount >= ws.tcap) return false;
  e0 = ws.tev[2 * ws.tcount];
  e1 = ws.tev[2 * ws.tcount + 1];
  return true;
}

// An iteration is queued whole, or its head alone: up to and including the
// kernel that tests the convergence of r_{k-1} (the rest, its tail, would
// only find the solve done).
enum Part { kWhole, kHead, kTail };

// V-cycle of iteration k on b = r_k (finest), writing z = z_k.
template <int DIM, typename T>
static void vcycle(hipStream_t st, PoissonWS &ws, int k, const CGArgs &cg, Part part = kWhole) {
  const Bnd &B = ws.bnd;
  const int nu = ws.nu;
  const SolverScalars *sc = ws.sc;
  void *z = ws.z[k & 1];
  const double *r = ws.r[k & 1];
  const double *rprev = ws.r[(k + 1) & 1];
  dim3 bb(kBX, kBY);
  for (int l = 0; l < ws.lc; ++l) {
    const Lay &L = ws.lev[l].lay, &Lc = ws.lev[l + 1].lay;
    T *xin = lev_xin<T>(ws, l, z);
    if (l == 0 && part == kTail) continue;
    if (fused_level(ws, l)) {
      const void *b = l == 0 ? (k >= 1 ? (const void *)rprev : (const void *)r) : ws.lev[l].b;
      Down2DArgs<T> a = down_args<T>(ws, l, k, b, xin, cg.x, cg.pnew, cg.q, ws.r[k & 1]);
      hipEvent_t e0 = nullptr, e1 = nullptr;
      const bool timed = l == 0 && timed_launch(ws, 0, e0, e1);
      launch_nu<T>(ws, l, nu, a, st, e0, e1);
      if (timed) ws.tk[ws.tcount++] = k;
      if (part == kHead) return;
    } else if (fused3d(ws, l)) {
      Fused3DArgs<T> a = f3_args<T>(ws, l, l == 0 ? (const void *)r : ws.lev[l].b, l == 0);
      a.xout = xin;
      hipEvent_t e0 = nullptr, e1 = nullptr;
      const bool timed = l == 0 && timed_launch(ws, 0, e0, e1);
      launch_3d<T>(nu, true, a, st, false, e0, e1);
      if (timed) ws.tk[ws.tcount++] = k;
    } else {
      dim3 g = grid_for(L);
      const T *rl = ws.vc ? (const T *)ws.rho[l] : nullptr;
      for (int s = 0; s < nu; ++s) {
        for (int color = 0; color < 2; ++color) {
          if (l == 0)
            hipLaunchKernelGGL((k_mg_smooth<DIM, T, double>), g, bb, 0, st, L, B, ih2_of<T>(ws, l), xin, r, color,
                               s == 0 && color == 0, sc, rl, ws.met);
          else
            hipLaunchKernelGGL((k_mg_smooth<DIM, T, T>), g, bb, 0, st, L, B, ih2_of<T>(ws, l), xin,
                               (const T *)ws.lev[l].b, color, s == 0 && color == 0, sc, rl, ws.met);
        }
      }
      if (l == 0)
        hipLaunchKernelGGL((k_mg_restrict<DIM, T, double>), grid_for(Lc), bb, 0, st, L, Lc, B, ih2_of<T>(ws, l),
                           xin, r, (T *)ws.lev[l + 1].b, sc, rl, ws.met);
      else
        hipLaunchKernelGGL((k_mg_restrict<DIM, T, T>), grid_for(Lc), bb, 0, st, L, Lc, B, ih2_of<T>(ws, l), xin,
                           (const T *)ws.lev[l].b, (T *)ws.lev[l + 1].b, sc, rl, ws.met);
    }
  }
  launch_coarse<DIM, T>(st, ws, z, r);
  for (int l = ws.lc - 1; l >= 0; --l) {
    const Lay &L = ws.lev[l].lay, &Lc = ws.lev[l + 1].lay;
    T *xin = lev_xin<T>(ws, l, z);
    T *xout = lev_xout<T>(ws, l, z);
    const T *xc = lev_xout<T>(ws, l + 1, z);
    if (fused_level(ws, l)) {
      const T *zold = (l == 0 && !ws.cgcg && k >= 1) ? (const T *)ws.z[(k + 1) & 1] : nullptr;
      Up2DArgs<T> a = up_args<T>(ws, l, xin, xc, l == 0 ? (const void *)r : ws.lev[l].b, xout, zold);
      launch_nu<T>(ws, l, nu, a, st, ws.cgcg && l == 0);
    } else if (fused3d(ws, l)) {
      Fused3DArgs<T> a = f3_args<T>(ws, l, l == 0 ? (const void *)r : ws.lev[l].b, l == 0);
      a.xpre = xin;
      a.xc = xc;
      a.xout = xout;
      const bool extra = l == 0 && w_in_up3d(ws);
      a.part_rz = ws.part_rz;
      a.np = (int)blocks3d(L, ti3(nu, false, extra));
      hipEvent_t e0 = nullptr, e1 = nullptr;
      const bool timed = l == 0 && timed_launch(ws, 1, e0, e1);
      launch_3d<T>(nu, false, a, st, extra, e0, e1);
      if (timed) ws.tk[ws.tcount++] = k;
    } else {
      dim3 g = grid_for(L);
      const T *rl = ws.vc ? (const T *)ws.rho[l] : nullptr;
      hipLaunchKernelGGL((k_mg_prolong<DIM, T>), g, bb, 0, st, L, Lc, xin, xc, sc);
      for (int s = 0; s < nu; ++s) {
        for (int cc = 0; cc < 2; ++cc) {
          const int color = 1 - cc;
          if (l == 0)
            hipLaunchKernelGGL((k_mg_smooth<DIM, T, double>), g, bb, 0, st, L, B, ih2_of<T>(ws, l), xin, r, color, 0,
                               sc, rl, ws.met);
          else
            hipLaunchKernelGGL((k_mg_smooth<DIM, T, T>), g, bb, 0, st, L, B, ih2_of<T>(ws, l), xin,
                               (const T *)ws.lev[l].b, color, 0, sc, rl, ws.met);
        }
      }
    }
  }
  if (!fused_level(ws, 0)) {
    CGArgs a = cg;
    a.rnew = ws.r[k & 1];
    a.z = z;
    a.zold = (!ws.cgcg && k >= 1) ? ws.z[(k + 1) & 1] : nullptr;
    a.np_rz = kRedBlocks;
    if (ws.cgcg) {
      if (!w_in_up3d(ws)) hipLaunchKernelGGL((k_cgcg_w<DIM, T>), dim3(kRedBlocks), dim3(kBlock), 0, st, a);
    } else
      hipLaunchKernelGGL((k_cg_rz<DIM, T>), dim3(kRedBlocks), dim3(kBlock), 0, st, a);
  }
}

static int np_rz_of(const PoissonWS &ws) {
  if (fused_level(ws, 0)) return tiles2d(ws.lay, tile_x(ws, 0), tile_y(ws, 0));
  if (w_in_up3d(ws)) return (int)blocks3d_w(ws);
  return kRedBlocks;
}

template <int DIM, typename T>
static void iteration(hipStream_t st, PoissonWS &ws, CGArgs a, int k, Part part) {
  a.k = k;
  if (ws.cgcg) {
    // single-reduction CG: the update runs in the finest down kernel, or
    // in its own kernel when that level is not tiled
    const bool tiled = fused_level(ws, 0);
    if (!tiled) {
      a.z = ws.z[0];
      a.pold = ws.p[(k - 1) & 1];
      a.pnew = ws.p[k & 1];
      a.rold = ws.r[(k - 1) & 1];
      a.rnew = ws.r[k & 1];
      a.np_rz = np_rz_of(ws);
      hipEvent_t e0 = nullptr, e1 = nullptr;
      const bool timed = part != kTail && timed_launch(ws, 2, e0, e1);
      if (part != kTail) {
        auto upd = &k_cgcg_update<T>;
        if (DIM == 3) {
          // a run of planes per block: about four blocks of eight wavefronts
          // per compute unit, at least 8 planes (two more are read)
          const Lay &L = ws.lay;
          const int tx = tiles_along(L.n[0], kUX), ty = tiles_along(L.n[1], kUY);
          const int nch = std::max(1, 1024 / (tx * ty));
          const int tz = std::max(8, tiles_along(L.n[2], nch));
          const dim3 g(tx * ty * tiles_along(L.n[2], tz)), b(kUX * kUY);
          auto march = ws.vc ? &k_cgcg_march<T, 2> : (ws.bnd.all_periodic ? &k_cgcg_march<T, 0> : &k_cgcg_march<T, 1>);
          if (timed)
            hipExtLaunchKernelGGL(march, g, b, 0, st, e0, e1, 0, a, kRedBlocks, tx, ty, tz);
          else
            hipLaunchKernelGGL(march, g, b, 0, st, a, kRedBlocks, tx, ty, tz);
        } else if (timed) {
          hipExtLaunchKernelGGL(upd, dim3(kRedBlocks), dim3(kBlock), 0, st, e0, e1, 0, a, kRedBlocks);
        } else {
          hipLaunchKernelGGL(upd, dim3(kRedBlocks), dim3(kBlock), 0, st, a, kRedBlocks);
        }
      }
      if (timed) ws.tk[ws.tcount++] = k;
      if (part == kHead) return;
    }
    vcycle<DIM, T>(st, ws, k, a, tiled ? part : kWhole);
    return;
  }
  // pq(k): p_k = z_{k-1} + beta p_{k-1}
  a.z = ws.z[(k - 1) & 1];
  a.pold = ws.p[(k - 1) & 1];
  a.pnew = ws.p[k & 1];
  a.np_rz = np_rz_of(ws);
  a.flexible = !ws.cgcg;
  if (part != kTail)
    hipLaunchKernelGGL((k_cg_pq<DIM, T>), dim3(kRedBlocks), dim3(kBlock), 0, st, a, kRedBlocks);
  if (part == kHead) return;
  a.np_pq = kRedBlocks;
  if (!fused_level(ws, 0)) {
    a.rold = ws.r[(k - 1) & 1];
    a.rnew = ws.r[k & 1];
    hipLaunchKernelGGL((k_cg_update<DIM>), dim3(kRedBlocks), dim3(kBlock), 0, st, a);
  }
  vcycle<DIM, T>(st, ws, k, a);
}

// Waits for the scalars of the solve queued last, into ws.host_sc. The last
// kernel writes them to pinned memory, which is watched for a while (the wait
// ends some microseconds before a stream wait would); a solve that takes
// longer, or a context without such memory, waits for the stream.
static hipError_t await_scalars(hipStream_t st, PoissonWS &ws) {
  if (!ws.host_out) {
    const hipError_t e = hipMemcpyAsync(ws.host_sc, ws.sc, sizeof(SolverScalars), hipMemcpyDeviceToHost, st);
    return e == hipSuccess ? hipStreamSynchronize(st) : e;
  }
  const auto until = std::chrono::steady_clock::now() + std::chrono::milliseconds(200);
  while (__atomic_load_n(&ws.host_out->seq, __ATOMIC_ACQUIRE) != ws.seq) {
    for (int q = 0; q < 64; ++q) __builtin_ia32_pause();
    if (std::chrono::steady_clock::now() > until) {
      const hipError_t e = hipStreamSynchronize(st);
      if (e != hipSuccess) return e;
      if (__atomic_load_n(&ws.host_out->seq, __ATOMIC_ACQUIRE) != ws.seq) return hipErrorUnknown;
    }
  }
  memcpy((void *)ws.host_sc, (const void *)&ws.host_out->sc, sizeof(SolverScalars));
  return hipSuccess;
}

// The whole solve as one k_pcg_block launch (ws.block_pcg). With a log the
// outcome is left on the device for the caller to read later; without one
// this waits for it.
template <int DIM, typename T>
static hipError_t solve_block(hipStream_t st, PoissonWS &ws, const double *bvec, const double *x0, double rtol,
                              int maxit, int *iters, double *relres, int *converged, SolveLog *log,
                              AfterSolve after) {
  BlockPCGArgs<T> pa;
  pa.ca = coarse_args<T>(ws, ws.z[0], ws.r[0]);
  pa.L = ws.lay;
  pa.B = ws.bnd;
  for (int d = 0; d < 3; ++d) {
    pa.n[d] = ws.lay.n[d];
    pa.ih2[d] = ws.lev[0].ih2[d];
    pa.ih[d] = std::sqrt(ws.lev[0].ih2[d]);
  }
  pa.dg = 2.0 * (pa.ih2[0] + pa.ih2[1] + (DIM == 3 ? pa.ih2[2] : 0.0));
  pa.b = bvec;
  pa.x0 = x0;
  pa.x = ws.x;
  pa.rho = ws.vc ? ws.rho64 : nullptr;
  pa.met = ws.met;
  pa.vol = ws.met ? ws.vol : nullptr;
  pa.mean_w = ws.met ? ws.volume : (double)ws.lay.ncells();
  pa.tol2 = rtol * rtol;
  pa.maxit = maxit;
  pa.cd = ws.ccd;
  pa.sc = ws.sc;
  pa.log = log;
  pa.host = log ? nullptr : ws.host_out;
  pa.seq = log ? 0 : ++ws.seq;
  ws.tol2 = pa.tol2;
  const bool plain = pa.ca.nq == 1;
  auto k = ws.vc ? (plain ? &k_pcg_block<DIM, T, true, true> : &k_pcg_block<DIM, T, true, false>)
                 : (plain ? &k_pcg_block<DIM, T, false, true> : &k_pcg_block<DIM, T, false, false>);
  hipLaunchKernelGGL(k, dim3(1), dim3(kBlkThreads<DIM>), 0, st, pa);
  hipError_t e = hipGetLastError();
  if (e == hipSuccess && after) e = after();
  if (e != hipSuccess || log) return e;
  e = await_scalars(st, ws);
  if (e != hipSuccess) return e;
  const SolverScalars &h = *ws.host_sc;
  *iters = h.iters;
  *relres = h.cc > 0 ? std::sqrt(h.rr / h.cc) : 0.0;
  *converged = h.done && !h.nonconv;
  return hipSuccess;
}

template <int DIM, typename T>
static hipError_t solve_dim(hipStream_t st, PoissonWS &ws, const double *bvec, const double *x0, double rtol,
                            int maxit, int expect, int *iters, double *relres, int *converged, SolveLog *log,
                            AfterSolve after) {
  if (ws.block_pcg) return solve_block<DIM, T>(st, ws, bvec, x0, rtol, maxit, iters, relres, converged, log, after);
  if (log) return hipErrorInvalidValue;
  CGArgs a;
  a.L = ws.lay;
  a.B = ws.bnd;
  for (int d = 0; d < 3; ++d) {
    a.ih2[d] = ws.lev[0].ih2[d];
    a.ih[d] = std::sqrt(ws.lev[0].ih2[d]);
  }
  a.b = bvec;
  a.x0 = x0;
  a.x = ws.x;
  a.rold = nullptr;
  a.rnew = ws.r[0];
  a.pold = a.pnew = nullptr;
  a.q = ws.q;
  a.z = a.zold = nullptr;
  a.part_cc = ws.part_cc;
  a.part_pq = ws.part_pq;
  a.part_rz = ws.part_rz;
  a.np_rz = np_rz_of(ws);
  a.np_pq = kRedBlocks;
  a.sc = ws.sc;
  a.tol2 = rtol * rtol;
  ws.tol2 = a.tol2;
  a.k = 0;
  a.flexible = !ws.cgcg;
  a.rho = ws.vc ? ws.rho64 : nullptr;
  a.met = ws.met;
  a.vol = ws.met ? ws.vol : nullptr;
  ws.tsolve0 = ws.tcount;
  hipError_t e = hipMemsetAsync(&ws.sc->done, 0, 4 * sizeof(int), st);  // done, iters, zero, nonconv
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((k_cg_init<DIM>), grid_for(ws.lay), dim3(kBX, kBY), 0, st, a, ws.partials);
  hipLaunchKernelGGL(k_fold_partials, dim3(kRedBlocks), dim3(kBlock), 0, st, (const double *)ws.partials,
                     nblocks_for(ws.lay), ws.part_cc);
  vcycle<DIM, T>(st, ws, 0, a);
  // Whole iterations up to the expected count (without one: about 0.7 per
  // decade of the tolerance, what the V-cycle takes), then the head of the
  // next, which finds whether they sufficed, and the work after the solve,
  // gated on the outcome: the device goes on with it while the host reads the
  // flag. Too few iterations cost an empty pass of the gated kernels; one
  // iteration too many would cost its nine or more launches (2 us each).
  int k = 1;
  int batch = expect > 0 ? expect : (int)std::max(2.0, -0.7 * std::log10(rtol) + 0.5);
  for (int pass = 0;; ++pass) {
    for (int q = 0; q < batch && k <= maxit; ++q, ++k) iteration<DIM, T>(st, ws, a, k, kWhole);
    iteration<DIM, T>(st, ws, a, k, kHead);
    // mean of the solution (the stored pressure is zero-mean)
    hipLaunchKernelGGL((k_sum_x<DIM>), dim3(kRedBlocks), dim3(kBlock), 0, st, ws.lay, (const double *)ws.x,
                       ws.partials, ws.met ? (const double *)ws.vol : (const double *)nullptr,
                       (const SolverScalars *)ws.sc);
    hipLaunchKernelGGL(k_fin_mean_x, dim3(1), dim3(kBlock), 0, st, (const double *)ws.partials, kRedBlocks,
                       ws.met ? ws.volume : (double)ws.lay.ncells(), ws.sc, ws.host_out, ++ws.seq);
    e = hipGetLastError();
    if (e == hipSuccess && after) e = after();
    if (e == hipSuccess) e = await_scalars(st, ws);
    if (e != hipSuccess) return e;
    if (ws.host_sc->done || k > maxit) break;
    iteration<DIM, T>(st, ws, a, k, kTail);
    ++k;
    batch = std::min(pass, 2);
  }
  const SolverScalars &h = *ws.host_sc;
  *iters = h.iters;
  // timed launches of this solve that did the full work of a CG iteration
  // with a previous direction: iterations 2 .. iters (iteration 0 has no
  // CG update, iteration 1 no old p and s; later ones found the solve done)
  for (int q = ws.tsolve0; q < ws.tcount; ++q)
    if (ws.tk[q] < 2 || ws.tk[q] > h.iters) ws.tk[q] = -1;
  *relres = h.cc > 0 ? std::sqrt(h.rr / h.cc) : 0.0;
  *converged = h.done && !h.nonconv;
  return hipSuccess;
}

hipError_t poisson_solve(hipStream_t st, PoissonWS &ws, const double *b, const double *x0, double rtol,
                         int maxit, int expect_iters, int *iters, double *relres, int *converged, SolveLog *log,
                         AfterSolve after) {
  const bool three = ws.lay.ndim == 3;
  auto solve = ws.mixed ? (three ? &solve_dim<3, float> : &solve_dim<2, float>)
                        : (three ? &solve_dim<3, double> : &solve_dim<2, double>);
  return solve(st, ws, b, x0, rtol, maxit, expect_iters, iters, relres, converged, log, after);
}

// ---------------------------------------------------------------------------
// Variable-coefficient set-up
// ---------------------------------------------------------------------------
// Face coefficients of the tiled 2D levels.
template <typename T>
static void launch_coef2d(hipStream_t st, PoissonWS &ws) {
  for (int l = 0; l < ws.lc; ++l)
    if (ws.vtx[l] > 0)
      hipLaunchKernelGGL((k_vc_coef2d<T>), grid_for(ws.lev[l].lay), dim3(kBX, kBY), 0, st, ws.lev[l].lay, ws.bnd,
                         (T)ws.lev[l].ih2[0], (T)ws.lev[l].ih2[1], (const T *)ws.rho[l], (T *)ws.cf[l][0],
                         (T *)ws.cf[l][1], (T *)ws.cf[l][2], ws.met);
}

template <int DIM, typename T>
static hipError_t set_beta_dim(hipStream_t st, PoissonWS &ws) {
  const dim3 bb(kBX, kBY);
  const bool cast = sizeof(T) != 8;
  hipLaunchKernelGGL((k_vc_rho0<DIM, T>), grid_for(ws.lay), bb, 0, st, ws.lay, (const double *)ws.rho64,
                     cast ? (T *)ws.rho[0] : (T *)nullptr, ws.sc);
  for (int l = 0; l + 1 < ws.nlev; ++l) {
    const Lay &Lf = ws.lev[l].lay, &Lc = ws.lev[l + 1].lay;
    if (l == 0)
      hipLaunchKernelGGL((k_vc_rho_down<DIM, double, T>), grid_for(Lc), bb, 0, st, Lf, Lc,
                         (const double *)ws.rho64, (T *)ws.rho[1]);
    else
      hipLaunchKernelGGL((k_vc_rho_down<DIM, T, T>), grid_for(Lc), bb, 0, st, Lf, Lc, (const T *)ws.rho[l],
                         (T *)ws.rho[l + 1]);
  }
  if (DIM == 2) launch_coef2d<T>(st, ws);
  launch_coarse_setup<DIM, T>(st, ws);
  return hipGetLastError();
}

// Stretched 2D grid: the cell ratio dx/dy of every cell of a level (the
// cell array face_coef turns into the volume-weighted face coefficients)
// and, on the finest level, the cell volumes.
template <typename T>
__global__ void __launch_bounds__(kBlock) k_met_level(Lay L, const double *wx, const double *wy, T *ratio,
                                                      double *vol) {
  CellPos p;
  if (!cell_of_thread(L, p)) return;
  ratio[p.c] = (T)(wx[p.i] / wy[p.j]);
  if (vol) vol[p.c] = wx[p.i] * wy[p.j];
}

template <typename T>
static hipError_t set_metric_t(hipStream_t st, PoissonWS &ws) {
  const dim3 bb(kBX, kBY);
  long off = 0;
  for (int l = 0; l < ws.nlev; ++l) {
    const Lay &L = ws.lev[l].lay;
    const double *wx = ws.met_w + off, *wy = wx + L.n[0];
    off += L.n[0] + L.n[1];
    if (l == 0) {
      hipLaunchKernelGGL((k_met_level<double>), grid_for(L), bb, 0, st, L, wx, wy, ws.rho64, ws.vol);
      if (sizeof(T) != 8)
        hipLaunchKernelGGL((k_met_level<T>), grid_for(L), bb, 0, st, L, wx, wy, (T *)ws.rho[0], (double *)nullptr);
    } else {
      hipLaunchKernelGGL((k_met_level<T>), grid_for(L), bb, 0, st, L, wx, wy, (T *)ws.rho[l], (double *)nullptr);
    }
  }
  ws.vc = 1;
  launch_coef2d<T>(st, ws);
  launch_coarse_setup<2, T>(st, ws);
  return hipGetLastError();
}

hipError_t poisson_set_metric(hipStream_t st, PoissonWS &ws, const double *wx, const double *wy) {
  if (!ws.met || ws.lay.ndim != 2 || ws.lev[ws.nlev - 1].lay.ncells() > kVcCoarsest) return hipErrorInvalidValue;
  // widths of every level: a coarse cell spans its two children
  std::vector<double> all;
  std::vector<double> cx(wx, wx + ws.lay.n[0]), cy(wy, wy + ws.lay.n[1]);
  double V = 0.0;
  {
    double sx = 0.0, sy = 0.0;
    for (double v : cx) sx += v;
    for (double v : cy) sy += v;
    V = sx * sy;
  }
  for (int l = 0; l < ws.nlev; ++l) {
    all.insert(all.end(), cx.begin(), cx.end());
    all.insert(all.end(), cy.begin(), cy.end());
    std::vector<double> nx(cx.size() / 2), ny(cy.size() / 2);
    for (size_t q = 0; q < nx.size(); ++q) nx[q] = cx[2 * q] + cx[2 * q + 1];
    for (size_t q = 0; q < ny.size(); ++q) ny[q] = cy[2 * q] + cy[2 * q + 1];
    cx.swap(nx);
    cy.swap(ny);
  }
  ws.volume = V;
  hipError_t e = hipMemcpyAsync(ws.met_w, all.data(), all.size() * 8, hipMemcpyHostToDevice, st);
  if (e == hipSuccess) e = hipStreamSynchronize(st);
  if (e != hipSuccess) return e;
  return ws.mixed ? set_metric_t<float>(st, ws) : set_metric_t<double>(st, ws);
}

hipError_t poisson_setup_device(hipStream_t st, PoissonWS &ws) {
  if (ws.lev[ws.nlev - 1].lay.ncells() > kVcCoarsest) return hipErrorInvalidValue;
  const hipError_t e = launch_geo(st, ws);
  if (e != hipSuccess) return e;
  const float *f = nullptr;
  const double *d = nullptr;
  if (ws.lay.ndim == 3) {
    if (ws.mixed) launch_pinv<3, float, true>(st, ws, f, (float *)ws.pinv);
    else launch_pinv<3, double, true>(st, ws, d, (double *)ws.pinv);
  } else {
    if (ws.mixed) launch_pinv<2, float, true>(st, ws, f, (float *)ws.pinv);
    else launch_pinv<2, double, true>(st, ws, d, (double *)ws.pinv);
  }
  return hipGetLastError();
}

hipError_t poisson_set_beta(hipStream_t st, PoissonWS &ws) {
  if (!ws.vc_cap) return hipErrorInvalidValue;
  hipError_t e = hipMemsetAsync(&ws.sc->rho_bad, 0, sizeof(int), st);
  if (e != hipSuccess) return e;
  if (ws.lay.ndim == 3) return ws.mixed ? set_beta_dim<3, float>(st, ws) : set_beta_dim<3, double>(st, ws);
  return ws.mixed ? set_beta_dim<2, float>(st, ws) : set_beta_dim<2, double>(st, ws);
}

// ---------------------------------------------------------------------------
// Timing hook: one launch of a kernel class on scratch arrays
// ---------------------------------------------------------------------------
template <int DIM, typename T>
static hipError_t bench_launch_dim(hipStream_t st, PoissonWS &ws, int which) {
  CGArgs a;
  a.L = ws.lay;
  a.B = ws.bnd;
  for (int d = 0; d < 3; ++d) {
    a.ih2[d] = ws.lev[0].ih2[d];
    a.ih[d] = std::sqrt(ws.lev[0].ih2[d]);
  }
  a.b = ws.r[0];
  a.x0 = nullptr;
  a.x = ws.x;
  a.rold = ws.r[0];
  a.rnew = ws.r[1];
  a.pold = ws.p[0];
  a.pnew = ws.p[1];
  // (where A p is not stored: a vector that the kernel does not use otherwise)
  a.q = ws.q ? ws.q : (which == 2 ? ws.r[1] : ws.p[0]);
  a.z = ws.z[0];
  a.zold = nullptr;
  a.part_cc = ws.part_cc;
  a.part_pq = ws.part_pq;
  a.part_rz = ws.part_rz;
  a.np_rz = np_rz_of(ws);
  a.np_pq = kRedBlocks;
  a.sc = ws.sc;
  a.tol2 = 0.0;
  a.k = 2;
  a.flexible = 0;
  a.rho = nullptr;
  switch (which) {
    case 0: {  // finest-level down kernel (fused) or one half-sweep
      if (fused_level(ws, 0)) {
        Down2DArgs<T> d = down_args<T>(ws, 0, 2, ws.r[1], (T *)ws.zpre, ws.x, ws.p[0], ws.q, ws.r[0]);
        d.tol2 = 0.0;  // never converged: time the full kernel
        launch_nu<T>(ws, 0, ws.nu, d, st);
      } else {
        hipLaunchKernelGGL((k_mg_smooth<DIM, T, double>), grid_for(ws.lay), dim3(kBX, kBY), 0, st, ws.lay, ws.bnd,
                           ih2_of<T>(ws, 0), (T *)ws.z[0], (const double *)ws.r[0], 1, 0, ws.sc, (const T *)nullptr, 0);
      }
      break;
    }
    case 2: hipLaunchKernelGGL((k_cg_pq<DIM, T>), dim3(kRedBlocks), dim3(kBlock), 0, st, a, kRedBlocks); break;
    case 3: {  // finest-level up kernel (fused) or restriction
      if (ws.lc == 0) return hipErrorInvalidValue;
      if (fused_level(ws, 0)) {
        Up2DArgs<T> u = up_args<T>(ws, 0, (const T *)ws.zpre, lev_xout<T>(ws, 1, ws.z[0]), ws.r[0], (T *)ws.z[0],
                                   nullptr);
        launch_nu<T>(ws, 0, ws.nu, u, st, ws.cgcg);
      } else {
        hipLaunchKernelGGL((k_mg_restrict<DIM, T, double>), grid_for(ws.lev[1].lay), dim3(kBX, kBY), 0, st,
                           ws.lay, ws.lev[1].lay, ws.bnd, ih2_of<T>(ws, 0), (const T *)ws.z[0],
                           (const double *)ws.r[0], (T *)ws.lev[1].b, ws.sc, (const T *)nullptr, 0);
      }
      break;
    }
    case 4: hipLaunchKernelGGL((k_cg_update<DIM>), dim3(kRedBlocks), dim3(kBlock), 0, st, a); break;
    case 5:
      launch_coarse<DIM, T>(st, ws, ws.z[0], ws.r[0]);
      break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t poisson_bench_launch(hipStream_t st, PoissonWS &ws, int which) {
  if (ws.lay.ndim == 3)
    return ws.mixed ? bench_launch_dim<3, float>(st, ws, which) : bench_launch_dim<3, double>(st, ws, which);
  return ws.mixed ? bench_launch_dim<2, float>(st, ws, which) : bench_launch_dim<2, double>(st, ws, which);
}

}  // namespace lm
