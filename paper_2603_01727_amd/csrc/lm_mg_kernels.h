// Fused 2D multigrid level kernels that work out of LDS tiles with temporal
// blocking (one launch per level and direction of the V-cycle), in the
// constant-coefficient form (beta = 1) and, with VC, in the
// variable-coefficient form beta = 1/rho_f (face_beta), whose level operators
// are rediscretised from the level's density (2^d-cell averages). The last
// tiles of a row or column may reach beyond the grid: positions past a
// periodic side are halo copies of the cells they wrap to, positions past
// another side are absent cells, and neither is written.
// Included by lm_solver.hip only.
#pragma once

#include <type_traits>

namespace lm {

// ---------------------------------------------------------------------------
// Fused 2D tile kernels
// ---------------------------------------------------------------------------
template <typename T>
struct Down2DArgs {
  Lay Lf, Lc;
  Bnd B;
  T ihx, ihy, idg;          // 1/h^2 per direction; 1/diag for interior cells
  const void *b;            // right-hand side (FP64 r_{k-1} on the finest level)
  T *xpre, *bc;             // outputs: pre-smoothed x, coarse right-hand side
  // finest-level CG update (k >= 1)
  double *x;
  const double *p, *q;
  double *rnew;
  const double *part_pq;
  int np_pq;
  SolverScalars *sc;
  int k;                    // CG iteration (0: plain V-cycle on r_0)
  int finest;
  int tiles_x;
  // single-reduction CG (Chronopoulos-Gear): p, s, x, r updated here
  int cgcg;
  const T *u;               // z_{k-1} = M r_{k-1}
  const double *w;          // A u
  const double *s_old;      // s_{k-2}
  double *s_new, *p_io;     // s_{k-1}; p updated in place
  const double *part_g, *part_cc;  // [gamma | delta | rr] x np_g; ||c||^2 x np_cc
  int np_g, np_cc;
  double tol2;
  const T *cfx, *cfy, *cig;  // variable-coefficient kernels: west/south face beta, 1/diagonal
};

template <typename T>
struct Up2DArgs {
  Lay Lf, Lc;
  Bnd B;
  T ihx, ihy, idg;
  double dihx, dihy;  // FP64 1/h^2: w = A u is formed in FP64 whatever T is
  const T *xpre, *xc;
  const void *b;      // FP64 r_k on the finest level
  T *xout;
  const T *zold;      // flexible CG: z_{k-1}
  double *part_rz;    // finest level: [rz | rr | rzo] x np, or [r.u | w.u | rr] x np
  int np;
  const SolverScalars *sc;
  int finest;
  int tiles_x;
  double *w;          // single-reduction CG: w = A u written on the finest level
  const T *cfx, *cfy, *cig;  // variable-coefficient kernels: west/south face beta, 1/diagonal
  const double *rho64;  // the finest level's FP64 density (FP32 kernels: w = A u in FP64)
  int met;              // stretched grid: rho64 holds dx/dy (face_coef)
};

__device__ inline int wrap_or_out(int g, int n, int periodic) {
  if (g >= 0 && g < n) return g;
  if (!periodic) return -1;
  return g < 0 ? g + n : g - n;
}

// Index of own cell (gx, gy) of a tile; in = false (and a valid index) for a
// position of an edge tile beyond the grid (ALL: the tile is whole).
template <bool ALL>
__device__ inline long own_cell(const Lay &L, int gx, int gy, bool &in) {
  in = ALL || (gx < L.n[0] && gy < L.n[1]);
  return in ? L.at(gx, gy, 0) : L.base;
}
// Runs f with a compile-time flag for whole tiles: their stores need no
// per-cell test (with one, each store group is a branch of its own).
template <typename F>
__device__ __attribute__((always_inline)) inline void whole_or_edge(bool whole, F &&f) {
  if (whole)
    f(std::true_type());
  else
    f(std::false_type());
}

// True when every frame position is a cell with all four neighbours, so
// the sweeps need no boundary tests (periodic directions always qualify).
__device__ inline bool frame_interior(const Bnd &B, int gx0, int gy0, int W, int HH, int nx, int ny) {
  const bool okx = B.periodic[0] || (gx0 > 0 && gx0 + W < nx);
  const bool oky = B.periodic[1] || (gy0 > 0 && gy0 + HH < ny);
  return okx && oky;
}

// Gauss-Seidel value of an interior cell. A cell is updated by its owner and
// by the halos of its neighbours' tiles, and all must get the same bits (the
// single-reduction CG needs w = A u consistent with the stored u): in FP32
// the expression is evaluated exactly as written, without contraction into
// fused multiply-adds.
template <typename T>
__device__ inline T gs5(T b, T xw, T xe, T xs_, T xn, T ihx, T ihy, T idg) {
  return (b + (ihx * (xw + xe) + ihy * (xs_ + xn))) * idg;
}
template <>
__device__ inline float gs5<float>(float b, float xw, float xe, float xs_, float xn, float ihx, float ihy, float idg) {
#pragma clang fp contract(off)
  return (b + (ihx * (xw + xe) + ihy * (xs_ + xn))) * idg;
}

// Gauss-Seidel value at frame offset o, general case: raw global position
// (gx, gy) possibly outside a non-periodic side, in which case the cell does
// not exist (returns false). A cell with all four neighbours takes exactly
// the arithmetic of the interior path (gs5), so that a tile computing it in
// its halo gets the owner's bits whichever path either tile runs.
template <typename T, int W>
__device__ inline bool gs_general(const T *xs, const T *bs, int o, int gx, int gy, int nx, int ny, const Bnd &B,
                                  T ihx, T ihy, T idg, bool zero_nb, T &out) {
  if (!B.periodic[0] && (gx < 0 || gx >= nx)) return false;
  if (!B.periodic[1] && (gy < 0 || gy >= ny)) return false;
  const bool inx = B.periodic[0] || (gx > 0 && gx + 1 < nx);
  const bool iny = B.periodic[1] || (gy > 0 && gy + 1 < ny);
  if (inx && iny) {
    out = zero_nb ? bs[o] * idg : gs5<T>(bs[o], xs[o - 1], xs[o + 1], xs[o - W], xs[o + W], ihx, ihy, idg);
    return true;
  }
  T sx = T(0), sy = T(0);
  int cx = 0, cy = 0;
  if (B.periodic[0] || gx > 0) {
    if (!zero_nb) sx += xs[o - 1];
    ++cx;
  }
  if (B.periodic[0] || gx + 1 < nx) {
    if (!zero_nb) sx += xs[o + 1];
    ++cx;
  }
  if (B.periodic[1] || gy > 0) {
    if (!zero_nb) sy += xs[o - W];
    ++cy;
  }
  if (B.periodic[1] || gy + 1 < ny) {
    if (!zero_nb) sy += xs[o + W];
    ++cy;
  }
  out = (bs[o] + (ihx * sx + ihy * sy)) / (ihx * (T)cx + ihy * (T)cy);
  return true;
}

// (L x) at frame offset o (cell known to exist).
template <typename T, int W, typename A = T>
__device__ inline A lx_general(const T *xs, int o, int gx, int gy, int nx, int ny, const Bnd &B, A ihx, A ihy) {
  A sx = A(0), sy = A(0);
  int cx = 0, cy = 0;
  if (B.periodic[0] || gx > 0) {
    sx += (A)xs[o - 1];
    ++cx;
  }
  if (B.periodic[0] || gx + 1 < nx) {
    sx += (A)xs[o + 1];
    ++cx;
  }
  if (B.periodic[1] || gy > 0) {
    sy += (A)xs[o - W];
    ++cy;
  }
  if (B.periodic[1] || gy + 1 < ny) {
    sy += (A)xs[o + W];
    ++cy;
  }
  return (ihx * (A)cx + ihy * (A)cy) * (A)xs[o] - (ihx * sx + ihy * sy);
}

// Half-sweeps s = S0 .. S1 on shrinking regions [s, W-s) x [s, HH-s) of a
// W x HH frame; colour of half-sweep s is (s + cshift) & 1 (0 = red).
// Cells of one colour are enumerated directly (two per row pair), so the
// loop has compile-time bounds and no parity test.
template <typename T, int W, int HH, int S0, int S1, int CSHIFT>
__device__ inline void sweeps(T *xs, const T *bs, int p0, int gx0, int gy0, int nx, int ny, const Bnd &B, T ihx,
                              T ihy, T idg, bool fast, bool zero_first) {
  const int tid = threadIdx.x;
#pragma unroll
  for (int s = S0; s <= S1; ++s) {
    const int color = (s + CSHIFT) & 1;
    const int w = W - 2 * s, rows = HH - 2 * s;
    const int half = w / 2;
    const int cnt = half * rows;
    const bool zn = zero_first && s == S0;
    for (int o = tid; o < cnt; o += kBlock) {
      const int ly = s + o / half;
      const int lx = s + 2 * (o % half) + ((color + p0 + ly + s) & 1);
      const int off = ly * W + lx;
      if (fast) {
        if (zn)
          xs[off] = bs[off] * idg;
        else
          xs[off] = gs5<T>(bs[off], xs[off - 1], xs[off + 1], xs[off - W], xs[off + W], ihx, ihy, idg);
      } else {
        T v;
        if (gs_general<T, W>(xs, bs, off, gx0 + lx, gy0 + ly, nx, ny, B, ihx, ihy, idg, zn, v)) xs[off] = v;
      }
    }
    __syncthreads();
  }
}

// ---- variable-coefficient frames (beta = 1/rho_f) --------------------------
// The frame holds, per position, beta of the cell's west face (fx) and
// south face (fy) and 1/diagonal of L (ig), precomputed once per solve for
// the level (k_vc_coef2d), 0 for faces through non-periodic sides and for
// positions outside the grid: one branch-free update then serves interior
// and boundary cells, and leaves missing cells at 0.

// Gauss-Seidel value with face coefficients (evaluated as written, no
// contraction: halo copies of a cell get the owner's bits).
template <typename T>
__device__ inline T gs_vc(T b, T xw, T xe, T xs_, T xn, T bw, T be, T bs_, T bn, T ihx, T ihy, T ig) {
#pragma clang fp contract(off)
  return (b + (ihx * (bw * xw + be * xe) + ihy * (bs_ * xs_ + bn * xn))) * ig;
}

// (L x) at frame offset o with the frame's face coefficients.
template <typename T, int W, typename A = T>
__device__ inline A lx_vc(const T *xs, const T *fx, const T *fy, int o, A ihx, A ihy) {
#pragma clang fp contract(off)
  const A bw = fx[o], be = fx[o + 1], bs_ = fy[o], bn = fy[o + W];
  const A dg = ihx * (bw + be) + ihy * (bs_ + bn);
  return dg * (A)xs[o] -
         (ihx * (bw * (A)xs[o - 1] + be * (A)xs[o + 1]) + ihy * (bs_ * (A)xs[o - W] + bn * (A)xs[o + W]));
}

// FP64 (L u) at an own cell (gx, gy) of the finest level, the face
// coefficients from the FP64 density in global memory, u from the frame.
template <typename T, int W>
__device__ inline double lx_vc64(const T *xs, int o, const double *rho64, const Lay &L, const Bnd &B, int gx, int gy,
                                 double ihx, double ihy, int met) {
#pragma clang fp contract(off)
  const long c = L.at(gx, gy, 0);
  const int nx = L.n[0], ny = L.n[1];
  const long sy = L.s[1];
  const double rc = rho64[c];
  double bw = 0.0, be = 0.0, bs_ = 0.0, bn = 0.0;
  if (B.periodic[0] || gx > 0) bw = face_coef<double>(rc, rho64[gx > 0 ? c - 1 : c + (nx - 1)], 0, met);
  if (B.periodic[0] || gx + 1 < nx) be = face_coef<double>(rc, rho64[gx + 1 < nx ? c + 1 : c - (nx - 1)], 0, met);
  if (B.periodic[1] || gy > 0) bs_ = face_coef<double>(rc, rho64[gy > 0 ? c - sy : c + (long)(ny - 1) * sy], 1, met);
  if (B.periodic[1] || gy + 1 < ny) bn = face_coef<double>(rc, rho64[gy + 1 < ny ? c + sy : c - (long)(ny - 1) * sy], 1, met);
  const double dg = ihx * (bw + be) + ihy * (bs_ + bn);
  return dg * (double)xs[o] - (ihx * (bw * (double)xs[o - 1] + be * (double)xs[o + 1]) +
                               ihy * (bs_ * (double)xs[o - W] + bn * (double)xs[o + W]));
}

// Variable-coefficient half-sweeps, same regions and colours as sweeps().
template <typename T, int W, int HH, int S0, int S1, int CSHIFT>
__device__ inline void sweeps_vc(T *xs, const T *bs, const T *fx, const T *fy, const T *ig, int p0, T ihx, T ihy,
                                 bool zero_first) {
  const int tid = threadIdx.x;
#pragma unroll
  for (int s = S0; s <= S1; ++s) {
    const int color = (s + CSHIFT) & 1;
    const int w = W - 2 * s, rows = HH - 2 * s;
    const int half = w / 2;
    const int cnt = half * rows;
    const bool zn = zero_first && s == S0;
    for (int o = tid; o < cnt; o += kBlock) {
      const int ly = s + o / half;
      const int lx = s + 2 * (o % half) + ((color + p0 + ly + s) & 1);
      const int off = ly * W + lx;
      if (zn)
        xs[off] = bs[off] * ig[off];
      else
        xs[off] = gs_vc<T>(bs[off], xs[off - 1], xs[off + 1], xs[off - W], xs[off + W], fx[off], fx[off + 1], fy[off],
                           fy[off + W], ihx, ihy, ig[off]);
    }
    __syncthreads();
  }
}

// Down: [CG update] + NU red-black sweeps from zero + residual + restriction.
template <typename T, int NU, int TXT, int TYT, bool VC = false>
__global__ void __launch_bounds__(kBlock) k_mg_down2d(Down2DArgs<T> a) {
  static_assert((TXT * TYT) % kBlock == 0 && TXT % 2 == 0 && TYT % 2 == 0, "tile shape");
  constexpr int H = 2 * NU + 1;
  constexpr int W = TXT + 2 * H, HH = TYT + 2 * H;
  constexpr int WV = VC ? W * HH : 1;
  __shared__ T xs[W * HH];
  __shared__ T bs[W * HH];
  __shared__ T fx[WV], fy[WV], ig[WV];
  __shared__ double sh[kBlock / 64];
  const bool cg = a.finest && a.k >= 1;
  if (cg && a.cgcg ? ended_before(a.sc, a.k) : a.sc->done != 0) return;
  const int nx = a.Lf.n[0], ny = a.Lf.n[1];
  const int tile = xcd_remap(blockIdx.x, gridDim.x);
  const int gx0 = (tile % a.tiles_x) * TXT - H, gy0 = (tile / a.tiles_x) * TYT - H;
  const int p0 = (gx0 + gy0) & 1;
  const int tid = threadIdx.x;
  const bool fast = frame_interior(a.B, gx0, gy0, W, HH, nx, ny);
  const bool whole = gx0 + H + TXT <= nx && gy0 + H + TYT <= ny;
  double alpha = 0.0, beta = 0.0;
  if (cg && a.cgcg) {
    // gamma = r.u, delta = (A u).u, rr = r.r of iteration k-1: convergence
    // test, then alpha and beta of the single-reduction recurrence
    double cc, g, d, rr;
    sum_cc3(a.k, a.part_cc, a.np_cc, a.sc, a.part_g, a.part_g + a.np_g, a.part_g + 2 * a.np_g, a.np_g, cc, g, d, rr);
    const bool conv = (cc == 0.0) || (rr <= a.tol2 * cc);
    if (a.k == 1) {
      alpha = g / d;
    } else {
      beta = g / a.sc->rzh[(a.k - 2) & 1];
      alpha = g / (d - beta * g / a.sc->alh[(a.k - 2) & 1]);
    }
    const bool broken = !isfinite(rr) || !isfinite(alpha) || !isfinite(beta);
    if (blockIdx.x == 0 && tid == 0) {
      a.sc->rzh[(a.k - 1) & 1] = g;
      a.sc->alh[(a.k - 1) & 1] = alpha;
      a.sc->rr = rr;
      a.sc->cc = cc;
      a.sc->iters = a.k - 1;
      if (conv || broken) {
        a.sc->zero = (cc == 0.0);
        a.sc->nonconv = broken && !conv;
        a.sc->done = a.k + 1;
      }
    }
    if (conv || broken) return;
  } else if (cg) {
    const double pq = sum_all(a.part_pq, a.np_pq, sh);
    alpha = a.sc->rzh[(a.k - 1) & 1] / pq;
  }
  // right-hand side on the frame minus its outer ring; all loads of the
  // phase are issued before any is used (addresses of absent cells are
  // replaced by a valid one and the value discarded)
  constexpr int NPOS = W * HH;
  constexpr int NIT = (NPOS + kBlock - 1) / kBlock;
  long gi[NIT];
  bool ok[NIT];
#pragma unroll
  for (int it = 0; it < NIT; ++it) {
    const int o = tid + it * kBlock;
    const int lx = o % W, ly = o / W;
    const bool ring = (lx == 0 || ly == 0 || lx == W - 1 || ly == HH - 1);
    const int gx = wrap_or_out(gx0 + lx, nx, a.B.periodic[0]);
    const int gy = wrap_or_out(gy0 + ly, ny, a.B.periodic[1]);
    ok[it] = o < NPOS && !ring && gx >= 0 && gy >= 0;
    gi[it] = ok[it] ? a.Lf.at(gx, gy, 0) : a.Lf.base;
  }
  if constexpr (VC) {
    // coefficients on the whole frame (ring included), 0 for missing cells;
    // x starts at 0 everywhere (missing cells stay 0)
    T gv[NIT], fv[NIT], hv[NIT];
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
      const int o = tid + it * kBlock;
      const int gx = wrap_or_out(gx0 + o % W, nx, a.B.periodic[0]);
      const int gy = wrap_or_out(gy0 + o / W, ny, a.B.periodic[1]);
      const bool okr = o < NPOS && gx >= 0 && gy >= 0;
      const long id = okr ? a.Lf.at(gx, gy, 0) : a.Lf.base;
      gv[it] = a.cig[id];
      fv[it] = a.cfx[id];
      hv[it] = a.cfy[id];
      if (!okr) gv[it] = fv[it] = hv[it] = T(0);
    }
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
      const int o = tid + it * kBlock;
      if (o < NPOS) {
        ig[o] = gv[it];
        fx[o] = fv[it];
        fy[o] = hv[it];
        xs[o] = T(0);
      }
    }
  }
  if (a.finest && cg && a.cgcg) {
    // r_k = r_{k-1} - alpha (w + beta s_{k-2}) on the frame
    const double *rb = (const double *)a.b;
    const bool old = a.k >= 2;
    double rv[NIT], wv[NIT], sv[NIT];
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
      rv[it] = rb[gi[it]];
      wv[it] = a.w[gi[it]];
      sv[it] = old ? a.s_old[gi[it]] : 0.0;
    }
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
      const int o = tid + it * kBlock;
      if (o < NPOS) bs[o] = ok[it] ? (T)(rv[it] - alpha * (wv[it] + beta * sv[it])) : T(0);
    }
    // own cells: p = u + beta p, s = w + beta s, x += alpha p, r -= alpha s
    whole_or_edge(whole, [&](auto Wh) __attribute__((always_inline)) {
      constexpr bool ALL = decltype(Wh)::value;
      constexpr int NOWN = TXT * TYT / kBlock;
      long oi[NOWN];
      bool in[NOWN];
      double ro[NOWN], wo[NOWN], so[NOWN], xo[NOWN], po[NOWN];
      T uo[NOWN];
#pragma unroll
      for (int u = 0; u < NOWN; ++u) {
        const int o = tid + u * kBlock;
        oi[u] = own_cell<ALL>(a.Lf, gx0 + H + o % TXT, gy0 + H + o / TXT, in[u]);
      }
#pragma unroll
      for (int u = 0; u < NOWN; ++u) {
        ro[u] = rb[oi[u]];
        wo[u] = a.w[oi[u]];
        so[u] = old ? a.s_old[oi[u]] : 0.0;
        po[u] = old ? a.p_io[oi[u]] : 0.0;
        xo[u] = a.x[oi[u]];
        uo[u] = a.u[oi[u]];
      }
#pragma unroll
      for (int u = 0; u < NOWN; ++u) {
        const double pn = (double)uo[u] + beta * po[u];
        const double sn = wo[u] + beta * so[u];
        if (!in[u]) continue;
        a.p_io[oi[u]] = pn;
        a.s_new[oi[u]] = sn;
        a.x[oi[u]] = xo[u] + alpha * pn;
        a.rnew[oi[u]] = ro[u] - alpha * (wo[u] + beta * so[u]);
      }
    });
  } else if (a.finest) {
    const double *rb = (const double *)a.b;
    double rv[NIT], qv[NIT];
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
      rv[it] = rb[gi[it]];
      qv[it] = cg ? a.q[gi[it]] : 0.0;
    }
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
      const int o = tid + it * kBlock;
      if (o < NPOS) bs[o] = ok[it] ? (T)(rv[it] - alpha * qv[it]) : T(0);
    }
    if (cg) {  // CG update of the tile's own cells
      whole_or_edge(whole, [&](auto Wh) __attribute__((always_inline)) {
        constexpr bool ALL = decltype(Wh)::value;
        constexpr int NOWN = TXT * TYT / kBlock;
        long oi[NOWN];
        bool in[NOWN];
        double ro[NOWN], qo[NOWN], xo[NOWN], po[NOWN];
#pragma unroll
        for (int u = 0; u < NOWN; ++u) {
          const int o = tid + u * kBlock;
          oi[u] = own_cell<ALL>(a.Lf, gx0 + H + o % TXT, gy0 + H + o / TXT, in[u]);
        }
#pragma unroll
        for (int u = 0; u < NOWN; ++u) {
          ro[u] = rb[oi[u]];
          qo[u] = a.q[oi[u]];
          xo[u] = a.x[oi[u]];
          po[u] = a.p[oi[u]];
        }
#pragma unroll
        for (int u = 0; u < NOWN; ++u) {
          if (!in[u]) continue;
          a.rnew[oi[u]] = ro[u] - alpha * qo[u];
          a.x[oi[u]] = xo[u] + alpha * po[u];
        }
      });
    }
  } else {
    const T *bb = (const T *)a.b;
    T v[NIT];
#pragma unroll
    for (int it = 0; it < NIT; ++it) v[it] = bb[gi[it]];
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
      const int o = tid + it * kBlock;
      if (o < NPOS) bs[o] = ok[it] ? v[it] : T(0);
    }
  }
  __syncthreads();
  // zero initial guess: the first (red) half-sweep reads no neighbours, and
  // every later half-sweep only reads cells updated before it
  if constexpr (VC) {
    sweeps_vc<T, W, HH, 1, 2 * NU, 1>(xs, bs, fx, fy, ig, p0, a.ihx, a.ihy, true);
  } else {
    sweeps<T, W, HH, 1, 2 * NU, 1>(xs, bs, p0, gx0, gy0, nx, ny, a.B, a.ihx, a.ihy, a.idg, fast, true);
  }
  whole_or_edge(whole, [&](auto Wh) __attribute__((always_inline)) {
    for (int o = tid; o < TXT * TYT; o += kBlock) {
      const int lx = H + o % TXT, ly = H + o / TXT;
      bool in;
      const long c = own_cell<decltype(Wh)::value>(a.Lf, gx0 + lx, gy0 + ly, in);
      if (in) a.xpre[c] = xs[ly * W + lx];
    }
  });
  for (int o = tid; o < (TXT / 2) * (TYT / 2); o += kBlock) {
    const int cx = o % (TXT / 2), cy = o / (TXT / 2);
    const int Cx = (gx0 + H) / 2 + cx, Cy = (gy0 + H) / 2 + cy;
    if (Cx >= a.Lc.n[0] || Cy >= a.Lc.n[1]) continue;
    T acc = T(0);
#pragma unroll
    for (int dy = 0; dy < 2; ++dy)
#pragma unroll
      for (int dx = 0; dx < 2; ++dx) {
        const int lx = H + 2 * cx + dx, ly = H + 2 * cy + dy;
        const int off = ly * W + lx;
        T Lx;
        if constexpr (VC)
          Lx = lx_vc<T, W>(xs, fx, fy, off, a.ihx, a.ihy);
        else if (fast)
          Lx = (T(2) * (a.ihx + a.ihy)) * xs[off] - (a.ihx * (xs[off - 1] + xs[off + 1]) + a.ihy * (xs[off - W] + xs[off + W]));
        else
          Lx = lx_general<T, W>(xs, off, gx0 + lx, gy0 + ly, nx, ny, a.B, a.ihx, a.ihy);
        acc += bs[off] - Lx;
      }
    a.bc[a.Lc.at(Cx, Cy, 0)] = acc * T(0.25);
  }
}

// Up: prolongation + NU black-red sweeps; finest level: r.z, r.r partials.
// With EXTRA = 1 the frame carries one more halo ring, so the smoothed u is
// valid one cell beyond the tile and w = A u is formed for the tile
// (single-reduction CG: partials of r.u, w.u and r.r).
template <typename T, int NU, int EXTRA, int TXT, int TYT, bool VC = false>
__global__ void __launch_bounds__(kBlock) k_mg_up2d(Up2DArgs<T> a) {
  static_assert((TXT * TYT) % kBlock == 0 && TXT % 2 == 0 && TYT % 2 == 0, "tile shape");
  constexpr int H = 2 * NU + EXTRA;
  constexpr int W = TXT + 2 * H, HH = TYT + 2 * H;
  constexpr int WV = VC ? W * HH : 1;
  __shared__ T xs[W * HH];
  __shared__ T bs[W * HH];
  __shared__ T fx[WV], fy[WV], ig[WV];
  if (a.sc->done) return;
  const int nx = a.Lf.n[0], ny = a.Lf.n[1];
  const int tile = xcd_remap(blockIdx.x, gridDim.x);
  const int gx0 = (tile % a.tiles_x) * TXT - H, gy0 = (tile / a.tiles_x) * TYT - H;
  const int p0 = (gx0 + gy0) & 1;
  const int tid = threadIdx.x;
  const bool fast = frame_interior(a.B, gx0, gy0, W, HH, nx, ny);
  const bool whole = gx0 + H + TXT <= nx && gy0 + H + TYT <= ny;
  constexpr int NPOS = W * HH;
  constexpr int NIT = (NPOS + kBlock - 1) / kBlock;
  long gi[NIT], ci[NIT];
  bool okx[NIT], okb[NIT];
#pragma unroll
  for (int it = 0; it < NIT; ++it) {
    const int o = tid + it * kBlock;
    const int lx = o % W, ly = o / W;
    const int gx = wrap_or_out(gx0 + lx, nx, a.B.periodic[0]);
    const int gy = wrap_or_out(gy0 + ly, ny, a.B.periodic[1]);
    const bool ring = (lx == 0 || ly == 0 || lx == W - 1 || ly == HH - 1);
    okx[it] = o < NPOS && gx >= 0 && gy >= 0;
    okb[it] = okx[it] && !ring;
    gi[it] = okx[it] ? a.Lf.at(gx, gy, 0) : a.Lf.base;
    ci[it] = okx[it] ? a.Lc.at(gx >> 1, gy >> 1, 0) : a.Lc.base;
  }
  constexpr int NV = VC ? NIT : 1;
  T xv[NIT], cv[NIT], bv[NIT], gv[NV], fv[NV], hv[NV];
#pragma unroll
  for (int it = 0; it < NIT; ++it) {
    xv[it] = a.xpre[gi[it]];
    cv[it] = a.xc[ci[it]];
    bv[it] = a.finest ? (T)((const double *)a.b)[gi[it]] : ((const T *)a.b)[gi[it]];
    if constexpr (VC) {
      gv[it] = a.cig[gi[it]];
      fv[it] = a.cfx[gi[it]];
      hv[it] = a.cfy[gi[it]];
    }
  }
#pragma unroll
  for (int it = 0; it < NIT; ++it) {
    const int o = tid + it * kBlock;
    if (o < NPOS) {
      xs[o] = okx[it] ? xv[it] + cv[it] : T(0);
      bs[o] = okb[it] ? bv[it] : T(0);
      if constexpr (VC) {
        ig[o] = okx[it] ? gv[it] : T(0);
        fx[o] = okx[it] ? fv[it] : T(0);
        fy[o] = okx[it] ? hv[it] : T(0);
      }
    }
  }
  __syncthreads();
  // regions shrink from the frame edge, so with the extra ring the last
  // half-sweep leaves u valid on the tile plus one cell
  if constexpr (VC) {
    sweeps_vc<T, W, HH, 1, 2 * NU, 0>(xs, bs, fx, fy, ig, p0, a.ihx, a.ihy, false);
  } else {
    sweeps<T, W, HH, 1, 2 * NU, 0>(xs, bs, p0, gx0, gy0, nx, ny, a.B, a.ihx, a.ihy, a.idg, fast, false);
  }
  whole_or_edge(whole, [&](auto Wh) __attribute__((always_inline)) {
    constexpr bool ALL = decltype(Wh)::value;
    double rz = 0.0, rr = 0.0, rzo = 0.0;
    constexpr int NOWN = TXT * TYT / kBlock;
    long oi[NOWN];
    bool in[NOWN];
    T zv[NOWN];
#pragma unroll
    for (int u = 0; u < NOWN; ++u) {
      const int o = tid + u * kBlock;
      const int lx = H + o % TXT, ly = H + o / TXT;
      oi[u] = own_cell<ALL>(a.Lf, gx0 + lx, gy0 + ly, in[u]);
      zv[u] = in[u] ? xs[ly * W + lx] : T(0);
      if (in[u]) a.xout[oi[u]] = zv[u];
    }
    if (EXTRA && a.finest) {
      double rv[NOWN];
#pragma unroll
      for (int u = 0; u < NOWN; ++u) rv[u] = in[u] ? ((const double *)a.b)[oi[u]] : 0.0;
      double ru = 0.0, wu = 0.0;
#pragma unroll
      for (int u = 0; u < NOWN; ++u) {
        const int o = tid + u * kBlock;
        const int lx = H + o % TXT, ly = H + o / TXT;
        const int off = ly * W + lx;
        if (!in[u]) continue;
        double Lu;
        if constexpr (VC) {
          if constexpr (sizeof(T) == 8)
            Lu = lx_vc<T, W, double>(xs, fx, fy, off, a.dihx, a.dihy);
          else
            Lu = lx_vc64<T, W>(xs, off, a.rho64, a.Lf, a.B, gx0 + lx, gy0 + ly, a.dihx, a.dihy, a.met);
        } else if (fast) {
          Lu = (2.0 * (a.dihx + a.dihy)) * (double)xs[off] -
               (a.dihx * ((double)xs[off - 1] + (double)xs[off + 1]) + a.dihy * ((double)xs[off - W] + (double)xs[off + W]));
        } else {
          Lu = lx_general<T, W, double>(xs, off, gx0 + lx, gy0 + ly, nx, ny, a.B, a.dihx, a.dihy);
        }
        const double wv = Lu;
        a.w[oi[u]] = wv;
        ru += rv[u] * (double)zv[u];
        wu += wv * (double)zv[u];
        rr += rv[u] * rv[u];
      }
      double v3[3] = {ru, wu, rr};
      block_allsum_n<3>(v3);
      if (linear_tid() == 0) {
        a.part_rz[blockIdx.x] = v3[0];
        a.part_rz[a.np + blockIdx.x] = v3[1];
        a.part_rz[2 * a.np + blockIdx.x] = v3[2];
      }
      return;
    }
    if (a.finest) {
      double rv[NOWN];
      T zo[NOWN];
#pragma unroll
      for (int u = 0; u < NOWN; ++u) {
        rv[u] = in[u] ? ((const double *)a.b)[oi[u]] : 0.0;
        zo[u] = a.zold && in[u] ? a.zold[oi[u]] : T(0);
      }
#pragma unroll
      for (int u = 0; u < NOWN; ++u) {
        rz += rv[u] * (double)zv[u];
        rr += rv[u] * rv[u];
        rzo += rv[u] * (double)zo[u];
      }
    }
    if (a.finest) {
      double v3[3] = {rz, rr, rzo};  // rzo stays 0 without z_old
      block_allsum_n<3>(v3);
      if (linear_tid() == 0) {
        a.part_rz[blockIdx.x] = v3[0];
        a.part_rz[a.np + blockIdx.x] = v3[1];
        a.part_rz[2 * a.np + blockIdx.x] = v3[2];
      }
    }
  });
}

}  // namespace lm
