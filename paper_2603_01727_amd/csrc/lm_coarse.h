// One-workgroup multigrid V-cycle over the coarse levels (at most
// kCoarseCells cells), and the whole pressure solve in one workgroup for
// grids that such a cycle covers from the finest level. Included by
// lm_solver.hip only.
//
// Work split. A thread owns one 2^DIM block of cells, the children of one
// cell of the next level, and keeps their values in registers through a
// leg of the cycle. Of the neighbours a cell reads, one per direction is
// its own block's; the other belongs to the adjacent block and is read
// from LDS, where every sub-cell position of the blocks has an array of its
// own (lanes read consecutive words: no bank conflicts, and one set of 2 DIM
// block indices serves all cells and both colours). The restriction and the
// prolongation stay inside the thread but for the coarse value itself.
// Levels of at most 64 blocks run in the first wavefront alone, which needs
// no barriers. The pseudo-inverse of the coarsest level sits in LDS (at
// most 64 cells) or is read by columns of 64-lane rows (it is symmetric),
// eight loads in flight, 32 in 3D.
//
// What bounds it: latency (one workgroup; about 30 dependent phases of one
// LDS round trip and a few FP64 operations each), on the largest level the
// LDS rate (six 8-byte accesses per thread and half-sweep). Measured, FP64:
// a cycle from 64^2 as its own launch 12.9 us, the 64^2 solve of 8 iterations
// 101 us. (Two cells of one colour per thread, found through index sets in
// LDS with two-way bank conflicts, and the CG vectors in L2 scratch: 20.4 us
// and 203 us; with variable coefficients, the face divisions redone in every
// half-sweep, 37 us per cycle against 13.8 us, FP32.)
#pragma once

namespace lm {

// Threads of the one-workgroup kernels: one per block of the largest level
// (kCoarseCells / 2^DIM).
template <int DIM>
constexpr int kBlkThreads = DIM == 3 ? 512 : 1024;
static_assert(kCoarseCells <= 4L * kBlkThreads<2> && kCoarseCells <= 8L * kBlkThreads<3>, "one block per thread");

constexpr int kCoarseLds = 5504;  // cells of all coarse levels together (4096 + 1024 + ... in 2D)
constexpr int kCoarseLev = 8;     // coarse levels handled by the one-workgroup kernel, at most
// LDS elements: x of every level (2^DIM arrays of blocks + 1 entries each),
// right-hand sides of the levels below the first (of all, if there is one
// level only: at most kMaxCoarsest cells)
constexpr int kBlkX = kCoarseLds + 8 * kCoarseLev + 64;
constexpr int kBlkB = 1536;
constexpr int kBlkPinv = 64;          // coarsest cells whose pseudo-inverse is held in LDS
constexpr int kBlkP = kBlkPinv * kBlkPinv;  // ... or as many partial products of a larger one
constexpr int kBlkCoef = 5504;        // face coefficients of the levels below the first
constexpr int kBlkGeo = 1376;         // blocks of all levels (1024 + 256 + ... in 2D)
static_assert(kMaxCoarsest + 1 <= kBlkB && kMaxCoarsest <= kBlkP, "coarsest level in LDS");

// Entries of a block's coefficient set (variable coefficients): faces
// inside the block, outside faces of every cell, 1/diagonal of every cell.
template <int DIM>
constexpr int kBlkSlots = DIM * (1 << DIM) / 2 + DIM * (1 << DIM) + (1 << DIM);

// A level as a leg of the cycle needs it (one scalar load: wavefront-uniform).
template <typename T>
struct BlkLevel {
  int nblk;      // blocks (0 on the last level)
  int xo, bo;    // LDS offsets of x and the right-hand side ...
  int xn, bn;    // ... and those of the next level
  int go;        // first entry of the geometry table
  int co;        // first coefficient (variable coefficients; [slot][block])
  int pad;
  T ih2[3];
  T idg, dg;     // 1/diagonal and diagonal of a cell with all its neighbours
};

// Geometry of a block, made once per context for all levels (k_blk_geo):
// neighbour blocks (nblk: none, a slot that holds 0) and the place of its
// parent cell in the next level's arrays.
struct alignas(16) BlkGeo {
  unsigned short lo[3], hi[3], parent, in;  // in: bits 2d, 2d + 1: the low / high neighbour along d exists
};

template <typename T>
struct CoarseArgs {
  int nq, nu;               // coarse levels, smoothing sweeps
  int per[3];               // periodic directions
  int walls;                // some direction is not periodic
  int nb[kCoarseLev][3];    // blocks per direction of level q (= cells of level q + 1)
  int ngeo;                 // blocks of all levels
  int n_last[3], N_last;    // cells of the last level
  int wave_q;               // first level the first wavefront runs alone (nq: none)
  BlkLevel<T> lev[kCoarseLev];
  T idg[kCoarseLev][8];     // 1/diagonal by neighbour code (bit d: both neighbours along d exist)
  Lay L0;                   // global layout of the first level
  const void *b0;           // its right-hand side
  int b0_double;
  T *x0;                    // global output: its correction
  const T *pinv;            // dense pseudo-inverse of the last level
  const T *cf;              // variable coefficients: level q at lev[q].co
  BlkGeo *geo;              // geometry of every level's blocks
};

// q = t / n, r = t % n
__device__ inline int c_divmod(int t, int n, int &r) {
  if ((n & (n - 1)) == 0) {
    r = t & (n - 1);
    return t >> __builtin_ctz(n);
  }
  const int q = (int)((unsigned)t / (unsigned)n);
  r = t - q * n;
  return q;
}
// Coordinates of compact index t (x fastest) on an n[0] x n[1] x n[2] box.
template <int DIM>
__device__ inline void c_decode(const int n[3], int t, int &i, int &j, int &k) {
  k = 0;
  const int row = c_divmod(t, n[0], i);
  if (DIM == 3)
    k = c_divmod(row, n[1], j);
  else
    j = row;
}

constexpr int blk_parity(int a) { return (a ^ (a >> 1) ^ (a >> 2)) & 1; }
// Index of the face along d inside a block, of the pair that cell a is in.
template <int DIM>
constexpr int blk_face(int d, int a) {
  return d * ((1 << DIM) / 2) + ((a & ((1 << d) - 1)) | ((a >> (d + 1)) << d));
}

// A thread's block on one level.
template <int DIM, typename T, bool CF>
struct BlkGeom {
  int lo[DIM], hi[DIM], parent;
  T ig[1 << DIM];
  T ci[CF ? DIM * (1 << DIM) / 2 : 1], co[CF ? DIM * (1 << DIM) : 1];
};

// LDS of a cycle.
template <typename T, bool CF>
struct BlkShared {
  BlkGeo geo[kBlkGeo];
  T xs[kBlkX], bs[kBlkB], P[kBlkP], idg[kCoarseLev * 8];
  T cf[CF ? kBlkCoef : 1];
};

// Coefficients of block t from an [slot][nblk] array.
template <int DIM, typename T>
__device__ __attribute__((always_inline)) inline void blk_coef(const T *cf, int nblk, int t, BlkGeom<DIM, T, true> &g) {
  constexpr int NC = 1 << DIM;
  const T *c = cf + t;
#pragma unroll
  for (int e = 0; e < DIM * NC / 2; ++e) g.ci[e] = c[e * nblk];
#pragma unroll
  for (int e = 0; e < DIM * NC; ++e) g.co[e] = c[(DIM * NC / 2 + e) * nblk];
#pragma unroll
  for (int e = 0; e < NC; ++e) g.ig[e] = c[(DIM * NC / 2 + DIM * NC + e) * nblk];
}

// Geometry of block t of level q from the table (variable coefficients: the
// caller adds them).
template <int DIM, typename T, bool CF>
__device__ __attribute__((always_inline)) inline void blk_geom(const CoarseArgs<T> &a, const BlkLevel<T> &L, int q,
                                                               const BlkShared<T, CF> &sm, int t,
                                                               BlkGeom<DIM, T, CF> &g) {
  constexpr int NC = 1 << DIM;
  const BlkGeo e = sm.geo[L.go + t];
#pragma unroll
  for (int d = 0; d < DIM; ++d) {
    g.lo[d] = e.lo[d];
    g.hi[d] = e.hi[d];
  }
  g.parent = e.parent;
  if constexpr (!CF) {
    if (a.walls) {
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        int code = 0;
#pragma unroll
        for (int d = 0; d < DIM; ++d) code |= ((e.in >> (2 * d + ((c >> d) & 1))) & 1) << d;
        g.ig[c] = sm.idg[8 * q + code];
      }
    } else {
#pragma unroll
      for (int c = 0; c < NC; ++c) g.ig[c] = L.idg;
    }
  }
}

// acc plus the scaled neighbour sum of cell A of the block: the partner
// inside the block and the value v[d] from the adjacent one, per direction.
template <int DIM, int A, typename T, bool CF>
__device__ inline T blk_add_nbs(T acc, const T (&x)[1 << DIM], const T (&v)[DIM], const T ih2[3],
                                const BlkGeom<DIM, T, CF> &g) {
#pragma unroll
  for (int d = 0; d < DIM; ++d) {
    if constexpr (CF)
      acc += g.ci[blk_face<DIM>(d, A)] * x[A ^ (1 << d)] + g.co[DIM * A + d] * v[d];
    else
      acc += ih2[d] * (x[A ^ (1 << d)] + v[d]);
  }
  return acc;
}
// Diagonal of cell A without variable coefficients on a grid with walls:
// 1 + (outside neighbour exists) per direction.
template <int DIM, int A, typename T, bool CF, typename H>
__device__ inline T blk_wall_diag(const H ih2[3], int nblk, const BlkGeom<DIM, T, CF> &g) {
  T dg = T(0);
#pragma unroll
  for (int d = 0; d < DIM; ++d) dg += (T)ih2[d] * ((((A >> d) & 1) ? g.hi[d] : g.lo[d]) != nblk ? T(2) : T(1));
  return dg;
}

// The values outside the block that cell A's stencil reads.
template <int DIM, int A, typename T, bool CF>
__device__ inline void blk_outside(const T *X, int st, const BlkGeom<DIM, T, CF> &g, T (&v)[DIM]) {
#pragma unroll
  for (int d = 0; d < DIM; ++d) v[d] = X[(A ^ (1 << d)) * st + (((A >> d) & 1) ? g.hi[d] : g.lo[d])];
}

// One half-sweep (COLOR 0 red, 1 black) of x = (b + neighbours) / diag on
// the block, the new values published in LDS.
template <int DIM, int COLOR, typename T, bool CF>
__device__ __attribute__((always_inline)) inline void blk_half(T *X, int st, int t, const T (&b)[1 << DIM],
                                                               T (&x)[1 << DIM], const T ih2[3],
                                                               const BlkGeom<DIM, T, CF> &g) {
  constexpr int NC = 1 << DIM;
  T v[NC][DIM];
  static_for<0, NC>([&](auto A) __attribute__((always_inline)) {
    constexpr int c = decltype(A)::value;
    if constexpr (blk_parity(c) == COLOR) blk_outside<DIM, c, T, CF>(X, st, g, v[c]);
  });
  static_for<0, NC>([&](auto A) __attribute__((always_inline)) {
    constexpr int c = decltype(A)::value;
    if constexpr (blk_parity(c) == COLOR) {
      x[c] = blk_add_nbs<DIM, c, T, CF>(b[c], x, v[c], ih2, g) * g.ig[c];
      X[c * st + t] = x[c];
    }
  });
}

// Orders a phase's LDS writes before the next one's reads: a barrier, or
// inside one wavefront (whose LDS operations complete in order) only a fence
// for the compiler.
template <bool WAVE>
__device__ inline void blk_sync() {
  if constexpr (WAVE) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  } else {
    __syncthreads();
  }
}

// Pre-smoothing from zero (red first) and restriction. After the last black
// half-sweep the black cells' residuals vanish, so only the red children
// are summed. Ends with a sync.
template <int DIM, typename T, bool CF, bool WAVE>
__device__ __attribute__((always_inline)) inline void blk_down(const BlkLevel<T> &L, int nu, int walls, T *xs, T *bs, int t,
                                                               const T (&b)[1 << DIM],
                                                               const BlkGeom<DIM, T, CF> &g) {
  constexpr int NC = 1 << DIM;
  const int nblk = L.nblk, st = nblk + 1;
  T *X = xs + L.xo;
  const bool on = t < nblk;
  T x[NC];
  if (on) {
    static_for<0, NC>([&](auto A) __attribute__((always_inline)) {
      constexpr int c = decltype(A)::value;
      if constexpr (blk_parity(c) == 0) {
        x[c] = b[c] * g.ig[c];
        X[c * st + t] = x[c];
      }
    });
  }
  blk_sync<WAVE>();
  if (on) blk_half<DIM, 1, T, CF>(X, st, t, b, x, L.ih2, g);
  blk_sync<WAVE>();
#pragma unroll 1
  for (int s = 1; s < nu; ++s) {
    if (on) blk_half<DIM, 0, T, CF>(X, st, t, b, x, L.ih2, g);
    blk_sync<WAVE>();
    if (on) blk_half<DIM, 1, T, CF>(X, st, t, b, x, L.ih2, g);
    blk_sync<WAVE>();
  }
  if (on) {
    T acc = T(0);
    static_for<0, NC>([&](auto A) __attribute__((always_inline)) {
      constexpr int c = decltype(A)::value;
      if constexpr (blk_parity(c) == 0) {
        T v[DIM];
        blk_outside<DIM, c, T, CF>(X, st, g, v);
        T dg;
        if constexpr (CF) {
          dg = T(0);
#pragma unroll
          for (int d = 0; d < DIM; ++d) dg += g.ci[blk_face<DIM>(d, c)] + g.co[DIM * c + d];
        } else {
          dg = walls ? blk_wall_diag<DIM, c, T, CF>(L.ih2, nblk, g) : L.dg;
        }
        acc += blk_add_nbs<DIM, c, T, CF>(b[c], x, v, L.ih2, g) - dg * x[c];
      }
    });
    bs[L.bn + g.parent] = acc * (DIM == 3 ? T(0.125) : T(0.25));
  }
  blk_sync<WAVE>();
}

// Prolongation (piecewise constant; red cells only, the first half-sweep
// overwrites every black cell from its red neighbours) and post-smoothing
// (black first). x returns the level's correction. Ends with a sync.
template <int DIM, typename T, bool CF, bool WAVE>
__device__ __attribute__((always_inline)) inline void blk_up(const BlkLevel<T> &L, int nu, T *xs, int t,
                                                             const T (&b)[1 << DIM], T (&x)[1 << DIM],
                                                             const BlkGeom<DIM, T, CF> &g) {
  constexpr int NC = 1 << DIM;
  const int nblk = L.nblk, st = nblk + 1;
  T *X = xs + L.xo;
  const bool on = t < nblk;
  if (on) {
    const T xc = xs[L.xn + g.parent];
    static_for<0, NC>([&](auto A) __attribute__((always_inline)) {
      constexpr int c = decltype(A)::value;
      if constexpr (blk_parity(c) == 0) {
        x[c] = X[c * st + t] + xc;
        X[c * st + t] = x[c];
      }
    });
  }
  blk_sync<WAVE>();
#pragma unroll 1
  for (int s = 0; s < nu; ++s) {
    if (on) blk_half<DIM, 1, T, CF>(X, st, t, b, x, L.ih2, g);
    blk_sync<WAVE>();
    if (on) blk_half<DIM, 0, T, CF>(X, st, t, b, x, L.ih2, g);
    blk_sync<WAVE>();
  }
}

// Right-hand side, geometry and coefficients of the thread's block on level
// q, from LDS; right-hand side and coefficients of level 0 (b0, g0) from the
// caller's registers.
template <int DIM, typename T, bool CF>
__device__ __attribute__((always_inline)) inline void blk_enter(const CoarseArgs<T> &a, const BlkLevel<T> &L, int q,
                                                                const BlkShared<T, CF> &sm, int t,
                                                                const T (&b0)[1 << DIM],
                                                                const BlkGeom<DIM, T, CF> &g0, T (&b)[1 << DIM],
                                                                BlkGeom<DIM, T, CF> &g) {
  if (t >= L.nblk) return;
  if (q == 0) {
    if constexpr (CF) g = g0;
#pragma unroll
    for (int c = 0; c < (1 << DIM); ++c) b[c] = b0[c];
  } else {
#pragma unroll
    for (int c = 0; c < (1 << DIM); ++c) b[c] = sm.bs[L.bo + c * (L.nblk + 1) + t];
    if constexpr (CF) blk_coef<DIM, T>(sm.cf + (L.co - a.lev[1].co), L.nblk, t, g);
  }
  blk_geom<DIM, T, CF>(a, L, q, sm, t, g);
}

// x = pinv b on the last level, whole block. The columns of the symmetric
// pinv are dealt to groups of (rows rounded up to 64) threads; each thread
// sums its row over its group's columns, and the groups' sums are added.
// One unit's worth of wavefronts cannot hide the memory latency of such a
// matrix, so a thread issues U loads before it uses the first (420 cells, FP32,
// three levels: 17.9 us for the cycle with 32, 28.8 us with 8). In 2D the last
// levels are rarely above 64 cells and 8 keeps the registers down.
template <int DIM, typename T>
__device__ inline void blk_pinv(const CoarseArgs<T> &a, T *xl, const T *bl, T *part, int tid) {
  constexpr int NT = kBlkThreads<DIM>;
  constexpr int U = DIM == 3 ? 32 : 8;
  const int N = a.N_last;
  const int NP = min((N + 63) & ~63, NT);
  const int S = NT / NP;
  const int s = tid / NP, r0 = tid - s * NP;
  const int per = (N + S - 1) / S, c0 = s * per, c1 = min(c0 + per, N);
  if (s < S)  // (threads beyond the last whole group have no columns)
    for (int r = r0; r < N; r += NP) {
      T acc[4] = {T(0), T(0), T(0), T(0)};
      int c = c0;
#pragma unroll 1
      for (; c + U <= c1; c += U) {
        T m[U];
#pragma unroll
        for (int e = 0; e < U; ++e) m[e] = a.pinv[(long)(c + e) * N + r];
#pragma unroll
        for (int e = 0; e < U; ++e) acc[e & 3] += m[e] * bl[c + e];
      }
#pragma unroll 1
      for (; c < c1; c += 8) {
        T m[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) m[e] = a.pinv[(long)min(c + e, c1 - 1) * N + r];
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e & 3] += m[e] * (c + e < c1 ? bl[c + e] : T(0));
      }
      const T sum = (acc[0] + acc[1]) + (acc[2] + acc[3]);
      if (S == 1)
        xl[r] = sum;
      else
        part[s * NP + r] = sum;
    }
  __syncthreads();
  if (S > 1) {
    if (tid < N) {
      T acc = part[tid];
      for (int q = 1; q < S; ++q) acc += part[q * NP + tid];
      xl[tid] = acc;
    }
    __syncthreads();
  }
}

// The same in the first wavefront, from LDS (N_last <= 64).
template <typename T>
__device__ inline void blk_pinv_wave(int N, const T *P, T *xl, const T *bl, int t) {
  // sixteen columns' loads in flight
  T acc[4] = {T(0), T(0), T(0), T(0)};
  const int r = t < N ? t : 0;
  int c = 0;
#pragma unroll 1
  for (; c + 16 <= N; c += 16) {
    T m[16], v[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      m[e] = P[(c + e) * N + r];
      v[e] = bl[c + e];
    }
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[e & 3] += m[e] * v[e];
  }
#pragma unroll 1
  for (; c + 4 <= N; c += 4)
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[e] += P[(c + e) * N + r] * bl[c + e];
  for (; c < N; ++c) acc[0] += P[c * N + r] * bl[c];
  if (t < N) xl[t] = (acc[0] + acc[1]) + (acc[2] + acc[3]);
}

// Fills what a cycle expects in LDS: the geometry of every level's blocks,
// the zero slots, 1/diagonals, a small pseudo-inverse, the coefficients of
// the levels below the first. No sync. Only independent loads: one memory
// round trip.
template <int DIM, typename T, bool CF>
__device__ inline void blk_prepare(const CoarseArgs<T> &a, BlkShared<T, CF> &sm, int tid) {
  constexpr int NT = kBlkThreads<DIM>, NC = 1 << DIM;
  constexpr int NG = (kBlkGeo + NT - 1) / NT, NP = kBlkP / NT;
  static_assert(sizeof(BlkGeo) == sizeof(uint4), "one 16-byte load per entry");
  const uint4 *gg = (const uint4 *)a.geo;
  uint4 g[NG];
#pragma unroll
  for (int e = 0; e < NG; ++e) g[e] = gg[min(tid + e * NT, kBlkGeo - 1)];
  const int np = a.N_last <= kBlkPinv ? a.N_last * a.N_last : 0;
  T p[NP];
#pragma unroll
  for (int e = 0; e < NP; ++e) p[e] = a.pinv[max(min(tid + e * NT, np - 1), 0)];
  if constexpr (CF) {
    if (a.nq > 2) {
      const int n = a.lev[a.nq - 2].co + kBlkSlots<DIM> * a.lev[a.nq - 2].nblk - a.lev[1].co;
#pragma unroll 6
      for (int e = tid; e < n; e += NT) sm.cf[e] = a.cf[a.lev[1].co + e];
    }
  }
  if (tid < kCoarseLev * 8) sm.idg[tid] = a.idg[tid >> 3][tid & 7];
  {
    const int q = tid / NC;  // thread (q, c): the zero slot of sub-cell array c of level q
    if (q + 1 < a.nq) sm.xs[a.lev[q].xo + (tid - q * NC) * (a.lev[q].nblk + 1) + a.lev[q].nblk] = T(0);
  }
#pragma unroll
  for (int e = 0; e < NG; ++e)
    if (tid + e * NT < a.ngeo) *(uint4 *)&sm.geo[tid + e * NT] = g[e];
#pragma unroll
  for (int e = 0; e < NP; ++e)
    if (tid + e * NT < np) sm.P[tid + e * NT] = p[e];
}

// The geometry table: one thread per block, grid y = level.
template <int DIM, typename T>
__global__ void __launch_bounds__(kBlock) k_blk_geo(CoarseArgs<T> a) {
  const int q = blockIdx.y, nblk = a.lev[q].nblk;
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= nblk) return;
  const int *nb = a.nb[q];
  int b[3];
  c_decode<DIM>(nb, t, b[0], b[1], b[2]);
  BlkGeo g;
  g.in = 0;
  g.lo[2] = g.hi[2] = 0;
  int st = 1;
#pragma unroll
  for (int d = 0; d < DIM; ++d) {
    const bool l = b[d] > 0, h = b[d] + 1 < nb[d], p = a.per[d] != 0;
    g.lo[d] = (unsigned short)(l ? t - st : (p ? t + (nb[d] - 1) * st : nblk));
    g.hi[d] = (unsigned short)(h ? t + st : (p ? t - (nb[d] - 1) * st : nblk));
    g.in |= (unsigned short)((((l || p) ? 1 : 0) | ((h || p) ? 2 : 0)) << (2 * d));
    st *= nb[d];
  }
  if (q + 2 == a.nq) {
    g.parent = (unsigned short)t;  // the last level is in plain order
  } else {
    const int *nn = a.nb[q + 1];
    const int sub = (b[0] & 1) | ((b[1] & 1) << 1) | (DIM == 3 ? (b[2] & 1) << 2 : 0);
    g.parent = (unsigned short)(sub * (a.lev[q + 1].nblk + 1) + (b[0] >> 1) +
                                nn[0] * ((b[1] >> 1) + (DIM == 3 ? nn[1] * (b[2] >> 1) : 0)));
  }
  a.geo[a.lev[q].go + t] = g;
}

// The V-cycle from level 0 (at least two levels) on the right-hand side b0
// of the thread's block; x returns its correction, which the neighbours
// find in sm.xs. g0: the block's coefficients on level 0 (variable
// coefficients only). Ends with a barrier.
template <int DIM, typename T, bool CF>
__device__ __attribute__((always_inline)) inline void blk_cycle(const CoarseArgs<T> &a, BlkShared<T, CF> &sm, int tid,
                                                                const T (&b0)[1 << DIM], T (&x)[1 << DIM],
                                                                const BlkGeom<DIM, T, CF> &g0) {
  constexpr int NC = 1 << DIM;
  const int last = a.nq - 1, nu = a.nu;
  const int wq = a.wave_q;
  // (levels are indexed by a scalar, so their descriptors are scalar loads)
  auto level = [&](int q) __attribute__((always_inline)) { return a.lev[__builtin_amdgcn_readfirstlane(q)]; };
#pragma unroll 1
  for (int q = 0; q < wq && q < last; ++q) {
    const BlkLevel<T> L = level(q);
    BlkGeom<DIM, T, CF> g;
    T b[NC];
    blk_enter<DIM, T, CF>(a, L, q, sm, tid, b0, g0, b, g);
    blk_down<DIM, T, CF, false>(L, nu, a.walls, sm.xs, sm.bs, tid, b, g);
  }
  if (wq <= last) {
    if (tid < 64) {
#pragma unroll 1
      for (int q = wq; q < last; ++q) {
        const BlkLevel<T> L = level(q);
        BlkGeom<DIM, T, CF> g;
        T b[NC];
        blk_enter<DIM, T, CF>(a, L, q, sm, tid, b0, g0, b, g);
        blk_down<DIM, T, CF, true>(L, nu, a.walls, sm.xs, sm.bs, tid, b, g);
      }
      {
        const BlkLevel<T> L = level(last);
        blk_pinv_wave<T>(a.N_last, sm.P, sm.xs + L.xo, sm.bs + L.bo, tid);
      }
      blk_sync<true>();
#pragma unroll 1
      for (int q = last - 1; q >= wq; --q) {
        const BlkLevel<T> L = level(q);
        BlkGeom<DIM, T, CF> g;
        T b[NC];
        blk_enter<DIM, T, CF>(a, L, q, sm, tid, b0, g0, b, g);
        blk_up<DIM, T, CF, true>(L, nu, sm.xs, tid, b, x, g);
      }
    }
    __syncthreads();
  } else {
    const BlkLevel<T> L = level(last);
    blk_pinv<DIM, T>(a, sm.xs + L.xo, sm.bs + L.bo, sm.P, tid);
  }
#pragma unroll 1
  for (int q = min(wq, last) - 1; q >= 0; --q) {
    const BlkLevel<T> L = level(q);
    BlkGeom<DIM, T, CF> g;
    T b[NC];
    blk_enter<DIM, T, CF>(a, L, q, sm, tid, b0, g0, b, g);
    blk_up<DIM, T, CF, false>(L, nu, sm.xs, tid, b, x, g);
  }
}

// One cycle on a single level: x = pinv b in LDS, b in bs[bo[0]].. plain
// order (filled and synced by the caller). Ends with a barrier.
template <int DIM, typename T, bool CF>
__device__ inline void blk_single(const CoarseArgs<T> &a, BlkShared<T, CF> &sm, int tid) {
  if (a.N_last <= kBlkPinv) {
    if (tid < 64) blk_pinv_wave<T>(a.N_last, sm.P, sm.xs + a.lev[0].xo, sm.bs + a.lev[0].bo, tid);
    __syncthreads();
  } else {
    blk_pinv<DIM, T>(a, sm.xs + a.lev[0].xo, sm.bs + a.lev[0].bo, sm.P, tid);
  }
}

// The coarse levels of the multi-kernel V-cycle: right-hand side and
// correction of the first coarse level in global memory.
template <int DIM, typename T, bool CF>
__global__ void __launch_bounds__(kBlkThreads<DIM>) k_mg_coarse(CoarseArgs<T> a, const SolverScalars *sc) {
  constexpr int NC = 1 << DIM, NT = kBlkThreads<DIM>;
  __shared__ BlkShared<T, CF> sm;
  const int tid = threadIdx.x;
  const int stop = sc->done;
  if (a.nq == 1) {
    if (stop) return;  // one level, any sizes: the dense inverse alone
    for (int t = tid; t < a.N_last; t += NT) {
      int i, j, k;
      c_decode<DIM>(a.n_last, t, i, j, k);
      const long g = a.L0.at(i, j, k);
      sm.bs[a.lev[0].bo + t] = a.b0_double ? (T)((const double *)a.b0)[g] : ((const T *)a.b0)[g];
    }
    blk_prepare<DIM, T, CF>(a, sm, tid);
    __syncthreads();
    blk_single<DIM, T, CF>(a, sm, tid);
    for (int t = tid; t < a.N_last; t += NT) {
      int i, j, k;
      c_decode<DIM>(a.n_last, t, i, j, k);
      a.x0[a.L0.at(i, j, k)] = sm.xs[a.lev[0].xo + t];
    }
    return;
  }
  // the right-hand side is in flight while the tables are made
  const BlkLevel<T> L = a.lev[0];
  const bool on = tid < L.nblk;
  T b[NC], x[NC];
  BlkGeom<DIM, T, CF> g;
  long g0 = 0;
  if (on) {
    int i, j, k;
    c_decode<DIM>(a.nb[0], tid, i, j, k);
    g0 = a.L0.at(2 * i, 2 * j, DIM == 3 ? 2 * k : 0);
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const long p = g0 + (c & 1) + ((c >> 1) & 1) * a.L0.s[1] + (c >> 2) * a.L0.s[2];
      b[c] = a.b0_double ? (T)((const double *)a.b0)[p] : ((const T *)a.b0)[p];
    }
    if constexpr (CF) blk_coef<DIM, T>(a.cf + L.co, L.nblk, tid, g);
  }
  if (stop) return;
  blk_prepare<DIM, T, CF>(a, sm, tid);
  __syncthreads();
  blk_cycle<DIM, T, CF>(a, sm, tid, b, x, g);
  if (on)
#pragma unroll
    for (int c = 0; c < NC; ++c) a.x0[g0 + (c & 1) + ((c >> 1) & 1) * a.L0.s[1] + (c >> 2) * a.L0.s[2]] = x[c];
}

// ---------------------------------------------------------------------------
// Variable coefficients: the coefficient sets of the coarse levels' blocks
// ---------------------------------------------------------------------------
template <typename R>
struct BlkCoefArgs {
  int nq;
  Bnd B;
  int met;
  Lay L[kCoarseLev];         // level layouts
  const R *rho[kCoarseLev];  // densities (or cell ratios dx/dy)
  double ih2[kCoarseLev][3];
  int co[kCoarseLev];
};

// One thread per block, grid y = level: face coefficients 1/h^2 beta (0
// through a non-periodic side) and 1/diagonal in the order of BlkGeom.
template <int DIM, typename R>
__global__ void __launch_bounds__(kBlock) k_blk_coef(BlkCoefArgs<R> a, R *out) {
#pragma clang fp contract(off)
  constexpr int NC = 1 << DIM;
  const int q = blockIdx.y;
  const Lay &L = a.L[q];
  const int nb[3] = {L.n[0] >> 1, L.n[1] >> 1, DIM == 3 ? L.n[2] >> 1 : 1};
  const int nblk = nb[0] * nb[1] * nb[2];
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= nblk) return;
  int b[3];
  c_decode<DIM>(nb, t, b[0], b[1], b[2]);
  const R *rho = a.rho[q];
  R *o = out + a.co[q] + t;
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const int p[3] = {2 * b[0] + (c & 1), 2 * b[1] + ((c >> 1) & 1), 2 * b[2] + (c >> 2)};
    const long g = L.at(p[0], p[1], DIM == 3 ? p[2] : 0);
    R dg = R(0);
#pragma unroll
    for (int d = 0; d < DIM; ++d) {
      const R ih2 = (R)a.ih2[q][d];
      const int up = (c >> d) & 1;
      const long inner = up ? g - L.s[d] : g + L.s[d];
      const long outer = nbr(L, a.B, g, p[d], d, up ? 1 : -1);
      const R fi = ih2 * face_coef<R>(rho[g], rho[inner], d, a.met);
      const R fo = outer >= 0 ? ih2 * face_coef<R>(rho[g], rho[outer], d, a.met) : R(0);
      if (!up) o[(long)blk_face<DIM>(d, c) * nblk] = fi;
      o[(long)(DIM * NC / 2 + DIM * c + d) * nblk] = fo;
      dg += fi + fo;
    }
    o[(long)(DIM * NC / 2 + DIM * NC + c) * nblk] = R(1) / dg;
  }
}

// ---------------------------------------------------------------------------
// The whole solve in one workgroup
// ---------------------------------------------------------------------------
// The single-reduction preconditioned CG of the multi-kernel path (same
// recurrences, same stopping rule, FP64 vectors), every CG vector in the
// registers of the thread that owns the block (PLAIN: of the cells tid,
// tid + threads, ... of a grid that is its own coarsest level). One launch
// per solve and no host round trip between iterations.
template <typename T>
struct BlockPCGArgs {
  CoarseArgs<T> ca;         // the V-cycle from the finest level
  Lay L;                    // finest layout of the global vectors
  Bnd B;
  int n[3];
  double ih2[3], ih[3];     // finest 1/h^2, 1/h (FP64 operator)
  double dg;                // its diagonal away from walls
  const double *b, *x0;     // right-hand side; warm start (NULL: zero)
  double *x;                // solution (fine layout)
  const double *rho;        // variable coefficients / cell ratios (FP64, fine layout), or NULL
  int met;                  // stretched grid: rho holds dx/dy
  const double *vol;        // stretched grid: cell volumes, else NULL
  double mean_w;            // weight of the solution mean: volume or cell count
  double tol2;
  int maxit;
  const double *cd;         // FP64 coefficient sets of the finest level (variable coefficients)
  SolverScalars *sc;
  SolveLog *log;            // optional copy of the outcome (deferred checks)
  HostSolve *host;          // optional: pinned memory the host watches for the scalars, with their number
  unsigned seq;
};

// Sums of three values over the NT threads, in every thread. With 4
// wavefronts per SIMD the instructions of a full wavefront reduction of
// every value are what costs, so each wavefront only folds its rows of 16 to
// 4 lanes; wavefront q then adds value q's NT/4 partials. red: LDS.
template <int NT>
__device__ inline void block_sum3(double &v0, double &v1, double &v2, double *red) {
  constexpr int NP = NT / 4;
  double v[3] = {v0, v1, v2};
  const int t = threadIdx.x;
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    v[q] = dpp_add<0x118, 0xf>(v[q]);  // lanes 8 .. 15 of a row: pairs 8 apart
    v[q] = dpp_add<0x114, 0xf>(v[q]);  // lanes 12 .. 15: the row's four sums
  }
  // (the last call's results were read before the barriers of the cycle)
  if ((t & 12) == 12) {
#pragma unroll
    for (int q = 0; q < 3; ++q) red[q * NP + (t >> 4) * 4 + (t & 3)] = v[q];
  }
  __syncthreads();
  const int w = t >> 6;
  if (w < 3) {
    double s = 0.0;
#pragma unroll
    for (int e = 0; e < NP / 64; ++e) s += red[w * NP + e * 64 + (t & 63)];
    s = wave_sum(s);
    if ((t & 63) == 0) red[3 * NP + w] = s;
  }
  __syncthreads();
  v0 = red[3 * NP];
  v1 = red[3 * NP + 1];
  v2 = red[3 * NP + 2];
}

// The outcome in sc for the host (one thread).
template <typename T>
__device__ inline void tell_outcome(const BlockPCGArgs<T> &a) {
  const SolverScalars *sc = a.sc;
  if (a.log) {
    a.log->rr = sc->rr;
    a.log->cc = sc->cc;
    a.log->mean_b = sc->mean_b;
    a.log->iters = sc->iters;
    a.log->done = sc->done;
    a.log->nonconv = sc->nonconv;
  }
  if (a.host) host_write(a.host, sc, a.seq);
}

template <int DIM, typename T, bool CF, bool PLAIN>
__global__ void __launch_bounds__(kBlkThreads<DIM>) k_pcg_block(BlockPCGArgs<T> a) {
  constexpr int NC = 1 << DIM, NT = kBlkThreads<DIM>;
  constexpr int NV = PLAIN ? (int)(kMaxCoarsest + NT - 1) / NT : NC;  // cells per thread
  constexpr bool kD = sizeof(T) == 8;
  __shared__ BlkShared<T, CF> sm;
  __shared__ double red[3 * NT / 4 + 3];
  SolverScalars *sc = a.sc;
  const CoarseArgs<T> &ca = a.ca;
  const int tid = threadIdx.x;
  if (a.rho && sc->rho_bad) {  // invalid density: the solve ends at once
    if (tid == 0) {
      sc->rr = sc->cc = 0.0;
      sc->done = 1;
      sc->iters = 0;
      sc->nonconv = 1;
      sc->zero = 0;
      tell_outcome(a);
    }
    return;
  }
  blk_prepare<DIM, T, CF>(ca, sm, tid);
  const int N = a.n[0] * a.n[1] * a.n[2];
  if (PLAIN && tid == 0) sm.xs[ca.lev[0].xo + N] = T(0);  // the missing neighbour
  BlkGeom<DIM, T, CF> g0;
  int bi = 0, bj = 0, bk = 0;
  const bool on = PLAIN || tid < ca.lev[0].nblk;
  if (!PLAIN && on) {
    c_decode<DIM>(ca.nb[0], tid, bi, bj, bk);
    if constexpr (CF) blk_coef<DIM, T>(ca.cf + ca.lev[0].co, ca.lev[0].nblk, tid, g0);
  }
  // cell number c of this thread; false if there is none
  auto cell = [&](int c, int q[3]) __attribute__((always_inline)) -> bool {
    if constexpr (PLAIN) {
      const int t = tid + c * NT;
      if (t >= N) return false;
      c_decode<DIM>(a.n, t, q[0], q[1], q[2]);
      return true;
    } else {
      q[0] = 2 * bi + (c & 1);
      q[1] = 2 * bj + ((c >> 1) & 1);
      q[2] = DIM == 3 ? 2 * bk + (c >> 2) : 0;
      return on;
    }
  };
  // PLAIN: neighbour indices in the last level's order and FP64 coefficients
  int nbp[PLAIN ? NV : 1][2 * DIM];
  double cfp[PLAIN ? NV : 1][2 * DIM], dgp[PLAIN ? NV : 1];
  const double mb = sc->mean_b, oc = sc->outflow_c;
  double r[NV], x[NV], p[NV], s[NV];
  double cc = 0.0;
#pragma unroll
  for (int c = 0; c < NV; ++c) {
    r[c] = x[c] = p[c] = s[c] = 0.0;
    int q[3];
    if (!cell(c, q)) continue;
    const long g = a.L.at(q[0], q[1], q[2]);
    // r_0 = c - L x0 with c the mean-free (volume-weighted) right-hand side
    double bb = a.b[g] - mb;
#pragma unroll
    for (int d = 0; d < DIM; ++d) {
      if (a.B.kind[d][0] == LM_SIDE_OUTFLOW && q[d] == 0) bb -= oc * a.ih[d];
      if (a.B.kind[d][1] == LM_SIDE_OUTFLOW && q[d] == a.n[d] - 1) bb -= oc * a.ih[d];
    }
    const double cv = a.vol ? -(bb * a.vol[g]) : -bb;
    double Lx = 0.0;
    if (a.x0) {
      double nbs, dd;
      x[c] = a.x0[g];
      if constexpr (CF)
        op_parts_vc<DIM, double, double, double>(a.L, a.B, a.ih2, a.rho, a.x0, q[0], q[1], q[2], g, nbs, dd, a.met);
      else
        op_parts<DIM, double, double>(a.L, a.B, a.ih2, a.x0, q[0], q[1], q[2], g, nbs, dd);
      Lx = dd * x[c] - nbs;
    }
    r[c] = cv - Lx;
    cc += cv * cv;
    if constexpr (PLAIN) {
      const int t = tid + c * NT;
      int st = 1;
      dgp[c] = 0.0;
#pragma unroll
      for (int d = 0; d < DIM; ++d) {
        const int wrap = (a.n[d] - 1) * st;
        const bool per = a.B.periodic[d] != 0;
        const bool l = q[d] > 0, h = q[d] + 1 < a.n[d];
        nbp[c][2 * d] = l ? t - st : (per ? t + wrap : N);
        nbp[c][2 * d + 1] = h ? t + st : (per ? t - wrap : N);
        double bl = (l || per) ? 1.0 : 0.0, bh = (h || per) ? 1.0 : 0.0;
        if constexpr (CF) {
          if (l || per) bl = face_coef<double>(a.rho[g], a.rho[nbr(a.L, a.B, g, q[d], d, -1)], d, a.met);
          if (h || per) bh = face_coef<double>(a.rho[g], a.rho[nbr(a.L, a.B, g, q[d], d, +1)], d, a.met);
        }
        cfp[c][2 * d] = a.ih2[d] * bl;
        cfp[c][2 * d + 1] = a.ih2[d] * bh;
        dgp[c] += a.ih2[d] * (bl + bh);
        st *= a.n[d];
      }
    }
  }
  __syncthreads();  // the LDS set-up

  // u = M r (V-cycle), w = L u, and the three inner products of the
  // single-reduction recurrence
  // (the thread index through an opaque copy: what the cycle derives from it
  // is recomputed every iteration, not held in registers across them)
  double u[NV], w[NV];
  auto precondition = [&](double &gam, double &del, double &rr) __attribute__((always_inline)) {
    int tv = tid;
    asm volatile("" : "+v"(tv));
    gam = del = rr = 0.0;
    if constexpr (PLAIN) {
#pragma unroll
      for (int c = 0; c < NV; ++c)
        if (tid + c * NT < N) sm.bs[ca.lev[0].bo + tid + c * NT] = (T)r[c];
      __syncthreads();
      blk_single<DIM, T, CF>(ca, sm, tv);
      const T *X = sm.xs + ca.lev[0].xo;
#pragma unroll
      for (int c = 0; c < NV; ++c) {
        u[c] = w[c] = 0.0;
        if (tid + c * NT >= N) continue;
        u[c] = (double)X[tid + c * NT];
        double nbs = 0.0;
#pragma unroll
        for (int m = 0; m < 2 * DIM; ++m) nbs += cfp[c][m] * (double)X[nbp[c][m]];
        w[c] = dgp[c] * u[c] - nbs;
      }
    } else {
      T b[NC], xt[NC];
#pragma unroll
      for (int c = 0; c < NC; ++c) {
        b[c] = (T)r[c];
        xt[c] = T(0);
      }
      blk_cycle<DIM, T, CF>(ca, sm, tv, b, xt, g0);
      if (on) {
        const T *X = sm.xs + ca.lev[0].xo;
        const int nblk = ca.lev[0].nblk, st = nblk + 1;
        BlkGeom<DIM, T, CF> g;
        blk_geom<DIM, T, CF>(ca, ca.lev[0], 0, sm, tv, g);
        static_for<0, NC>([&](auto A) __attribute__((always_inline)) {
          constexpr int c = decltype(A)::value;
          T v[DIM];
          blk_outside<DIM, c, T, CF>(X, st, g, v);
          u[c] = (double)xt[c];
          double nbs = 0.0, dg = a.dg;
          if constexpr (CF)
            dg = 0.0;
          else if (ca.walls)
            dg = 0.0;
#pragma unroll
          for (int d = 0; d < DIM; ++d) {
            const double in = (double)xt[c ^ (1 << d)], out = (double)v[d];
            if constexpr (CF) {
              double fi, fo;
              if constexpr (kD) {
                fi = g0.ci[blk_face<DIM>(d, c)];
                fo = g0.co[DIM * c + d];
              } else {
                fi = a.cd[(long)blk_face<DIM>(d, c) * nblk + tid];
                fo = a.cd[(long)(DIM * NC / 2 + DIM * c + d) * nblk + tid];
              }
              nbs += fi * in + fo * out;
              dg += fi + fo;
            } else {
              nbs += a.ih2[d] * (in + out);
              if (ca.walls) dg += a.ih2[d] * ((((c >> d) & 1) ? g.hi[d] : g.lo[d]) != nblk ? 2.0 : 1.0);
            }
          }
          w[c] = dg * u[c] - nbs;
        });
      } else {
#pragma unroll
        for (int c = 0; c < NC; ++c) u[c] = w[c] = 0.0;
      }
    }
#pragma unroll
    for (int c = 0; c < NV; ++c) {
      gam += r[c] * u[c];
      del += w[c] * u[c];
      rr += r[c] * r[c];
    }
  };

  double gam = 0.0, del = 0.0, rr = 0.0;
  double g_prev = 0.0, al_prev = 0.0, alpha = 0.0, beta = 0.0;
  int iters = 0, done = 0, nonconv = 0;
#pragma unroll 1
  for (int k = 1; k <= a.maxit + 1; ++k) {
    // the cycle's first LDS writes follow the barriers of the last sums,
    // which follow every read of u
    precondition(gam, del, rr);
    block_sum3<NT>(gam, del, rr, red);
    if (k == 1) {
      double v1[1] = {cc};
      block_allsum_n<1>(v1);
      cc = v1[0];
    }
    const bool conv = (cc == 0.0) || (rr <= a.tol2 * cc);
    beta = 0.0;
    if (k == 1) {
      alpha = gam / del;
    } else {
      beta = gam / g_prev;
      alpha = gam / (del - beta * gam / al_prev);
    }
    const bool broken = !isfinite(rr) || !isfinite(alpha) || !isfinite(beta);
    iters = k - 1;
    if (conv || broken) {
      done = 1;
      nonconv = broken && !conv;
      break;
    }
    if (k == a.maxit + 1) break;  // out of iterations: not converged
    g_prev = gam;
    al_prev = alpha;
    // p = u + beta p, s = w + beta s, x += alpha p, r -= alpha s (beta, p
    // and s are 0 in the first iteration)
#pragma unroll
    for (int c = 0; c < NV; ++c) {
      p[c] = u[c] + beta * p[c];
      s[c] = w[c] + beta * s[c];
      x[c] += alpha * p[c];
      r[c] -= alpha * s[c];
    }
  }

  // the solution and its (volume-weighted) mean
  double sx = 0.0;
#pragma unroll
  for (int c = 0; c < NV; ++c) {
    int q[3];
    if (!cell(c, q)) continue;
    const long g = a.L.at(q[0], q[1], q[2]);
    a.x[g] = x[c];
    sx += a.vol ? x[c] * a.vol[g] : x[c];
  }
  {
    double v1[1] = {sx};
    block_allsum_n<1>(v1);
    sx = v1[0];
  }
  if (tid == 0) {
    sc->rr = rr;
    sc->cc = cc;
    sc->iters = iters;
    sc->done = done;
    sc->zero = (cc == 0.0);
    sc->nonconv = nonconv;
    sc->mean_x = sx / a.mean_w;
    tell_outcome(a);
  }
}

}  // namespace lm
