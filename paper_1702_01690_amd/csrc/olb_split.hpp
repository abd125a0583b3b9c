// olb_split.hpp -- the stage update split by velocity rows, for lattices too
// small to fill the chip with the stage kernel's tiles.  Included by
// olb_kernels.hip, whose node functions it shares.
//
// The stage kernel streams the 25 populations through one workgroup, a barrier
// each: about 20 us from the first load to the last store, whatever the
// lattice (FP64 32 x 32: 20.9 us a stage; the split kernel takes 8.4 us, of
// which the loads of a tile are a third and the face reconstructions another;
// with walls 28 against 10 us, in a box 31 against 10 us).  Here five groups of
// waves take the five velocity rows (ky) of a tile at the same time, with every
// population of the tile in LDS: a thread owns one node and the populations
// (0..4, ky), reconstructs their left and lower faces, and gathers their force
// term from the node's 25 values.  A sixth group takes the node's moments,
// force and equilibrium.  Each accumulator receives its terms in the stage
// kernel's order, so both give the same bits.
//
// split_stage_kernel  one RK stage, 16 x 8 tiles; wall ghosts are formed in LDS
//                     by the tiles at a wall (no wall launch)
// resident_kernel     whole RK-3 steps of lattices that fit one workgroup, f in
//                     LDS from the first stage to the last
#pragma once

namespace olbk {

// Between the steps of a thread's work: the values are computed here (left
// alone, the compiler sinks arithmetic to its use and keeps every step's LDS
// reads live until then), and the LDS reads of later steps stay after them.
template <typename V>
__device__ __forceinline__ void pin(V& v) { asm volatile("" : "+v"(v)); }
template <typename... V>
__device__ __forceinline__ void keep_order(V&... v) {
  (pin(v), ...);
  __builtin_amdgcn_sched_barrier(0);
}

// Equilibrium of one node in factors per axis, SLOTS values of type Real:
//   FP64: sn w_x (1 + hx) [5], w_y (1 + hy) [5]
//   FP32: px [5], qx [5], by [5], hy_w [5] (stage_tile)
template <typename Real>
constexpr int eq_slots() { return std::is_same<Real, float>::value ? 20 : 10; }

template <typename Real, typename Put>
__device__ __forceinline__ void put_equilibrium(const StageArgs& a, const MomSum& fsum, Put put) {
  constexpr bool F32 = std::is_same<Real, float>::value;
  double sn = fsum.n, se = fsum.e;
  if (F32) {
    sn += a.rho0;
    se = fmadd(2.0 * a.rho0, a.tref, se);
  }
  const double inv_n = 1.0 / sn;
  const double ux = fsum.jx * inv_n, uy = fsum.jy * inv_n;
  const double T = temperature(se, inv_n, ux, uy);
  double hx[5], hy[5];
  hfac(ux, T - 1.0, hx);
  hfac(uy, T - 1.0, hy);
  if constexpr (F32) {
    Fp32Equilibrium q;
    q.set(a, sn, hx, hy);
#pragma unroll
    for (int i = 0; i < 5; ++i) {
      put(i, q.px[i]);
      put(5 + i, q.qx[i]);
      put(10 + i, q.by[i]);
      put(15 + i, q.hy_w[i]);
    }
  } else {
#pragma unroll
    for (int i = 0; i < 5; ++i) {
      put(i, sn * (Wk[i] * (1.0 + hx[i])));
      put(5 + i, Wk[i] * (1.0 + hy[i]));
    }
  }
}

// New value of population (kx, ky) from its accumulator and those factors.
template <typename Real, typename Get>
__device__ __forceinline__ Real with_equilibrium(const StageArgs& a, Real acc, int kx, int ky, Get get) {
  if constexpr (std::is_same<Real, float>::value)
    return __builtin_fmaf(get(kx), get(10 + ky), __builtin_fmaf(get(5 + kx), get(15 + ky), acc));
  else
    return fmadd((a.B * a.dt) * a.inv_tau, get(kx) * get(5 + ky), acc);
}

// Force component along x (axis 0) or y (axis 1) of a node (Eq. F_def): p and
// n give the carried Delta p and n at an offset (l, m).
template <typename P, typename N>
__device__ __forceinline__ double node_force(const StageArgs& a, double inv_nc, P p, N n) {
  double g = 0.0, q = 0.0;
#pragma unroll
  for (int l = 1; l <= 3; ++l) {
#pragma unroll
    for (int m = -3; m <= 3; ++m) {
      const int am = m < 0 ? -m : m;
      if (GW[l][am] != 0.0) g = fmadd(l * GW[l][am], p(l, m) - p(-l, m), g);
      if (GL[l - 1][am] != 0.0) q = fmadd(GL[l - 1][am], n(l, m) - n(-l, m), q);
    }
    keep_order(g, q);
  }
  return fmadd(a.sigma, q * a.inv_ds3, (g * a.inv_ds) * inv_nc);
}

// WENO-5 face value from the five values v0 .. v4 in upwind order
__device__ __forceinline__ double face_value(const StageArgs& a, double v0, double v1, double v2, double v3, double v4) {
  return weno_rec(v0, v1, v2, v3, v4, a.wguard);
}
__device__ __forceinline__ float face_value(const StageArgs&, float v0, float v1, float v2, float v3, float v4) {
  return weno_rec(v0, v1, v2, v3, v4);
}
// and on the face between c[2] and c[3] for a velocity of the given sign (a
// constant at every call)
template <typename Real>
__device__ __forceinline__ Real face_value(const StageArgs& a, const Real (&c)[6], bool positive) {
  return positive ? face_value(a, c[0], c[1], c[2], c[3], c[4]) : face_value(a, c[5], c[4], c[3], c[2], c[1]);
}

// M, p_y and |p_y| by row, for kernels whose velocity row is a (uniform) value
struct RowTables {
  double m[5][5], p[5], speed[5];
};
constexpr RowTables make_row_tables() {
  RowTables t{};
  for (int k = 0; k < 5; ++k) {
    for (int j = 0; j < 5; ++j) t.m[k][j] = MT.v[k][j];
    t.p[k] = Rk[k];
    t.speed[k] = Rk[k] < 0.0 ? -Rk[k] : Rk[k];
  }
  return t;
}
__constant__ const RowTables row_tables = make_row_tables();

// The accumulators of one node's populations (0..4, row): the RK base term is
// in acc on entry; own and force terms and advection are added source by
// source in population order, as the stage kernel adds them.  f(ky, kx) is the
// node's value of a population, adv[kx] the advection difference of (kx, row).
// The row is a uniform value rather than a template argument, which would
// multiply the code of the faces by five and runs no faster.
template <typename Real, typename F>
__device__ __forceinline__ void row_terms(const StageArgs& a, int row, double Fx, double Fy, Real acc[5],
                                          const Real adv[5], F f) {
  constexpr bool F32 = std::is_same<Real, float>::value;
  const __attribute__((address_space(4))) float* const fbase =
      (const __attribute__((address_space(4))) float*)a.base;
  const double Bdt = a.B * a.dt;
  const Real cx = (Real)(-Bdt * Fx), cy = (Real)(-Bdt * Fy);
  const Real tfac = (Real)(a.B * fmadd(-a.dt, a.inv_tau, 1.0));
  const Real cadv = (Real)(-Bdt * a.inv_ds);
  // the five values of the next source row are read while one is added
  Real mrow[5], cur[5], next[5];
#pragma unroll
  for (int kx = 0; kx < 5; ++kx) {
    mrow[kx] = (Real)row_tables.m[row][kx];
    cur[kx] = f(0, kx);
  }
#pragma unroll
  for (int ky = 0; ky < 5; ++ky) {
#pragma unroll
    for (int kx = 0; kx < 5; ++kx) next[kx] = f(ky < 4 ? ky + 1 : 4, kx);
    const Real m = mrow[ky];
    Real ff[5], tfy[5];
#pragma unroll
    for (int kx = 0; kx < 5; ++kx) {
      ff[kx] = F32 ? cur[kx] + (Real)fbase[5 * ky + kx] : cur[kx];
      tfy[kx] = cy * ff[kx];
    }
    if (ky != row) {
#pragma unroll
      for (int kx = 0; kx < 5; ++kx) acc[kx] = fmadd(m, tfy[kx], acc[kx]);
    } else {
#pragma unroll
      for (int kx = 0; kx < 5; ++kx) {
        const Real tfx = cx * ff[kx];
        acc[kx] = fmadd(tfac, cur[kx], acc[kx]);
        // the population's own x and y terms come in the order of the smaller
        // of its two target indices (x first on a tie)
        if (kx > row) acc[kx] = fmadd(m, tfy[kx], acc[kx]);
#pragma unroll
        for (int i = 0; i < 5; ++i) acc[i] = fmadd((Real)MT.v[i][kx], tfx, acc[i]);
        if (kx <= row) acc[kx] = fmadd(m, tfy[kx], acc[kx]);
        if (!(kx == 2 && row == 2)) acc[kx] = fmadd(cadv, adv[kx], acc[kx]);
      }
    }
#pragma unroll
    for (int kx = 0; kx < 5; ++kx) cur[kx] = next[kx];
    keep_order(acc[0], acc[1], acc[2], acc[3], acc[4]);
  }
}

// Carried (n, Delta p) and, on request, the sums themselves of a node's 25
// values.
template <typename F>
__device__ __forceinline__ MomSum node_sums(F f) {
  MomSum s;
#pragma unroll
  for (int k = 0; k < 25; ++k) {
    s.add(k, (double)f(k));
    if (k % 5 == 4) keep_order(s.n, s.jx, s.jy, s.e);
  }
  return s;
}

// --------------------------------------------------------------------------
// ghost rows of LDS-held lattices (walls_kernel's arithmetic)
// --------------------------------------------------------------------------

// One wall side of a block of LDS columns: rows r0, r1, r2 are the interior
// rows next to the wall, g[j] the ghost rows (-1: not held).  Two passes with
// a barrier between them: the extrapolated (or mirrored) rows and each
// column's ten face fluxes, then n_w and the emitted rows.
struct WallSide {
  int high;            // 0: low end of y, 1: high end
  int r0, r1, r2, g[3];
};

// pass 1 of population k of a column: at(k, row) is its LDS value; rec
// receives the wall-face value of populations moving towards the wall
template <typename Real, typename At>
__device__ __forceinline__ void wall_pass1(const InstDesc& d, const WallSide& w, int k, At at, double& rec) {
  const int kx = k % 5, ky = k / 5;
  rec = 0.0;
  if (!w.high && d.g.walls == 2) {
    const int km = 5 * (4 - ky) + kx;
    const int rows[3] = {w.r0, w.r1, w.r2};
#pragma unroll
    for (int j = 0; j < 3; ++j)
      if (w.g[j] >= 0) at(k, w.g[j]) = at(km, rows[j]);
    return;
  }
  if (w.high ? ky < 2 : ky > 2) return;
  const Real v0 = at(k, w.r0), v1 = at(k, w.r1), v2 = at(k, w.r2);
  Real e[3];
  wall_extrapolate(v0, v1, v2, e[0], e[1], e[2]);
#pragma unroll
  for (int j = 0; j < 3; ++j)
    if (w.g[j] >= 0) at(k, w.g[j]) = e[j];
  if (ky != 2) rec = (double)weno_rec(v2, v1, v0, e[0], e[1]);
}

// pass 2: n_w of a column (Eq. nw; recs(j, kx): its wall-face values; the
// denominator sums g_kx(u_w, T_w) g_ky(0, T_w) p_ky over the wall-emitted
// velocities, and sum_kx g_kx = 1 leaves sum_ky g_ky(0, T_w) p_ky), and the
// value of an emitted population
template <typename Real>
struct WallEmission {
  static constexpr bool F32 = std::is_same<Real, float>::value;
  double bw[5], wx[5], wy[5], den;   // base factors, w (1 + h) of the wall state per axis
  __device__ __forceinline__ void set(const InstDesc& d, int high) {
    double h0[5], hx[5], hy[5];
    base_h0(d.tref, h0);
    hfac(d.uw[high], d.tw[high] - 1.0, hx);
    hfac(0.0, d.tw[high] - 1.0, hy);
    den = 0.0;
#pragma unroll
    for (int i = 0; i < 5; ++i) {
      bw[i] = Wk[i] * (1.0 + h0[i]);
      wx[i] = Wk[i] * (1.0 + hx[i]);
      wy[i] = Wk[i] * (1.0 + hy[i]);
      if (high ? i < 2 : i > 2) den = fmadd(wy[i], Rk[i], den);
    }
  }
  template <typename Recs>
  __device__ __forceinline__ double density(const InstDesc& d, int high, Recs recs) const {
    double out = 0.0;
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int kx = 0; kx < 5; ++kx) {
        const double p = high ? Rk[3 + j] : Rk[j], by = high ? bw[3 + j] : bw[j];
        double rec = recs(j, kx);
        if (F32) rec = fmadd(bw[kx] * by, d.rho0, rec);
        out = fmadd(p, rec, out);
      }
    return -out / den;
  }
  // emitted population (kx, 3 + j) at the low end, (kx, j) at the high end
  __device__ __forceinline__ Real value(const InstDesc& d, int high, double nw, int kx, int j) const {
    auto pick = [&](const double* v) { return high ? (j ? v[1] : v[0]) : (j ? v[4] : v[3]); };
    double v = (nw * wx[kx]) * pick(wy);
    if (F32) v = fmadd(-(bw[kx] * pick(bw)), d.rho0, v);
    return (Real)v;
  }
};

// --------------------------------------------------------------------------
// one stage, 16 x 8 tiles
// --------------------------------------------------------------------------

// Threads: six groups of two waves, a lane per node (16 columns x 4 rows per
// wave), three waves on every SIMD.  All 25 planes of the tile and its 3-node
// halo sit in LDS (61.6 KB in FP64, two workgroups per CU).  Groups 0..4 take
// the velocity rows; row 2 has no y faces and reconstructs the tile's extra
// faces instead (320 across y, 160 across x, at most four per lane).  Group 5
// takes the moments, the force and the equilibrium meanwhile, and the carry at
// the end.  Once every face is reconstructed the halo rows are dead, and the
// faces are handed over through them.
//
// Planes of the rows with p_y < 0 are kept upside down (row r of the tile at
// LDS row SPH - 1 - r): their upwind side is then below too, a thread's own
// face is the one below it in LDS, and p_y (f_up - f_down) is |p_y| times
// (next face - own face) in every row, to the bit.
constexpr int SPW = SPLIT_X + 6, SPH = SPLIT_Y + 6, SPN = SPW * SPH;
constexpr int SPLIT_NODES = SPLIT_X * SPLIT_Y;
constexpr int SPLIT_THREADS = 6 * SPLIT_NODES;
static_assert(SPLIT_X == 16 && SPLIT_Y == 8, "lane layout: 16 columns x 4 rows per wave, two waves per group");

template <typename Real>
struct SplitLds {
  Real f[26][SPN];               // (the 26th takes the load of threads with one plane fewer)
  double cm[2][SPN];             // carried n and Delta p
  double F[2][SPLIT_NODES];
  union {
    Real eq[eq_slots<Real>()][SPLIT_NODES];
    struct {                     // at a wall, before the equilibrium
      double rec[2][10][SPW];    // wall-face values
      WallEmission<Real> em[2];
    };
  };
};

// tile row r (halo included) of population k in LDS
__device__ __forceinline__ int lds_row(int k, int r) { return k < 10 ? SPH - 1 - r : r; }

// place of own face `row` (1..8) of a column in a plane's dead halo rows:
// rows 0..2 (66 places) hold faces 1..4, rows 11..13 faces 5..8
__device__ __forceinline__ int dead_place(int row, int col) {
  const int i = (row - 1) * SPLIT_X + col;
  return i + (row > 4 ? 11 * SPW - 4 * SPLIT_X : 0);
}
// place of the tile's right face in row `row`: the right halo
__device__ __forceinline__ int dead_right(int row) { return (row + 3) * SPW + 19; }

// the tile's extra face number e (0..479; the faces after the last row and
// column): the place of the first of its six values in upwind order, the step
// between them and the place it goes to
struct ExtraFace {
  int pos, st, place;
};
__device__ __forceinline__ ExtraFace extra_face(int e) {
  const bool top = e < 20 * SPLIT_X;
  const int f = top ? e : e - 20 * SPLIT_X;
  const int j = top ? f / SPLIT_X : f / SPLIT_Y, i = top ? f % SPLIT_X : f % SPLIT_Y;
  const int j4 = j / 4, j5 = j / 5;
  const int q = top ? j5 : j - 4 * j4;   // which of the four moving rows / columns
  const int mv = q + (q > 1 ? 1 : 0);
  const int k = top ? 5 * mv + (j - 5 * j5) : 5 * j4 + mv;
  const int pt = SPLIT_Y * SPW + 3 + i, px = (i + 3) * SPW + SPLIT_X + (q < 2 ? 5 : 0);
  const int dt = dead_place(SPLIT_Y, i), dx = dead_right(i);
  return ExtraFace{k * SPN + (top ? pt : px), top ? SPW : (q < 2 ? -1 : 1), k * SPN + (top ? dt : dx)};
}
constexpr int EXTRAS = 20 * (SPLIT_X + SPLIT_Y), EXTRA_PASSES = (EXTRAS + SPLIT_NODES - 1) / SPLIT_NODES;

// Velocity row `ky` (uniform) of a tile.
template <typename Real, bool FN>
__device__ __forceinline__ void split_rows(const StageArgs& a, SplitLds<Real>& sm, int ky, const Real* fn, int lane,
                                           int ownb, uint32_t pbytes, uint32_t rbytes) {
  const int col = lane % SPLIT_X, trow = lane / SPLIT_X;
  const int row = ky < 2 ? SPLIT_Y - 1 - trow : trow;   // in LDS
  const int ctr = (row + 3) * SPW + col + 3;
  Real* const own = &sm.f[5 * ky][ctr];
  // faces of the own populations
  Real rxl[5], ryl[5];
#pragma unroll
  for (int kx = 0; kx < 5; ++kx) {
    const Real* const P = own + kx * SPN;
    rxl[kx] = 0;
    if (kx != 2) {
      const Real c[6] = {P[-3], P[-2], P[-1], P[0], P[1], P[2]};
      rxl[kx] = face_value<Real>(a, c, kx > 2);
    }
    if (kx & 1) keep_order(rxl[kx - 1], rxl[kx]);
  }
  keep_order(rxl[4]);
  if (ky == 2) {
    // (lanes past the last extra face repeat it: the same value, stored twice)
    Real rex[EXTRA_PASSES];
    int place[EXTRA_PASSES];
#pragma unroll
    for (int p = 0; p < EXTRA_PASSES; ++p) {
      const ExtraFace e = extra_face(min(lane + p * SPLIT_NODES, EXTRAS - 1));
      const Real* P = sm.f[0] + e.pos;
      rex[p] = face_value(a, P[0], P[e.st], P[2 * e.st], P[3 * e.st], P[4 * e.st]);
      place[p] = e.place;
      keep_order(rex[p], place[p]);
    }
    __syncthreads();
    // hand the faces over through the dead halo
#pragma unroll
    for (int p = 0; p < EXTRA_PASSES; ++p) sm.f[0][place[p]] = rex[p];
  } else {
#pragma unroll
    for (int kx = 0; kx < 5; ++kx) {
      const Real* const P = own + kx * SPN;
      ryl[kx] = face_value(a, P[-3 * SPW], P[-2 * SPW], P[-SPW], P[0], P[SPW]);
      if (kx & 1) keep_order(ryl[kx - 1], ryl[kx]);
    }
    keep_order(ryl[4]);
    __syncthreads();
    if (row > 0) {
      Real* const at = &sm.f[5 * ky][dead_place(row, col)];
#pragma unroll
      for (int kx = 0; kx < 5; ++kx) at[kx * SPN] = ryl[kx];
    }
  }
  __syncthreads();
  Real acc[5], adv[5];
#pragma unroll
  for (int kx = 0; kx < 5; ++kx) {
    acc[kx] = FN ? (Real)a.A * fn[kx] : (Real)0;
    adv[kx] = 0;
    if (kx != 2) {
      // (the shift reads a lane's value only while that lane is active: every
      // lane takes part, then column 15 takes the tile's right face)
      const Real next = lane_next(rxl[kx]), edge = sm.f[5 * ky + kx][dead_right(row)];
      const Real rxr = col == SPLIT_X - 1 ? edge : next;
      adv[kx] = (Real)Rk[kx] * (rxr - rxl[kx]);
    }
  }
  if (ky != 2) {
    const Real* const up = &sm.f[5 * ky][dead_place(row + 1, col)];
    const Real speed = (Real)row_tables.speed[ky];
#pragma unroll
    for (int kx = 0; kx < 5; ++kx) adv[kx] = fmadd(speed, up[kx * SPN] - ryl[kx], adv[kx]);
  }
  const int c0 = (SPLIT_Y + 2 - trow) * SPW + col + 3, c1 = (trow + 3) * SPW + col + 3;
  row_terms<Real>(a, ky, sm.F[0][lane], sm.F[1][lane], acc, adv,
                  [&](int sy, int kx) { return sm.f[5 * sy + kx][sy < 2 ? c0 : c1]; });
#pragma unroll
  for (int kx = 0; kx < 5; ++kx) {
    acc[kx] = with_equilibrium<Real>(a, acc[kx], kx, ky, [&](int j) { return sm.eq[j][lane]; });
    bstore<Real>(acc[kx], plane_rsrc(a.fdst, 5 * ky + kx, pbytes, rbytes), ownb);
  }
  __syncthreads();   // every read of the own values is done
#pragma unroll
  for (int kx = 0; kx < 5; ++kx) own[kx * SPN] = acc[kx];
  __syncthreads();
}

// The sixth group: force, moments and equilibrium, then the carry.  Meets the
// same barriers as split_rows.
template <typename Real>
__device__ __forceinline__ void split_moments(const StageArgs& a, SplitLds<Real>& sm, int lane, bool active,
                                              int64_t node, int64_t N) {
  const int col = lane % SPLIT_X, trow = lane / SPLIT_X;
  const int c0 = (SPLIT_Y + 2 - trow) * SPW + col + 3, c1 = (trow + 3) * SPW + col + 3;
  const double* const mn = sm.cm[0] + c1;
  const double* const mp = sm.cm[1] + c1;
  auto own = [&](int k) { return sm.f[k][k < 10 ? c0 : c1]; };
  __builtin_amdgcn_s_setprio(2);   // the other groups wait for this one's longer chain
  put_equilibrium<Real>(a, node_sums(own), [&](int j, Real v) { sm.eq[j][lane] = v; });
  const double inv_nc = 1.0 / mn[0];
  sm.F[0][lane] = node_force(a, inv_nc, [&](int l, int m) { return mp[m * SPW + l]; },
                             [&](int l, int m) { return mn[m * SPW + l]; });
  sm.F[1][lane] = node_force(a, inv_nc, [&](int l, int m) { return mp[l * SPW + m]; },
                             [&](int l, int m) { return mn[l * SPW + m]; });
  __syncthreads();
  __syncthreads();
  __syncthreads();
  __syncthreads();
  if (active) {
    double cn, cdp;
    carry_finish<std::is_same<Real, float>::value>(node_sums(own), a.rho0, a.tref, a.a, a.b, cn, cdp);
    as_global(a.cout)[node] = cn;
    as_global(a.cout)[N + node] = cdp;
    if (!(fabs(cn) < INFINITY)) a.flag[0] = 1;
  }
}

// v mod n for v near [0, n) (a tile's halo): a step or two unless n is tiny
__device__ __forceinline__ int wrap_near(int v, int n) {
  while (v < 0) v += n;
  while (v >= n) v -= n;
  return v;
}

template <typename Real, bool WALLS, bool FN, bool XSPEC>
__global__ void __launch_bounds__(SPLIT_THREADS, 6) split_stage_kernel(const BatchArgs ba) {
  __shared__ SplitLds<Real> sm;
  const int bid = blockIdx.x;
  // contiguous runs of tiles per XCD (see stage_kernel)
  const int q8 = ba.total_tiles >> 3, r8 = ba.total_tiles & 7, xcd = bid & 7;
  const int t = xcd * q8 + (xcd < r8 ? xcd : r8) + (bid >> 3);
  const int inst = __builtin_amdgcn_readfirstlane(find_instance(ba.inst, ba.ninst, t));
  const InstDesc& d = ba.inst[inst];
  const StageArgs a = stage_args(ba, d);
  const int local = t - d.tile_base;
  const int tile_y = local / d.tiles_x, x0 = (local - tile_y * d.tiles_x) * SPLIT_X, y0 = tile_y * SPLIT_Y;
  const int nx = a.g.nx, ny = a.g.ny;
  const int64_t ps = a.g.ps, N = (int64_t)nx * ny;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  constexpr int RB = (int)sizeof(Real);
  const uint32_t pbytes = (uint32_t)ps * RB, rbytes = (uint32_t)((ny + 5) * a.g.rs + nx) * RB;

  // the tile: threads 0..383 load the even planes and n, the others the odd
  // planes and Delta p, each thread one place of every plane
  constexpr int HALF = SPLIT_THREADS / 2;
  static_assert(HALF % 64 == 0 && HALF >= SPN, "a half's waves cover a plane");
  const int half = wave >= HALF / 64 ? 1 : 0;
  const int place = tid - half * HALF;
  const int pi = min(place, SPN - 1), pr = pi / SPW, pc = pi - pr * SPW;
  int gx, gy = y0 - 3 + pr, my;
  bool flip = false;
  if (XSPEC) {
    const int g = x0 - 3 + pc;
    flip = g < 0 || g >= nx;
    gx = g < 0 ? -1 - g : (g >= nx ? 2 * nx - 1 - g : g);
    gx = min(max(gx, 0), nx - 1);
  } else {
    gx = wrap_near(x0 - 3 + pc, nx);
  }
  if (WALLS) {
    my = gy < 0 ? -1 - gy : (gy >= ny ? 2 * ny - 1 - gy : gy);
    my = min(max(my, 0), ny - 1);
    gy = min(max(gy, 0), ny - 1);   // ghost rows are formed in LDS
  } else {
    gy = my = wrap_near(gy, ny);
  }
  const int soff = (gy + 3) * (int)a.g.rs + gx, moff = my * nx + gx;
  // planes half, half + 2, ...; the 13th of the second half is past the last
  // plane: it loads plane 24 again, into the spare plane
  Real v[13];
#pragma unroll
  for (int j = 0; j < 13; ++j) {
    const int k = 2 * j + half;
    if constexpr (XSPEC) {
      const gmem<const Real>* src = as_global(reinterpret_cast<const Real*>(a.fsrc));
      v[j] = src[(int64_t)min(flip ? 5 * (k / 5) + 4 - k % 5 : k, 24) * ps + soff];
    } else {
      v[j] = bload<Real>(plane_rsrc(a.fsrc, min(k, 24), pbytes, rbytes), soff * RB);
    }
  }
  const double cv = as_global(a.cin)[half * N + moff];

  // the node's own f^n (the group's row)
  const int ky = wave >> 1;   // 5: the sixth group
  const int lane = tid - ky * SPLIT_NODES;
  const int x = x0 + lane % SPLIT_X, y = y0 + lane / SPLIT_X;
  const bool active = x < nx && y < ny;
  const int own = (min(y, ny - 1) + 3) * (int)a.g.rs + min(x, nx - 1);
  Real fn[5];
#pragma unroll
  for (int kx = 0; kx < 5; ++kx)
    fn[kx] = FN ? bload<Real>(plane_rsrc(a.fn, min(5 * ky + kx, 24), pbytes, rbytes), own * RB) : (Real)0;

  const int down = (SPH - 1 - pr) * SPW + pc;   // planes 0..9 are upside down
  if (place < SPN) {
#pragma unroll
    for (int j = 0; j < 13; ++j) sm.f[2 * j + half][j < 5 ? down : place] = v[j];
    sm.cm[half][place] = cv;
  }
  __syncthreads();

  if (WALLS && (y0 == 0 || y0 + SPLIT_Y + 3 > ny)) {   // uniform over the workgroup
    const int top = ny - y0 + 3;   // LDS row of the first ghost row at the high end
    auto side = [&](int s) {
      if (s == 0) return WallSide{0, 3, 4, 5, {2, 1, 0}};
      return WallSide{1, top - 1, top - 2, top - 3,
                      {top, top + 1 < SPH ? top + 1 : -1, top + 2 < SPH ? top + 2 : -1}};
    };
    auto has = [&](int s) { return s == 0 ? y0 == 0 : top < SPH; };
    if (tid >= SPLIT_THREADS - 2) sm.em[tid & 1].set(d, tid & 1);
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      if (has(s) && tid < 25 * SPW) {
        const int k = tid / SPW, c = tid - k * SPW;
        double rec;
        wall_pass1<Real>(d, side(s), k, [&](int kk, int r) -> Real& { return sm.f[kk][lds_row(kk, r) * SPW + c]; }, rec);
        const int j = s ? k / 5 - 3 : k / 5;   // towards the wall, p_y != 0
        if (j == 0 || j == 1) sm.rec[s][5 * j + k % 5][c] = rec;
      }
    }
    __syncthreads();
    if (tid < 4 * SPW) {
      const int s = tid / (2 * SPW), j = (tid / SPW) & 1, c = tid % SPW;
      const int g = x0 - 3 + c;
      // past a specular x plane the column is the mirror of an interior one
      // with kx reversed: the same sums in the same order
      const bool fl = XSPEC && (g < 0 || g >= nx);
      const bool mirror = s == 0 && d.g.walls == 2;
      if (has(s)) {
        const WallSide w = side(s);
        double nw = 0.0;
        if (!mirror) {
          const WallEmission<Real>& em = sm.em[s];
          nw = em.density(d, s, [&](int jj, int kx) { return sm.rec[s][5 * jj + (fl ? 4 - kx : kx)][c]; });
#pragma unroll
          for (int kx = 0; kx < 5; ++kx) {
            const Real val = em.value(d, s, nw, kx, j);
            const int k = 5 * (s ? j : 3 + j) + (fl ? 4 - kx : kx);
#pragma unroll
            for (int q = 0; q < 3; ++q)
              if (w.g[q] >= 0) sm.f[k][lds_row(k, w.g[q]) * SPW + c] = val;
          }
        }
        const bool owner = s == 0 || (y0 <= ny - 1 && ny - 1 < y0 + SPLIT_Y);
        if (j == 0 && owner && c >= 3 && c < 3 + SPLIT_X && g < nx) d.nw[s * nx + g] = nw;
      }
    }
    __syncthreads();
  }

  const int ownb = active ? own * RB : -1;   // past every array: nothing is stored
  if (ky < 5)
    split_rows<Real, FN>(a, sm, ky, fn, lane, ownb, pbytes, rbytes);
  else
    split_moments<Real>(a, sm, lane, active, (int64_t)y * nx + x, N);
}

// --------------------------------------------------------------------------
// whole steps of lattices that fit one workgroup
// --------------------------------------------------------------------------

// A workgroup per instance runs `nsteps` RK-3 steps with f in LDS throughout
// (f^n in registers): a stage costs no launch and no trip to memory.  Lattices
// of up to 64 NG nodes, periodic or with walls across y, periodic in x (the
// rows of waves and half-channel columns of the one-dimensional tests).  The
// bound is the chain of one stage: sums and carry, force, terms, four barriers
// (six with walls), with the faces beside them; the sums and the force are
// taken by waves of their own where 1024 threads allow it (NG < 3), by row 2's
// otherwise.  At 128 registers (above that a compute unit runs one of the
// smaller workgroups instead of two) the FP64 forms spill a few: NG = 2 20 with
// walls and 2 without, NG = 3 with walls 14, up to 36 bytes a lane and a handful
// of reloads a stage; the walled forms of every NG also keep 19 to 27 scalar
// registers in vector lanes.
// Measured (FP64): 13 half channels of 1 x 160 nodes 44 -> 6.5 us a stage, of
// which the faces are a third, the terms a fifth and the wall ghosts a sixth;
// 315 waves of 20 .. 60 nodes 33 -> 3.8 us.
// Directions one node wide have no advection and no force (every difference
// along them is exactly zero, or not a number where Delta p is not finite, which
// the other direction then shows) and are skipped.
// Node i = y nx + x is at LDS place i, after three ghost rows with walls.
template <int NG>
struct Resident {
  static constexpr int NODES = 64 * NG;
  static constexpr int PLACES = resident_places(NG);   // stride of a plane, ghost rows included
  static constexpr int GROUPS = NG < 3 ? 7 : 5;
  static constexpr int THREADS = NODES * GROUPS;
  static constexpr int COLS = PLACES / 9;              // widest walled lattice: (3 + 6) rows
};

template <typename Real, int NG>
struct ResidentLds {
  using R = Resident<NG>;
  Real f[25][R::PLACES];
  Real xf[20][R::PLACES], yf[20][R::PLACES];   // left and lower faces, by moving row / column
  double cm[2][R::NODES];
  double F[2][R::NODES];
  Real eq[eq_slots<Real>()][R::NODES];
  double rec[2][10][R::COLS];
  WallEmission<Real> em[2];
  int cc[7][R::NODES], cr[7][R::NODES];        // neighbours in the carried fields
};

template <typename Real, int NG, bool WALLS>
__global__ void __launch_bounds__(Resident<NG>::THREADS, 4) resident_kernel(const BatchArgs ba, int nsteps) {
  using R = Resident<NG>;
  constexpr bool F32 = std::is_same<Real, float>::value;
  constexpr int GH = WALLS ? 3 : 0;
  __shared__ ResidentLds<Real, NG> sm;
  const InstDesc& d = ba.inst[blockIdx.x];
  BatchArgs b0 = ba;
  b0.stage = 0;
  StageArgs a = stage_args(b0, d);
  const int nx = a.g.nx, ny = a.g.ny, P = nx * ny;
  const int tid = threadIdx.x, group = __builtin_amdgcn_readfirstlane(tid / R::NODES), i = tid - group * R::NODES;
  const bool active = i < P, rows = group < 5, moments = group == (R::GROUPS == 7 ? 5 : 2),
             forces = group == (R::GROUPS == 7 ? 6 : 2);
  const int ky = rows ? group : 0, mv = ky - (ky > 2 ? 1 : 0);   // moving row
  const bool do_x = nx > 1, do_y = WALLS || ny > 1;
  const int n = active ? i : 0, y = n / nx, x = n - y * nx;
  const int own = n + GH * nx;
  // places of the six values around the left face and of the five, in upwind
  // order, of the lower face; the faces on the other side
  int xo[6], yo[5];
#pragma unroll
  for (int j = 0; j < 6; ++j) xo[j] = own - x + wrap_near(x - 3 + j, nx);
#pragma unroll
  for (int j = 0; j < 5; ++j) {
    const int r = ky > 2 ? j - 3 : 2 - j;
    yo[j] = WALLS ? own + r * nx : wrap_near(y + r, ny) * nx + x;
  }
  const int xr = n - x + (x + 1 < nx ? x + 1 : 0), yu = WALLS ? n + nx : (y + 1 < ny ? n + nx : x);
  // neighbours in the carried fields (columns -3 .. 3, rows -3 .. 3)
  if (forces) {
#pragma unroll
    for (int j = 0; j < 7; ++j) {
      sm.cc[j][i] = wrap_near(x + j - 3, nx);
      const int r = y + j - 3;
      sm.cr[j][i] = nx * (WALLS ? min(max(r < 0 ? -1 - r : r >= ny ? 2 * ny - 1 - r : r, 0), ny - 1) : wrap_near(r, ny));
    }
  }
  const gmem<Real>* const f0 = as_global(reinterpret_cast<Real*>(d.f[0]));
  const int64_t at = (int64_t)(y + 3) * a.g.rs + x;
  Real out[5] = {};
  if (rows) {
#pragma unroll
    for (int kx = 0; kx < 5; ++kx) out[kx] = f0[(5 * ky + kx) * a.g.ps + at];
  }
  MomSum fs;
  double cn = 0.0, cdp = 0.0;
  if (moments) {
    cn = as_global(d.carry[ba.cur])[n];
    cdp = as_global(d.carry[ba.cur])[P + n];
  }
  bool bad = false;
  auto publish = [&]() {
    if (rows && active) {
#pragma unroll
      for (int kx = 0; kx < 5; ++kx) sm.f[5 * ky + kx][own] = out[kx];
    }
    __syncthreads();
  };
  if (WALLS && tid < 2) sm.em[tid].set(d, tid);
  publish();
  if (moments) fs = node_sums([&](int k) { return sm.f[k][own]; });

#pragma unroll 1
  for (int step = 0; step < nsteps; ++step) {
    Real fn[5];
#pragma unroll
    for (int kx = 0; kx < 5; ++kx) fn[kx] = out[kx];
#pragma unroll 1
    for (int s = 0; s < 3; ++s) {
      a.A = s == 0 ? RK_A[0] : s == 1 ? RK_A[1] : RK_A[2];
      a.B = s == 0 ? RK_B[0] : s == 1 ? RK_B[1] : RK_B[2];
      auto mine = [&](int k) { return sm.f[k][own]; };
      if (WALLS) {
        // ghost rows: a lane per (population, side, column)
        for (int e = tid; e < 50 * nx; e += R::THREADS) {
          const int k = e / (2 * nx), sc = e - 2 * nx * k, side = sc >= nx ? 1 : 0, c = sc - side * nx;
          const int first = side ? ny + 2 : 3, in = side ? -1 : 1;   // LDS row of the wall's lattice row
          const WallSide w{side, first, first + in, first + 2 * in, {first - in, first - 2 * in, first - 3 * in}};
          double rec;
          wall_pass1<Real>(d, w, k, [&](int kk, int r) -> Real& { return sm.f[kk][r * nx + c]; }, rec);
          const int j = side ? k / 5 - 3 : k / 5;
          if (j == 0 || j == 1) sm.rec[side][5 * j + k % 5][c] = rec;
        }
        __syncthreads();
        // a lane per (emitted population, side, column)
        for (int e = tid; e < 20 * nx; e += R::THREADS) {
          const int q = e / nx, c = e - q * nx, hi = q >= 10 ? 1 : 0, j = (q - 10 * hi) / 5, kx = q - 10 * hi - 5 * j;
          double nw = 0.0;
          if (hi || d.g.walls != 2) {
            const WallEmission<Real>& em = sm.em[hi];
            nw = em.density(d, hi, [&](int jj, int kk) { return sm.rec[hi][5 * jj + kk][c]; });
            const Real v = em.value(d, hi, nw, kx, j);
#pragma unroll
            for (int r = 0; r < 3; ++r) sm.f[5 * (hi ? j : 3 + j) + kx][(hi ? ny + 3 + r : r) * nx + c] = v;
          }
          if (q - 10 * hi == 0) d.nw[hi * nx + c] = nw;
        }
        __syncthreads();
      }
      // faces; meanwhile the sums of the source (those of the last stage's
      // result) and its carry
      Real rxl[5] = {}, ryl[5] = {};
      auto faces = [&](int from, int to) {
#pragma unroll
        for (int kx = 0; kx < 5; ++kx) {
          if (kx < from || kx >= to) continue;
          const Real* const q = sm.f[5 * ky + kx];
          if (do_x && kx != 2) {
            const Real c[6] = {q[xo[0]], q[xo[1]], q[xo[2]], q[xo[3]], q[xo[4]], q[xo[5]]};
            rxl[kx] = face_value<Real>(a, c, kx > 2);
            sm.xf[4 * ky + kx - (kx > 2 ? 1 : 0)][n] = rxl[kx];
          }
          if (do_y && ky != 2) {
            ryl[kx] = face_value(a, q[yo[0]], q[yo[1]], q[yo[2]], q[yo[3]], q[yo[4]]);
            sm.yf[5 * mv + kx][n] = ryl[kx];
          }
          keep_order(rxl[kx], ryl[kx]);
        }
      };
      if (moments && active) {
        sm.cm[0][i] = cn;
        sm.cm[1][i] = cdp;
      }
      if (rows && active) faces(0, 3);
      __syncthreads();
      if (moments && active) put_equilibrium<Real>(a, fs, [&](int j, Real v) { sm.eq[j][i] = v; });
      if (forces && active) {
        const double inv_nc = 1.0 / sm.cm[0][i];
        int cc[7], cr[7];
#pragma unroll
        for (int j = 0; j < 7; ++j) {
          cc[j] = sm.cc[j][i];
          cr[j] = sm.cr[j][i];
        }
        auto pp = [&](int l, int m) { return sm.cm[1][cr[m + 3] + cc[l + 3]]; };
        auto nn = [&](int l, int m) { return sm.cm[0][cr[m + 3] + cc[l + 3]]; };
        if (do_x) sm.F[0][i] = node_force(a, inv_nc, pp, nn);
        if (do_y)
          sm.F[1][i] = node_force(a, inv_nc, [&](int l, int m) { return pp(m, l); },
                                  [&](int l, int m) { return nn(m, l); });
      }
      if (rows && active) faces(3, 5);
      if (WALLS && rows && ky != 2 && i < 5 * nx) {
        // the faces above the last row: lane (kx, x)
        const int kx = i / nx, c = i - kx * nx;
        const Real* const q = sm.f[5 * ky + kx] + (ky > 2 ? ny : ny + 5) * nx + c;
        const int st = ky > 2 ? nx : -nx;
        sm.yf[5 * mv + kx][P + c] = face_value(a, q[0], q[st], q[2 * st], q[3 * st], q[4 * st]);
      }
      __syncthreads();
      if (rows && active) {
        Real acc[5], adv[5];
        const Real p = (Real)row_tables.p[ky];
#pragma unroll
        for (int kx = 0; kx < 5; ++kx) {
          acc[kx] = (Real)a.A * fn[kx];
          adv[kx] = 0;
          if (do_x && kx != 2)
            adv[kx] = (Real)Rk[kx] * (sm.xf[4 * ky + kx - (kx > 2 ? 1 : 0)][xr] - rxl[kx]);
          if (do_y && ky != 2) adv[kx] = fmadd(p, sm.yf[5 * mv + kx][yu] - ryl[kx], adv[kx]);
        }
        row_terms<Real>(a, ky, do_x ? sm.F[0][i] : 0.0, do_y ? sm.F[1][i] : 0.0, acc, adv,
                        [&](int sy, int kx) { return sm.f[5 * sy + kx][own]; });
#pragma unroll
        for (int kx = 0; kx < 5; ++kx)
          out[kx] = with_equilibrium<Real>(a, acc[kx], kx, ky, [&](int j) { return sm.eq[j][i]; });
      }
      __syncthreads();   // every read of the source is done
      publish();
      if (moments && active) {
        fs = node_sums(mine);
        carry_finish<F32>(fs, a.rho0, a.tref, a.a, a.b, cn, cdp);
        if (!(fabs(cn) < INFINITY)) bad = true;
      }
    }
  }
  if (rows && active) {
    gmem<Real>* const fd = as_global(reinterpret_cast<Real*>(d.f[0]));
#pragma unroll
    for (int kx = 0; kx < 5; ++kx) fd[(5 * ky + kx) * a.g.ps + at] = out[kx];
  }
  if (moments && active) {
    gmem<double>* const co = as_global(d.carry[ba.cur ^ (nsteps & 1)]);
    co[n] = cn;
    co[P + n] = cdp;
    if (bad) ba.flag[0] = 1;
  }
}

}  // namespace olbk
