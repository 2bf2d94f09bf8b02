// Sequences of Crank-Nicolson steps on independent windows of a system (gfx950, FP64 complex).
//
// The inverse of T = 1 + i tau H (real potential) decays away from its diagonal whatever the
// potential is.  With kappa the magnitude of T's off-diagonals, conjugating T by exp(eta j)
// changes its Hermitian part by at most theta = 2 kappa sinh(eta), so for theta < 1
//     |(T^-1)_ij| <= exp(-eta |i-j|) / (1 - theta),
// and one step, the Cayley transform (1 - i tau H) T^-1, has conjugated norm at most
// r = (1 + theta) / (1 - theta).  Cutting the line's couplings at a distance D from a row
// therefore changes that row after s steps by at most  r^s exp(-eta D) / (2 sinh eta)  times
// the norm of the state (the largest group velocity of the lattice plus the decay of T^-1).
// The host takes the smallest halo D for which that is below 2^-70 of the state, i.e. nothing
// in FP64; a few hundred rows serve a hundred steps.
//
// k_window: one workgroup owns a window of T = 64 W M rows of one system, cut off from the rest,
// and runs s steps on it with the rows in registers; of the result it stores the rows that lie
// at least the halo away from the window's cut ends (those of the neighbouring windows overlap
// them).  No window waits for another and a step touches no memory: s steps cost one read of
// the state and the potential and one write.
//
// A step is T psi' = (1 - i tau H) psi with the coefficients and the right-hand side of the other
// forms in their order of operations (cn_rows), so its rounding errors are theirs.  Forms with fewer
// operations were less exact: T y = psi and psi' = 2 y - psi saves 4 of 26 per row (200 steps of
// 65536 rows: 260 us), but leaves 2.4e-14 instead of 4.9e-15 after 175 steps of 5806 rows at
// kappa = 0.33; rows divided by kappa (off-diagonals 1) and psi' = psi - 2 w, T w = i tau H psi, saves
// 2, but its rounded quotients leave up to 1.35 times the error after those 200 steps, and rough states
// twice the error from kappa = 1 on.
// Inside the window the solve is the nested partition (Sec. 4): every lane reduces its M rows in
// the RD form (reduce_block_rd), and LV binary levels join 2^LV lane blocks.  Blocks of M * 2^LV
// rows couple their two joint lines by less than 2^-66 of the diagonal (the host takes LV from
// the same bound), so the reduced system on their joint lines is diagonal: each joint line needs
// its own two slots only, and the levels above it are not run.
#pragma once
#include "nshaped_kernels.hpp"

namespace nsd {

constexpr int kWinSteps = 128;  // most steps of one launch (their fields travel in the arguments)

struct WinArgs {
  const cd* in[2];  // state (and, NR = 2, the gradient) before the launch's steps
  cd* out[2];       // and after them; out[1] of a forward step and out[i] = null are not stored
  int64_t ibs[2], obs[2];  // elements between systems of in and out
  const double* V;
  const double* xg;
  int64_t vbs;  // elements between systems of V and xg (0: one potential for every system)
  int64_t n;    // rows per system
  int64_t nwin;  // windows per system
  int64_t vr, halo;  // window t starts at row t * vr; its results hold `halo` rows from a cut end
  double vscale, tau, kap, idx2;
  int nst;
  // NR = 2: dV_j += acc Im(conj(lambda_j) mu_j) summed over the steps (lambda and mu twice the means
  // of a step's two gradients and states), and per step k and
  // wavefront the sum of xg_j times the same term (acc without vscale) in part[k * nparts + ...]
  double* dV;
  double acc_dV, acc_dE;  // factors: of the term in dV, of x_j times the term in dE
  double* part;
  int64_t nparts;
  int* status;
  // per system: bit r set when a window met a non-finite value of in/out[r].  One such value
  // makes the whole line non-finite in exact steps: with `later` (not the first launch of a
  // sequence) the windows of a marked system take their input as NaN
  int* bad;
  int later;
  double E[kWinSteps];
};

// arguments of the kernel that ends a sequence (k_window_end)
struct WinEnd {
  int* bad;
  int64_t n;
  cd* x[2];
  int64_t bs[2];
  double* dV;
  int64_t vbs;
  // checkpoints after the first one (which holds the input): elements between them and between
  // their systems
  cd* ckpt;
  int64_t nck, cspan, cbs;
};

// The rows are multiplied by i, which makes the off-diagonals real: with v the imaginary part of T's
// diagonal, row j reads
//     kappa y_{j-1} + (i - v_j) y_j + kappa y_{j+1} = (i + v_j) psi_j - kappa (psi_{j-1} + psi_{j+1}).
// The first row of a block has its right-hand side split like its diagonal: -kappa psi_{j-1} is in
// the D slot of the block before.  T is symmetric, so a reduced block has one coupling C instead of
// two (UC = DB), and the products of Table 1's multipliers that JU needs are the beta of the RD rows
// with the other sign: with g_i the reciprocal pivots and h_i = kappa g_i, beta_1 = h_1,
// beta_i = -beta_{i-1} h_i, gamma_i = h_i and the forward sum of reduce_block_rd is
//     y_{J+1} = D_1 - sum_{k >= 2} beta_{k-1} D_k - (beta_1 - sum_{k >= 2} beta_{k-1} beta_k) y_J
//     + ...
struct WBlk {
  cd UA, C, DA;
};
template <int NR>
struct WRhs {
  cd UD[NR], DD[NR];
};
// The imaginary part of T's diagonal, in cn_rows' order: its rounding is that of the other forms.
__device__ __forceinline__ double wdiag(double tau, double idx2, double v) {
#pragma clang fp contract(off)
  return tau * (idx2 + v);
}
// The right-hand side of a row with the sum s of its neighbours, in cn_rows' order.
__device__ __forceinline__ cd wrhs(double v, double kap, cd z, cd s) {
  return mk(fma(v, z.x, fma(-kap, s.x, -z.y)), fma(v, z.y, fma(-kap, s.y, z.x)));
}
// An eliminated joint line: the reciprocal of its pivot, its couplings to the left and right
// neighbours and the scaled row (B, C) that the way down applies.
struct WNode {
  cd ia, rU, rD, B, C;
};

__device__ __forceinline__ void wmerge(WBlk& b, const WBlk& o, WNode& t) {
  t.ia = crecip(cadd(b.DA, o.UA));
  t.rU = b.C;
  t.rD = o.C;
  t.B = cmul(t.rU, t.ia);
  t.C = cmul(t.rD, t.ia);
  b.UA = cfms(t.rU, t.B, b.UA);
  b.DA = cfms(t.rD, t.C, o.DA);
  b.C = cneg(cmul(t.rU, t.C));
}
template <int NR>
__device__ __forceinline__ void wmerge_rhs(WRhs<NR>& b, const WRhs<NR>& o, const cd ia, const cd rU,
                                           const cd rD, cd (&dl)[NR]) {
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    dl[r] = cmul(cadd(b.DD[r], o.UD[r]), ia);
    b.UD[r] = cfms(rU, dl[r], b.UD[r]);
    b.DD[r] = cfms(rD, dl[r], o.DD[r]);
  }
}

// The levels up of the matrix: the node of level m's joint line goes to nodes[lane + m], where
// the same lane reads it back.
template <int m>
__device__ __forceinline__ void wlevel_fac(WBlk& b, WNode* nodes, int lane) {
  WBlk o;
  o.UA = xmove<m>(b.UA);
  o.C = xmove<m>(b.C);
  o.DA = xmove<m>(b.DA);
  WNode t;
  wmerge(b, o, t);
  if ((lane & (2 * m - 1)) == 0) nodes[lane + m] = t;
}
template <int m, int NR>
__device__ __forceinline__ void wlevel_rhs(WRhs<NR>& b, const WNode* nodes, cd (*dl)[NR],
                                           int lane) {
  const WNode& t = nodes[(lane + m) & 63];
  WRhs<NR> o;
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    o.UD[r] = xmove<m>(b.UD[r]);
    o.DD[r] = xmove<m>(b.DD[r]);
  }
  cd d[NR];
  wmerge_rhs<NR>(b, o, t.ia, t.rU, t.rD, d);
  if ((lane & (2 * m - 1)) == 0) {
#pragma unroll
    for (int r = 0; r < NR; ++r) dl[lane + m][r] = d[r];
  }
}
// Matrix and right-hand sides at once (the matrix changes from step to step).
template <int m, int NR>
__device__ __forceinline__ void wlevel_both(WBlk& b, WRhs<NR>& c, WNode* nodes, cd (*dl)[NR],
                                            int lane) {
  WBlk o;
  o.UA = xmove<m>(b.UA);
  o.C = xmove<m>(b.C);
  o.DA = xmove<m>(b.DA);
  WRhs<NR> p;
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    p.UD[r] = xmove<m>(c.UD[r]);
    p.DD[r] = xmove<m>(c.DD[r]);
  }
  WNode t;
  wmerge(b, o, t);
  cd d[NR];
  wmerge_rhs<NR>(c, p, t.ia, t.rU, t.rD, d);
  if ((lane & (2 * m - 1)) == 0) {
    nodes[lane + m].B = t.B;
    nodes[lane + m].C = t.C;
#pragma unroll
    for (int r = 0; r < NR; ++r) dl[lane + m][r] = d[r];
  }
}
template <int m, int NR>
__device__ __forceinline__ void wlevel_down(cd (&pJ)[NR], cd (&pM)[NR], const WNode* nodes,
                                            const cd (*dl)[NR], int lane) {
  const cd B = nodes[(lane + m) & 63].B, C = nodes[(lane + m) & 63].C;
  const int low = lane & (2 * m - 1);
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    const cd pK = cfms(C, pM[r], cfms(B, pJ[r], dl[(lane + m) & 63][r]));
    const cd oK = xmove<m>(pK);
    const cd oM = xmove<m>(pM[r]);
    if (low == m) {
      pJ[r] = oK;
      pM[r] = oM;
    }
    if (low == 0) pM[r] = pK;
  }
}

__device__ __forceinline__ cd lane_get(cd v, int src) {
  cd z;
  z.x = __shfl(v.x, src, 64);
  z.y = __shfl(v.y, src, 64);
  return z;
}

template <int M, int W, int NR, bool XG>
struct WinSmem {
  // per wavefront: the staging buffer of the loads and stores; between them the nodes of the
  // levels, their right-hand sides and (XG) the diagonal's two terms per row
  static constexpr size_t kNode = sizeof(WNode) * 64;
  static constexpr size_t kDl = sizeof(cd) * 64 * NR;
  static constexpr size_t kDiag = XG ? sizeof(double) * 64 * M * 2 : 0;
  static constexpr size_t kStage = sizeof(cd) * Stage<M>::QS;
  static constexpr size_t kUse = kNode + kDl + kDiag;
  static constexpr size_t kBytes = ((kUse > kStage ? kUse : kStage) + 15) / 16 * 16;
  cd buf[W][kBytes / 16];
  // hand-over between the wavefronts, two buffers by step parity: UA, UD of a wavefront's first
  // block and DA, DD of its last one
  cd ua[2][W], da[2][W], ud[2][W][NR], dd[2][W][NR];
};

// IN: no row of the wavefront nor of its neighbours lies past an end of the window.
// XG: the potential has a field term that changes from step to step, so every step reduces the
// matrix anew; without it the matrix is reduced once (pivots, beta and the nodes stay) and a step
// runs the updates of the right-hand side alone (the stored r factors of Sec. 5.2.4).
template <int M, int W, int LV, int NR, bool XG, bool IN>
__device__ __forceinline__ void window_run(const WinArgs& A, WinSmem<M, W, NR, XG>& sm,
                                           int64_t sys, int64_t win, int64_t row0, int nloc) {
  using S = Stage<M>;
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int w0 = wave * 64 * M;
  const int J = w0 + lane * M;
  cd* buf = sm.buf[wave];
  double* bufd = reinterpret_cast<double*>(buf);
  WNode* nodes = reinterpret_cast<WNode*>(buf);
  cd(*dl)[NR] = reinterpret_cast<cd(*)[NR]>(nodes + 64);
  double* keep = reinterpret_cast<double*>(dl + 64);

  // ---- loads (coalesced), transposed to lane blocks through the staging buffer
  const double kap = A.kap;
  cd z[NR][M], zM[NR];  // the state; its row J + M, which the next lane (or wavefront) owns
  double va[M];  // imaginary part of T's diagonal; with a field, V
  auto row = [&](int k) {
    const int r = w0 + 64 * k + lane;
    return IN ? r : (r < nloc ? r : nloc - 1);
  };
  {
    cd raw[M];
    double rv[M], rx[XG ? M : 1], xt[XG ? M : 1];
    const double* gv = A.V + sys * A.vbs + row0;
    const int next = IN || w0 + 64 * M < nloc ? w0 + 64 * M : nloc - 1;
    cd edge[NR];
#pragma unroll
    for (int r = 0; r < NR; ++r)
      edge[r] = sel(true, (A.in[r] + sys * A.ibs[r] + row0)[next], czero());
#pragma unroll
    for (int k = 0; k < M; ++k) raw[k] = sel(true, (A.in[0] + sys * A.ibs[0] + row0)[row(k)], czero());
#pragma unroll
    for (int k = 0; k < M; ++k) rv[k] = sel(true, gv[row(k)], 0.0);
    if constexpr (XG) {
      const double* gx = A.xg + sys * A.vbs + row0;
#pragma unroll
      for (int k = 0; k < M; ++k) rx[k] = sel(true, gx[row(k)], 0.0);
    }
#pragma unroll
    for (int r = 0; r < NR; ++r) {
#pragma unroll
      for (int k = 0; k < M; ++k) buf[S::addr(1 + 64 * k + lane)] = raw[k];
      if (r + 1 < NR) {
        const cd* g = A.in[r + 1 < NR ? r + 1 : r] + sys * A.ibs[r + 1 < NR ? r + 1 : r] + row0;
#pragma unroll
        for (int k = 0; k < M; ++k) raw[k] = sel(true, g[row(k)], czero());
      }
      wave_sync();
#pragma unroll
      for (int j = 0; j < M; ++j) {
        z[r][j] = buf[S::addr(lane * M + j + 1)];
        if constexpr (!IN) z[r][j] = csel(J + j < nloc, z[r][j], czero());
      }
      zM[r] = csel(lane == 63, edge[r], lane_get(z[r][0], (lane + 1) & 63));
      if constexpr (!IN) zM[r] = csel(J + M < nloc, zM[r], czero());
      wave_sync();
    }
#pragma unroll
    for (int k = 0; k < M; ++k) bufd[S::addr(1 + 64 * k + lane)] = rv[k];
    wave_sync();
#pragma unroll
    for (int j = 0; j < M; ++j) {
      const double v = A.vscale * bufd[S::addr(lane * M + j + 1)];
      va[j] = XG ? v : wdiag(A.tau, A.idx2, v);
      if constexpr (!IN) va[j] = J + j < nloc ? va[j] : (XG ? -A.idx2 : 0.0);
    }
    wave_sync();
    if constexpr (XG) {
#pragma unroll
      for (int k = 0; k < M; ++k) bufd[S::addr(1 + 64 * k + lane)] = rx[k];
      wave_sync();
#pragma unroll
      for (int j = 0; j < M; ++j) {
        xt[j] = bufd[S::addr(lane * M + j + 1)];
        if constexpr (!IN) xt[j] = J + j < nloc ? xt[j] : 0.0;
      }
      wave_sync();
#pragma unroll
      for (int j = 0; j < M; ++j) {
        keep[j * 64 + lane] = va[j];
        keep[(M + j) * 64 + lane] = xt[j];
      }
    }
  }
  if (A.later) {
    const int seen = A.bad[sys];
#pragma unroll
    for (int r = 0; r < NR; ++r)
      if ((seen >> r) & 1) {
#pragma unroll
        for (int j = 0; j < M; ++j) z[r][j] = mk(__builtin_nan(""), __builtin_nan(""));
        zM[r] = z[r][0];
      }
  }
  // rows of this window whose result is stored
  const int lo = win == 0 ? 0 : (int)A.halo;
  const int hi = win == A.nwin - 1 ? nloc : (int)(A.vr + A.halo);

  // v where rows J + i - 1 and J + i are both of the window, else zero
  auto cpl = [&](int i, cd v) { return IN ? v : csel(J + i < nloc && J + i > 0, v, czero()); };
  constexpr int SP = 1 << LV;
  cd g[M], beta[M];  // [1 .. M-1]; XG: of the current step
  cd ip = czero(), ipn = czero();  // reciprocal pivots of the joint lines at the block's two ends
  double acc[NR > 1 ? M : 1];
  if constexpr (NR > 1) {
#pragma unroll
    for (int j = 0; j < M; ++j) acc[j] = 0.0;
  }
  auto pot = [&](int j, double E) {
    if constexpr (XG)
      return wdiag(A.tau, A.idx2, fma(keep[(M + j) * 64 + lane], E, keep[j * 64 + lane]));
    return va[j];
  };
  auto diag = [&](int j, double E) { return mk(-pot(j, E), 1.0); };
  // RD of the matrix, JD and JU
  auto reduce_matrix = [&](double E, WBlk& b) {
    g[1] = crecip(diag(1, E));
    cd h = rmul(kap, g[1]);
    beta[1] = cpl(1, h);
    cd fb = beta[1];
#pragma unroll
    for (int i = 2; i < M; ++i) {
      g[i] = crecip(rfms(kap, cpl(i, h), diag(i, E)));
      h = rmul(kap, g[i]);
      beta[i] = cpl(i, cneg(cmul(beta[i - 1], h)));
      fb = cfms(beta[i - 1], beta[i], fb);
    }
    b.UA = rfms(kap, fb, diag(0, E));
    b.C = cpl(M, rmul(-kap, beta[M - 1]));
    b.DA = cpl(M, rmul(-kap, h));
  };
  auto reduce_rhs = [&](double E, cd (&D)[NR][M], WRhs<NR>& c) {
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      auto rhs = [&](int i) {
        const cd hi = i + 1 < M ? z[r][i + 1 < M ? i + 1 : i] : zM[r];
        const cd s = i > 0 ? cadd(cpl(i, z[r][i > 0 ? i - 1 : 0]), hi) : hi;
        return wrhs(pot(i, E), kap, z[r][i], s);
      };
      D[r][1] = cmul(rhs(1), g[1]);
      cd fd = D[r][1];
#pragma unroll
      for (int i = 2; i < M; ++i) {
        D[r][i] = cmul(rfms(kap, cpl(i, D[r][i - 1]), rhs(i)), g[i]);
        fd = cfms(beta[i - 1], D[r][i], fd);
      }
      c.UD[r] = rfms(kap, fd, rhs(0));
      c.DD[r] = cpl(M, rmul(-kap, cadd(z[r][M - 1], D[r][M - 1])));
    }
  };
  WBlk b;
  if constexpr (!XG) {
    reduce_matrix(0.0, b);
    if constexpr (LV > 0) wlevel_fac<1>(b, nodes, lane);
    if constexpr (LV > 1) wlevel_fac<2>(b, nodes, lane);
    if constexpr (LV > 2) wlevel_fac<4>(b, nodes, lane);
    if constexpr (LV > 3) wlevel_fac<8>(b, nodes, lane);
    if constexpr (LV > 4) wlevel_fac<16>(b, nodes, lane);
    if constexpr (LV > 5) wlevel_fac<32>(b, nodes, lane);
  }
  for (int k = 0; k < A.nst; ++k) {
    cd D[NR][M];
    WRhs<NR> c;
    if constexpr (XG) reduce_matrix(A.E[k], b);
    reduce_rhs(XG ? A.E[k] : 0.0, D, c);
    // ---- LV levels; afterwards the lanes with the low LV bits clear hold decoupled blocks
    if constexpr (XG) {
      if constexpr (LV > 0) wlevel_both<1, NR>(b, c, nodes, dl, lane);
      if constexpr (LV > 1) wlevel_both<2, NR>(b, c, nodes, dl, lane);
      if constexpr (LV > 2) wlevel_both<4, NR>(b, c, nodes, dl, lane);
      if constexpr (LV > 3) wlevel_both<8, NR>(b, c, nodes, dl, lane);
      if constexpr (LV > 4) wlevel_both<16, NR>(b, c, nodes, dl, lane);
      if constexpr (LV > 5) wlevel_both<32, NR>(b, c, nodes, dl, lane);
    } else {
      if constexpr (LV > 0) wlevel_rhs<1, NR>(c, nodes, dl, lane);
      if constexpr (LV > 1) wlevel_rhs<2, NR>(c, nodes, dl, lane);
      if constexpr (LV > 2) wlevel_rhs<4, NR>(c, nodes, dl, lane);
      if constexpr (LV > 3) wlevel_rhs<8, NR>(c, nodes, dl, lane);
      if constexpr (LV > 4) wlevel_rhs<16, NR>(c, nodes, dl, lane);
      if constexpr (LV > 5) wlevel_rhs<32, NR>(c, nodes, dl, lane);
    }
    // ---- the joint lines of those blocks: own U slot plus the D slot of the block before
    const int par = k & 1;
    const bool fac = XG || k == 0;  // the joint lines' pivots are formed
    if constexpr (W > 1) {
      if (lane == 0) {
        if (fac) sm.ua[par][wave] = b.UA;
#pragma unroll
        for (int r = 0; r < NR; ++r) sm.ud[par][wave][r] = c.UD[r];
      }
      if (lane == 64 - SP) {
        if (fac) sm.da[par][wave] = b.DA;
#pragma unroll
        for (int r = 0; r < NR; ++r) sm.dd[par][wave][r] = c.DD[r];
      }
    }
    cd qD[NR];
#pragma unroll
    for (int r = 0; r < NR; ++r) qD[r] = czero();
    if constexpr (LV < 6) {
#pragma unroll
      for (int r = 0; r < NR; ++r) qD[r] = lane_get(c.DD[r], (lane - SP) & 63);
    }
    if constexpr (W > 1) __syncthreads();
    if (fac) {
      cd qA = czero(), nA = czero();
      if constexpr (LV < 6) qA = lane_get(b.DA, (lane - SP) & 63);
      if (lane < SP) qA = czero();
      if constexpr (W > 1) {
        if (lane < SP && wave > 0) qA = sm.da[par][wave - 1];
        if (wave + 1 < W) nA = sm.ua[par][wave + 1];
      }
      ip = crecip(cadd(qA, b.UA));
      if constexpr (W > 1) ipn = crecip(cadd(b.DA, nA));
    }
    cd pJ[NR], pM[NR];
    if (lane < SP) {
#pragma unroll
      for (int r = 0; r < NR; ++r) qD[r] = czero();
      if constexpr (W > 1) {
        if (wave > 0) {
#pragma unroll
          for (int r = 0; r < NR; ++r) qD[r] = sm.dd[par][wave - 1][r];
        }
      }
    }
#pragma unroll
    for (int r = 0; r < NR; ++r) pJ[r] = cmul(cadd(qD[r], c.UD[r]), ip);
    if constexpr (LV < 6) {
#pragma unroll
      for (int r = 0; r < NR; ++r) pM[r] = lane_get(pJ[r], (lane + SP) & 63);
    }
    if (lane >= 64 - SP) {
      // the last block's end: the next wavefront's first joint line, or past the window
#pragma unroll
      for (int r = 0; r < NR; ++r) pM[r] = czero();
      if constexpr (W > 1) {
        if (wave + 1 < W) {
#pragma unroll
          for (int r = 0; r < NR; ++r)
            pM[r] = cmul(cadd(c.DD[r], sm.ud[par][wave + 1][r]), ipn);
        }
      }
    }
    // ---- down the levels
    if constexpr (LV > 5) wlevel_down<32, NR>(pJ, pM, nodes, dl, lane);
    if constexpr (LV > 4) wlevel_down<16, NR>(pJ, pM, nodes, dl, lane);
    if constexpr (LV > 3) wlevel_down<8, NR>(pJ, pM, nodes, dl, lane);
    if constexpr (LV > 2) wlevel_down<4, NR>(pJ, pM, nodes, dl, lane);
    if constexpr (LV > 1) wlevel_down<2, NR>(pJ, pM, nodes, dl, lane);
    if constexpr (LV > 0) wlevel_down<1, NR>(pJ, pM, nodes, dl, lane);
    // ---- the rows of the block, upwards
    {
      double part = 0.0;
      cd y[NR];
#pragma unroll
      for (int r = 0; r < NR; ++r) zM[r] = pM[r];
#pragma unroll
      for (int i = M - 1; i >= 0; --i) {
#pragma unroll
        for (int r = 0; r < NR; ++r) {
          const cd w = i < M - 1 ? z[r][i < M - 1 ? i + 1 : i] : pM[r];
          const cd n = i > 0 ? cfms(g[i > 0 ? i : 1], rmul(kap, w),
                                    cfms(beta[i > 0 ? i : 1], pJ[r], D[r][i > 0 ? i : 1]))
                             : pJ[r];
          if constexpr (NR > 1) y[r] = cadd(z[r][i], n);
          z[r][i] = n;
        }
        if constexpr (NR > 1) {
          // twice (psi_k + psi_k+1) / 2 of the state, twice lambda of the gradient
          const double q = y[1].x * y[0].y - y[1].y * y[0].x;
          acc[i] += q;
          if constexpr (XG) {
            const bool own = J + i >= lo && J + i < hi;
            part = own ? fma(keep[(M + i) * 64 + lane], q, part) : part;
          }
        }
      }
      if constexpr (NR > 1 && XG) {
        if (A.part) {
          part = wave_sum(part);
          if (lane == 0)
            A.part[k * A.nparts + (sys * A.nwin + win) * W + wave] = A.acc_dE * part;
        }
      }
    }
  }

  // ---- stores of the rows that hold, coalesced through the staging buffer
  int sl = lane;
  asm volatile("" : "+v"(sl));
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    bool bad = false;
#pragma unroll
    for (int j = 0; j < M; ++j) bad |= J + j >= lo && J + j < hi && !cfinite(z[r][j]);
    if (__any(bad) && lane == 0) {
      atomicOr(A.status, 1);
      atomicOr(A.bad + sys, 1 << r);
    }
    if (A.out[r]) {
      wave_sync();
#pragma unroll
      for (int j = 0; j < M; ++j)
        buf[S::addr(lane * M + j + 1)] = z[r][j];
      wave_sync();
      cd* o = A.out[r] + sys * A.obs[r] + row0;
#pragma unroll
      for (int k = 0; k < M; ++k) {
        const int q = w0 + 64 * k + sl;
        if (q >= lo && q < hi) o[q] = buf[S::addr(1 + 64 * k + sl)];
      }
    }
  }
  if constexpr (NR > 1) {
    if (A.dV) {
      wave_sync();
#pragma unroll
      for (int j = 0; j < M; ++j) bufd[S::addr(lane * M + j + 1)] = acc[j];
      wave_sync();
      double* o = A.dV + sys * A.vbs + row0;
#pragma unroll
      for (int k = 0; k < M; ++k) {
        const int q = w0 + 64 * k + sl;
        if (q >= lo && q < hi) o[q] += A.acc_dV * bufd[S::addr(1 + 64 * k + sl)];
      }
    }
  }
}

// One workgroup per window: blockIdx.x = system * nwin + window.
template <int M, int W, int LV, int NR, bool XG>
__global__ __launch_bounds__(64 * W, NR == 1 && M < 8 ? 3 : 2) void k_window(WinArgs A) {
  __shared__ WinSmem<M, W, NR, XG> sm;
  constexpr int T = 64 * W * M;
  const int64_t sys = blockIdx.x / A.nwin, win = blockIdx.x - sys * A.nwin;
  const int64_t row0 = win * A.vr;
  const int nloc = (int)(A.n - row0 < T ? A.n - row0 : T);
  const int w0 = (threadIdx.x >> 6) * 64 * M;
  if (w0 >= 1 && nloc >= w0 + 64 * M + 1)
    window_run<M, W, LV, NR, XG, true>(A, sm, sys, win, row0, nloc);
  else
    window_run<M, W, LV, NR, XG, false>(A, sm, sys, win, row0, nloc);
}

}  // namespace nsd
