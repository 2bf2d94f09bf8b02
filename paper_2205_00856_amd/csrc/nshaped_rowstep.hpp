// A Crank-Nicolson step of a batch of contiguous systems in one pass (gfx950, FP64 complex).
//
// A workgroup takes a tile of T = 64 W M rows of one system: a whole system, or one of its tiles.
// Its rows and its solve are those of k_window: every lane reduces its M rows, lv binary levels join
// 2^lv lanes, after which the joint lines are decoupled in every real potential (the host takes lv
// from the bound), and each joint takes its own two slots, those across wavefronts through LDS.
// Against k_tile (levels over the whole workgroup, the upper six in one wavefront between two
// barriers) a tile has lv levels, one barrier, one edge row, and 104 registers or fewer.  The forms
// T y = psi, psi' = 2 y - psi or y - i tau H y need no edge row, but their rounding errors are larger:
// 1.7 times after 60 steps at kappa = 0.33, and 1.1 times in the second form.
//
// Tiles of a longer system exchange the slots of their first and last block through lines in
// memory, as in k_tile<PH_LINK>: word by word, all-ones words marking what has not arrived, two
// buffers in turn.  k_rowstep_fix runs the tiles whose wait reached its bound, from the lines, and
// makes systems with a non-finite row all NaN.  In place: a tile stores only when both neighbours
// have published, so after the one before has loaded its edge row here; a tile that is left keeps
// the edge row that it has loaded.
//
// Bound by memory (40 bytes a row): 4096 systems of 4096 rows 138 -> 132 us (5.1 TB/s), 1000 of
// 1531 rows 23.5 -> 17.8, 10^4 of 300 rows 49.6 -> 31 us; systems of several tiles, before in two
// passes: 64 of 65536 rows 65 -> 33 us, 2^24 rows 222 -> 131 us.
#pragma once
#include "nshaped_windows.hpp"

namespace nsd {

struct RowStepArgs {
  const cd* in;
  cd* out;
  const double* V;
  const double* xg;
  int64_t n, bs, vbs;  // rows; elements between systems of the state and of V, xg
  int64_t ntiles;      // tiles of a system
  int lv;
  double vscale, E, tau, kap, idx2;
  // partial waves: system s carries l = l0 + s, whose V gains l (l + 1) / (2 r^2), r = (row + 1) dr
  int64_t l0;
  double dr;  // 0: none
  double* lk;  // lines: [2][lk_n][8]
  int64_t lk_n;
  int *st, *done, *bad;  // as in k_colstep
  cd* edge;              // of a tile left to the fix: psi of the row after its last one
  int* status;
  int spin;  // polls of a line before its tile is left
};

struct RowNode {
  cd B, C, dl;
};
template <int m>
__device__ __forceinline__ void rlevel_up(WBlk& b, WRhs<1>& c, RowNode* nodes, int lane) {
  WBlk o;
  o.UA = xmove<m>(b.UA);
  o.C = xmove<m>(b.C);
  o.DA = xmove<m>(b.DA);
  WRhs<1> p;
  p.UD[0] = xmove<m>(c.UD[0]);
  p.DD[0] = xmove<m>(c.DD[0]);
  WNode t;
  wmerge(b, o, t);
  cd dl[1];
  wmerge_rhs<1>(c, p, t.ia, t.rU, t.rD, dl);
  if ((lane & (2 * m - 1)) == 0) {
    nodes[lane + m].B = t.B;
    nodes[lane + m].C = t.C;
    nodes[lane + m].dl = dl[0];
  }
}
template <int m>
__device__ __forceinline__ void rlevel_down(cd& pJ, cd& pM, const RowNode* nodes, int lane) {
  const RowNode t = nodes[(lane + m) & 63];
  const cd pK = cfms(t.C, pM, cfms(t.B, pJ, t.dl));
  const cd oK = xmove<m>(pK);
  const cd oM = xmove<m>(pM);
  const int low = lane & (2 * m - 1);
  if (low == m) {
    pJ = oK;
    pM = oM;
  }
  if (low == 0) pM = pK;
}

template <int M, int W>
struct RowStepSmem {
  static constexpr size_t kStage = sizeof(cd) * Stage<M>::QS;
  static constexpr size_t kUse = sizeof(RowNode) * 64;
  static constexpr size_t kBytes = ((kUse > kStage ? kUse : kStage) + 15) / 16 * 16;
  cd buf[W][kBytes / 16];
  cd ua[W], da[W], ud[W], dd[W];  // a wavefront's first block's U slot, its last one's D slot
  int bad[W], ok[2];
  cd edge;  // psi of the row after the tile
};

// Four doubles of a line (two complex values) to or from memory, by lanes 0 .. 3 of a wavefront.
__device__ __forceinline__ void line_put(double* line, cd a, cd d, int src, int lane) {
  const double v[4] = {a.x, a.y, d.x, d.y};
  double mine = 0.0;
#pragma unroll
  for (int f = 0; f < 4; ++f) {
    const double w = __shfl(v[f], src, 64);
    mine = lane == f ? w : mine;
  }
  if (lane < 4) __hip_atomic_store(line + lane, mine, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// False when the line did not arrive within the bound of the wait.
template <bool FIX>
__device__ __forceinline__ bool line_get(const double* line, cd& a, cd& d, int lane, int spin) {
  const long long* src = reinterpret_cast<const long long*>(line) + (lane & 3);
  long long v = -1ll;
  for (int it = 0; it < (FIX ? 1 : spin); ++it) {
    v = __hip_atomic_load(src, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (FIX || __all(v != -1ll)) break;
    __builtin_amdgcn_s_sleep(1);
  }
  const double q = __longlong_as_double(v);
  a = mk(__shfl(q, 0, 64), __shfl(q, 1, 64));
  d = mk(__shfl(q, 2, 64), __shfl(q, 3, 64));
  return __all(v != -1ll);
}

template <int M, int W, bool XG, bool FIX, bool IN>
__device__ __forceinline__ void rowstep_run(const RowStepArgs& A, RowStepSmem<M, W>& sm,
                                            int64_t gt, int64_t sys, int64_t tile, int e) {
  using S = Stage<M>;
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int64_t row0 = tile * (64 * W * M);  // the tile's first row
  const int nloc = (int)(A.n - row0 < 64 * W * M + 1 ? A.n - row0 : 64 * W * M + 1);
  const int w0 = wave * 64 * M;
  const int J = w0 + lane * M;
  cd* buf = sm.buf[wave];
  double* bufd = reinterpret_cast<double*>(buf);
  RowNode* nodes = reinterpret_cast<RowNode*>(buf);
  const double kap = A.kap;
  const cd zero = czero();
  const bool multi = A.ntiles > 1;

  // ---- loads (coalesced), transposed to lane blocks
  cd D[M], zM;  // psi; its row J + M
  double va[M];
  {
    cd raw[M];
    double rv[M], rx[XG ? M : 1];
    auto row = [&](int k) {
      const int r = w0 + 64 * k + lane;
      return IN ? r : (r < nloc ? r : nloc - 1);
    };
    const cd* gp = A.in + sys * A.bs + row0;
    const double* gv = A.V + sys * A.vbs + row0;
    cd edge = sel(true, gp[IN || w0 + 64 * M < nloc ? w0 + 64 * M : nloc - 1], zero);
#pragma unroll
    for (int k = 0; k < M; ++k) raw[k] = sel(true, gp[row(k)], zero);
#pragma unroll
    for (int k = 0; k < M; ++k) rv[k] = sel(true, gv[row(k)], 0.0);
    if constexpr (XG) {
      const double* gx = A.xg + sys * A.vbs + row0;
#pragma unroll
      for (int k = 0; k < M; ++k) rx[k] = sel(true, gx[row(k)], 0.0);
    }
#pragma unroll
    for (int k = 0; k < M; ++k) buf[S::addr(1 + 64 * k + lane)] = raw[k];
    if (multi && wave == W - 1 && tile + 1 < A.ntiles) {
      // (in place, the next tile may have stored by the time of the fix)
      if constexpr (FIX) edge = A.edge[gt];
      else if (lane == 0) sm.edge = edge;
    }
    if (lane == 0) buf[S::addr(S::QN - 1)] = edge;
    wave_sync();
#pragma unroll
    for (int j = 0; j < M; ++j) {
      D[j] = buf[S::addr(lane * M + j + 1)];
      if constexpr (!IN) D[j] = csel(J + j < nloc, D[j], zero);
    }
    zM = buf[S::addr(lane * M + M + 1)];
    if constexpr (!IN) zM = csel(J + M < nloc, zM, zero);
    wave_sync();
    // the diagonal in the loads' order, where a potential of its own costs no second transposition
#pragma unroll
    for (int k = 0; k < M; ++k) {
      double v = A.vscale * rv[k];
      if constexpr (XG) v = fma(rx[k], A.E, v);
      if (A.dr > 0.0) {
        const double r = (double)(row0 + w0 + 64 * k + lane + 1) * A.dr;
        const double l = (double)(A.l0 + sys);
        v += l * (l + 1.0) / (2.0 * r * r);
      }
      bufd[S::addr(1 + 64 * k + lane)] = wdiag(A.tau, A.idx2, v);
    }
    wave_sync();
#pragma unroll
    for (int j = 0; j < M; ++j) {
      va[j] = bufd[S::addr(lane * M + j + 1)];
      if constexpr (!IN) va[j] = J + j < nloc ? va[j] : 0.0;
    }
    wave_sync();
  }
  // v where rows J + i - 1 and J + i are both of the system, else zero
  auto cpl = [&](int i, cd v) {
    return IN ? v : csel(J + i < nloc && row0 + J + i > 0, v, zero);
  };
  WBlk b;
  WRhs<1> c;
  {
    cd p = D[0];  // psi of the row before (rows past the end hold zero and have no right-hand side)
    D[0] = wrhs(va[0], kap, p, D[1]);
    if constexpr (!IN) D[0] = csel(J < nloc, D[0], zero);
    cd h = zero, beta = zero, fb = zero, fd = zero;
#pragma unroll
    for (int i = 1; i < M; ++i) {
      cd d = wrhs(va[i], kap, D[i], cadd(p, i + 1 < M ? D[i + 1 < M ? i + 1 : i] : zM));
      if constexpr (!IN) d = csel(J + i < nloc, d, zero);
      p = D[i];
      if (i == 1) {
        const cd g = crecip(mk(-va[1], 1.0));
        h = rmul(kap, g);
        D[1] = cmul(d, g);
        fb = beta = cpl(1, h);
        fd = D[1];
      } else {
        const cd g = crecip(rfms(kap, cpl(i, h), mk(-va[i], 1.0)));
        h = rmul(kap, g);
        D[i] = cmul(rfms(kap, cpl(i, D[i - 1]), d), g);
        fd = cfms(beta, D[i], fd);
        const cd bi = cpl(i, cneg(cmul(beta, h)));
        fb = cfms(beta, bi, fb);
        beta = bi;
      }
    }
    b.UA = rfms(kap, fb, mk(-va[0], 1.0));
    b.C = cpl(M, rmul(-kap, beta));
    b.DA = cpl(M, rmul(-kap, h));
    c.UD[0] = rfms(kap, fd, D[0]);
    c.DD[0] = cpl(M, rmul(-kap, cadd(p, D[M - 1])));
  }
  // a non-finite row of the block shows in its U slot
  bool bad = __any(!cfinite(b.UA) || !cfinite(c.UD[0]));
  const int lv = A.lv, sp = 1 << lv;
  rlevel_up<1>(b, c, nodes, lane);
  rlevel_up<2>(b, c, nodes, lane);
  rlevel_up<4>(b, c, nodes, lane);
  if (lv > 3) rlevel_up<8>(b, c, nodes, lane);
  if (lv > 4) rlevel_up<16>(b, c, nodes, lane);
  if (lv > 5) rlevel_up<32>(b, c, nodes, lane);

  // ---- the blocks' joint lines: own U slot plus the D slot of the block before
  double* mine = A.lk + ((int64_t)e * A.lk_n + gt) * 8;
  if (multi && !FIX) {
    double* next = A.lk + ((int64_t)(1 - e) * A.lk_n + gt) * 8;
    if (wave == 0) line_put(mine, b.UA, c.UD[0], 0, lane);
    if (wave == W - 1) line_put(mine + 4, b.DA, c.DD[0], 64 - sp, lane);
    if (wave == 0 && lane < 8) next[lane] = __longlong_as_double(-1ll);
  }
  if constexpr (W > 1) {
    if (lane == 0) {
      sm.ua[wave] = b.UA;
      sm.ud[wave] = c.UD[0];
      sm.bad[wave] = bad;
    }
    if (lane == 64 - sp) {
      sm.da[wave] = b.DA;
      sm.dd[wave] = c.DD[0];
    }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < W; ++w) bad |= sm.bad[w] != 0;
  }
  cd lA = zero, lD = zero, rA = zero, rD = zero;  // the slots beyond the wavefront's ends
  bool have = true;
  if (wave > 0) {
    lA = sm.da[wave - 1];
    lD = sm.dd[wave - 1];
  } else if (tile > 0) {
    have = line_get<FIX>(mine - 8 + 4, lA, lD, lane, A.spin);
  }
  const bool past = wave == W - 1 && tile + 1 >= A.ntiles;  // the system's end
  if (wave + 1 < W) {
    rA = sm.ua[wave + 1];
    rD = sm.ud[wave + 1];
  } else if (!past) {
    const bool h = line_get<FIX>(mine + 8, rA, rD, lane, A.spin);
    have = have && h;
  }
  if (multi && !FIX) {
    if (lane == 0 && wave == 0) sm.ok[0] = have;
    if (lane == 0 && wave == W - 1) sm.ok[1] = have;
    if constexpr (W > 1) __syncthreads();
    else wave_sync();
    const bool ok = sm.ok[0] && sm.ok[1];
    if (threadIdx.x == 0) {
      A.done[gt] = ok;
      if (!ok || bad) A.st[2 + e] = 1;
      if (bad) A.bad[(int64_t)e * (A.lk_n / A.ntiles) + sys] = 1;
      if (tile == 0) A.bad[(int64_t)(1 - e) * (A.lk_n / A.ntiles) + sys] = 0;
      if (gt == 0) {
        A.st[1] = e;
        A.st[2 + (1 - e)] = 0;
      }
    }
    if (!ok) {
      if (threadIdx.x == 0) A.edge[gt] = sm.edge;
      return;
    }
  }
  cd qA = lane_get(b.DA, (lane - sp) & 63), qD = lane_get(c.DD[0], (lane - sp) & 63);
  qA = csel(lane < sp, lA, qA);
  qD = csel(lane < sp, lD, qD);
  cd pJ = cmul(cadd(qD, c.UD[0]), crecip(cadd(qA, b.UA)));
  cd pM = lane_get(pJ, (lane + sp) & 63);
  const cd pE = cmul(cadd(c.DD[0], rD), crecip(cadd(b.DA, rA)));
  pM = csel(lane >= 64 - sp, csel(past, zero, pE), pM);
  if (lv > 5) rlevel_down<32>(pJ, pM, nodes, lane);
  if (lv > 4) rlevel_down<16>(pJ, pM, nodes, lane);
  if (lv > 3) rlevel_down<8>(pJ, pM, nodes, lane);
  rlevel_down<4>(pJ, pM, nodes, lane);
  rlevel_down<2>(pJ, pM, nodes, lane);
  rlevel_down<1>(pJ, pM, nodes, lane);

  // ---- the pivots again (the empty asm hides that they are the same), psi' upwards
#pragma unroll
  for (int j = 1; j < M; ++j) asm volatile("" : "+v"(va[j]));
  {
    cd h[M];
    h[1] = rmul(kap, crecip(mk(-va[1], 1.0)));
    cd beta = cpl(1, h[1]);
    D[1] = cfms(beta, pJ, D[1]);
#pragma unroll
    for (int i = 2; i < M; ++i) {
      h[i] = rmul(kap, crecip(rfms(kap, cpl(i, h[i - 1]), mk(-va[i], 1.0))));
      beta = cpl(i, cneg(cmul(beta, h[i])));
      D[i] = cfms(beta, pJ, D[i]);
    }
    cd y = pM;
#pragma unroll
    for (int i = M - 1; i >= 1; --i) D[i] = y = cfms(h[i], y, D[i]);
    D[0] = pJ;
  }
  if (FIX) bad = A.bad[(int64_t)e * (A.lk_n / A.ntiles) + sys] != 0;
  bool inf = false;
#pragma unroll
  for (int j = 0; j < M; ++j) {
    const double nan = __builtin_nan("");
    D[j] = csel(bad, mk(nan, nan), D[j]);
    inf |= (IN || J + j < nloc) && !cfinite(D[j]);
  }
  if (__any(inf) && lane == 0) atomicOr(A.status, 1);
  wave_sync();
#pragma unroll
  for (int j = 0; j < M; ++j) buf[S::addr(lane * M + j + 1)] = D[j];
  wave_sync();
  int sl = lane;
  asm volatile("" : "+v"(sl));
  cd* o = A.out + sys * A.bs + row0;
#pragma unroll
  for (int k = 0; k < M; ++k) {
    const int q = w0 + 64 * k + sl;
    if (IN || (q < nloc && q < 64 * W * M)) o[q] = buf[S::addr(1 + 64 * k + sl)];
  }
}

template <int M, int W, bool XG, bool FIX>
__device__ __forceinline__ void rowstep_tile(const RowStepArgs& A, RowStepSmem<M, W>& sm,
                                             int64_t gt, int e) {
  const int64_t sys = gt / A.ntiles, tile = gt - sys * A.ntiles;
  const int64_t w0 = tile * (64 * W * M) + (threadIdx.x >> 6) * 64 * M;
  if (w0 >= 1 && w0 + 64 * M + 1 <= A.n)
    rowstep_run<M, W, XG, FIX, true>(A, sm, gt, sys, tile, e);
  else
    rowstep_run<M, W, XG, FIX, false>(A, sm, gt, sys, tile, e);
}

template <int M, int W, bool XG>
__global__ __launch_bounds__(64 * W, 4) void k_rowstep(RowStepArgs A) {
  __shared__ RowStepSmem<M, W> sm;
  rowstep_tile<M, W, XG, false>(A, sm, blockIdx.x, A.ntiles > 1 ? A.st[0] & 1 : 0);
}

// After a pass over systems of several tiles (as k_colstep_fix).
template <int M, int W, bool XG>
__global__ __launch_bounds__(64 * W) void k_rowstep_fix(RowStepArgs A) {
  __shared__ RowStepSmem<M, W> sm;
  const int e = A.st[1], ask[2] = {A.st[2], A.st[3]};
  if (ask[e]) {
    constexpr int64_t T = 64 * W * M;
    for (int64_t gt = blockIdx.x; gt < A.lk_n; gt += gridDim.x) {
      const int64_t sys = gt / A.ntiles, tile = gt - sys * A.ntiles;
      if (!A.done[gt]) {
        rowstep_tile<M, W, XG, true>(A, sm, gt, e);
      } else if (A.bad[(int64_t)e * (A.lk_n / A.ntiles) + sys]) {
        const double nan = __builtin_nan("");
        for (int64_t r = tile * T + threadIdx.x; r < (tile + 1) * T && r < A.n; r += 64 * W)
          A.out[sys * A.bs + r] = mk(nan, nan);
      }
      __syncthreads();
    }
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) A.st[0] = e ^ 1;
}

}  // namespace nsd
