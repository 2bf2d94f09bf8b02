// A Crank-Nicolson step of an interleaved batch in one pass (gfx950, FP64 complex).
//
// As in k_cols, a wavefront's 64 lanes take 64 neighbouring systems (every row one coalesced
// access) and a workgroup a tile of T = W M rows of them.  As in k_tile<PH_LINK>, a tile takes psi
// at its two joint lines from its own slots and its neighbours': the host launches this form only
// when joints T rows apart are decoupled in every real potential (decoupled(): 2^-66 of the
// diagonal), so no reduced system is solved at all.  The rows are those of k_window; a wavefront
// loads the row after its block as well, mostly from the L2 that its neighbour fills.  In place: as
// in k_rowstep a tile stores once both neighbours have published, and a tile that is left keeps the
// edge row that it has loaded.  The pivots are formed a second time on the way back: across the
// exchange a row keeps D and the diagonal, 6 registers.
//
// The tile's line (DA, DD, UA, UD of 64 systems) is published word by word, all-ones words marking
// what has not arrived; lines alternate between two buffers, and a pass clears the one of the
// next.  A tile whose wait reaches its bound is left to k_colstep_fix, which runs it from the
// lines, all there by then, with the same bits.  A system with a non-finite row is marked, and
// k_colstep_fix makes all of it NaN, as exact steps would.
//
// Workgroups are numbered in bands of kColBand column groups, tile by tile: a wait is for the
// workgroup kColBand ids later, which has to be resident beside this one (with 16 rows per lane 256
// are), and 4096 neighbouring systems keep the accesses long.  Numbered over all groups of a wider
// batch the waits ran to their bound and every tile was left.
//
// Bound by memory: 40 bytes a row and the lines (8 KB written and 4 KB read per tile of 64 rows of
// 64 systems, 160 KB of rows).  4096 x 4096 rows: 231 us in two passes (64 bytes a row, the second
// pass at one wavefront per SIMD) -> 148; 1531 systems of 1000 rows 40.5 -> 17.7 us.
#pragma once
#include "nshaped_windows.hpp"

namespace nsd {

constexpr uint32_t kColBand = 64;

struct ColStepArgs {
  const cd* in;
  cd* out;
  const double* V;
  const double* xg;
  int64_t n, es, batch, ntiles;  // rows and their stride, systems (stride 1), tiles of a system
  double vscale, E, tau, kap, idx2;
  double* lk;     // lines: [2][lk_n][8][64]
  int64_t lk_n;   // tiles of all column groups
  int* st;        // [buffer of the next pass, of this pass, whether pass of buffer 0, 1 needs a fix]
  int* done;      // per tile: finished by the pass
  int* bad;       // [2][batch]: systems with a non-finite row
  cd* edge;       // [lk_n][64]: of a tile left to the fix, psi of the row after its last one
  int* status;
  int spin;       // polls of a line before its tile is left
};

template <int W>
struct ColStepSmem {
  WBlk b[W][64];      // the blocks' matrix slots; after the elimination (B, C, dl) of joint w
  WRhs<1> c[W][64];
  cd jpsi[W + 1][64];  // the solution at the tile's joint lines
  cd edge[64];         // psi of the row after the tile
  int ok;
};

// Tile gt = tile * (column groups) + group, whose lines are in buffer e.  FIX: the lines are
// complete, and the lanes of marked systems store NaN.
template <int M, int W, bool XG, bool FIX, bool IN>
__device__ __forceinline__ void colstep_run(const ColStepArgs& A, ColStepSmem<W>& sm, int64_t gt,
                                            int64_t ncg, int64_t tile, int64_t c0, int e) {
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const bool live = c0 + lane < A.batch;
  const uint32_t ob16 = (uint32_t)((live ? lane : A.batch - 1 - c0) * 16), ob8 = ob16 / 2;
  const int64_t r0 = tile * (M * W) + (int64_t)wave * M, n = A.n;
  const double kap = A.kap;
  const cd zero = czero();

  cd D[M], zM;  // psi; its row r0 + M
  double va[M];
  {
    double v[M], xv[XG ? M : 1];
    auto row = [&](int j) { return IN ? r0 + j : (r0 + j < n ? r0 + j : n - 1); };
#pragma unroll
    for (int j = 0; j < M; ++j) D[j] = col_at(A.in + c0, ob16, row(j), A.es);
    zM = col_at(A.in + c0, ob16, row(M), A.es);
#pragma unroll
    for (int j = 0; j < M; ++j) v[j] = col_at(A.V + c0, ob8, row(j), A.es);
    if constexpr (XG) {
#pragma unroll
      for (int j = 0; j < M; ++j) xv[j] = col_at(A.xg + c0, ob8, row(j), A.es);
    }
    if (wave == W - 1 && tile + 1 < A.ntiles) {
      // (in place, the next tile may have stored by the time of the fix)
      if constexpr (FIX) zM = A.edge[gt * 64 + lane];
      else sm.edge[lane] = zM;
    }
    if constexpr (!IN) zM = csel(r0 + M < n, zM, zero);
#pragma unroll
    for (int j = 0; j < M; ++j) {
      va[j] = wdiag(A.tau, A.idx2, XG ? fma(xv[XG ? j : 0], A.E, A.vscale * v[j])
                                      : A.vscale * v[j]);
      if constexpr (!IN) {
        D[j] = csel(r0 + j < n, D[j], zero);
        va[j] = r0 + j < n ? va[j] : 0.0;
      }
    }
  }
  // v where rows r0 + i - 1 and r0 + i are both of the system, else zero
  auto cpl = [&](int i, cd v) { return IN ? v : csel(r0 + i < n && r0 + i > 0, v, zero); };
  WBlk b;
  WRhs<1> c;
  {
    cd p = D[0];  // psi of the row before (rows past the end hold zero and have no right-hand side)
    D[0] = wrhs(va[0], kap, p, D[1]);
    if constexpr (!IN) D[0] = csel(r0 < n, D[0], zero);
    cd h = zero, beta = zero, fb = zero, fd = zero;
#pragma unroll
    for (int i = 1; i < M; ++i) {
      cd d = wrhs(va[i], kap, D[i], cadd(p, i + 1 < M ? D[i + 1 < M ? i + 1 : i] : zM));
      if constexpr (!IN) d = csel(r0 + i < n, d, zero);
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
  sm.b[wave][lane] = b;
  sm.c[wave][lane] = c;
  if constexpr (!FIX) {
    // a non-finite row of the block shows in its U slot; marked before the wait, so whether or not
    // this pass finishes the tile
    const bool nf = live && !(cfinite(b.UA) && cfinite(c.UD[0]));
    if (nf) A.bad[(int64_t)e * A.batch + c0 + lane] = 1;
    if (__any(nf) && lane == 0) A.st[2 + e] = 1;
  }
  __syncthreads();
  if (wave == 0) {
#pragma unroll 1
    for (int w = 1; w < W; ++w) {
      const WBlk o = sm.b[w][lane];
      const WRhs<1> p = sm.c[w][lane];
      WNode t;
      wmerge(b, o, t);
      cd dl[1];
      wmerge_rhs<1>(c, p, t.ia, t.rU, t.rD, dl);
      sm.b[w][lane].UA = t.B;
      sm.b[w][lane].C = t.C;
      sm.b[w][lane].DA = dl[0];
    }
    // ---- the joint lines of the tile from its own and its neighbours' slots
    double* mine = A.lk + ((int64_t)e * A.lk_n + gt) * 512 + lane;
    const bool left = tile > 0, right = tile + 1 < A.ntiles;
    if constexpr (!FIX) {
      const double v[8] = {b.DA.x, b.DA.y, c.DD[0].x, c.DD[0].y,
                           b.UA.x, b.UA.y, c.UD[0].x, c.UD[0].y};
#pragma unroll
      for (int f = 0; f < 8; ++f)
        __hip_atomic_store(mine + 64 * f, v[f], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      double* next = A.lk + ((int64_t)(1 - e) * A.lk_n + gt) * 512 + lane;
#pragma unroll
      for (int f = 0; f < 8; ++f) next[64 * f] = __longlong_as_double(-1ll);
    }
    const long long* sl = reinterpret_cast<const long long*>(mine - (left ? ncg * 512 : 0));
    const long long* sr = reinterpret_cast<const long long*>(mine + (right ? ncg * 512 : 0)) + 256;
    long long q[8];
#pragma unroll
    for (int f = 0; f < 8; ++f) q[f] = (f < 4 ? left : right) ? -1ll : 0ll;
    bool in = false;
    for (int it = 0; it < (FIX ? 1 : A.spin); ++it) {
#pragma unroll
      for (int f = 0; f < 4; ++f) {
        q[f] = left ? __hip_atomic_load(sl + 64 * f, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
        q[4 + f] =
            right ? __hip_atomic_load(sr + 64 * f, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
      }
      if constexpr (FIX) break;
      in = true;
#pragma unroll
      for (int f = 0; f < 8; ++f) in = in && q[f] != -1ll;
      if (__all(in)) break;
      __builtin_amdgcn_s_sleep(1);
    }
    double d[8];
#pragma unroll
    for (int f = 0; f < 8; ++f) d[f] = __longlong_as_double(q[f]);
    const cd pJ = cmul(cadd(mk(d[2], d[3]), c.UD[0]), crecip(cadd(mk(d[0], d[1]), b.UA)));
    const cd pM = right ? cmul(cadd(c.DD[0], mk(d[6], d[7])), crecip(cadd(b.DA, mk(d[4], d[5]))))
                        : zero;
    sm.jpsi[0][lane] = pJ;
    sm.jpsi[W][lane] = pM;
    cd y = pM;
#pragma unroll 1
    for (int w = W - 1; w >= 1; --w) {
      const WBlk t = sm.b[w][lane];
      y = cfms(t.C, y, cfms(t.UA, pJ, t.DA));
      sm.jpsi[w][lane] = y;
    }
    if constexpr (!FIX) {
      const bool ok = __all(in);
      if (lane == 0) {
        sm.ok = ok;
        A.done[gt] = ok;
        if (!ok) A.st[2 + e] = 1;
        if (gt == 0) {
          A.st[1] = e;
          A.st[2 + (1 - e)] = 0;
        }
      }
      if (tile == 0 && live) A.bad[(int64_t)(1 - e) * A.batch + c0 + lane] = 0;
    }
  }
  __syncthreads();
  if constexpr (!FIX) {
    if (!sm.ok) {
      if (wave == W - 1) A.edge[gt * 64 + lane] = sm.edge[lane];
      return;
    }
  }
  // ---- psi' upwards
  const cd pJ = sm.jpsi[wave][lane];
  const cd pM = sm.jpsi[wave + 1][lane];
  bool bad = false;
  bool seen = false;
  if constexpr (FIX) seen = live && A.bad[(int64_t)e * A.batch + c0 + lane];
  auto put = [&](int i, cd p) {
    const double nan = __builtin_nan("");
    if constexpr (FIX) p = csel(seen, mk(nan, nan), p);
    if (live && (IN || r0 + i < n)) {
      col_at(A.out + c0, ob16, r0 + i, A.es) = p;
      bad |= !cfinite(p);
    }
  };
  // the pivots again (the empty asm hides that they are the same), dp_i = D_i - beta_i pJ
#pragma unroll
  for (int j = 1; j < M; ++j) asm volatile("" : "+v"(va[j]));
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
  for (int i = M - 1; i >= 1; --i) {
    y = cfms(h[i], y, D[i]);
    put(i, y);
  }
  put(0, pJ);
  if (__any(bad) && lane == 0) atomicOr(A.status, 1);
}

template <int M, int W, bool XG, bool FIX>
__device__ __forceinline__ void colstep_tile(const ColStepArgs& A, ColStepSmem<W>& sm,
                                             uint32_t tile, uint32_t cg, int e) {
  const int64_t ncg = (A.batch + 63) / 64, gt = tile * ncg + cg, c0 = (int64_t)cg * 64;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t r0 = (int64_t)tile * (M * W) + (int64_t)wave * M;
  if (r0 >= 1 && r0 + M < A.n)
    colstep_run<M, W, XG, FIX, true>(A, sm, gt, ncg, tile, c0, e);
  else
    colstep_run<M, W, XG, FIX, false>(A, sm, gt, ncg, tile, c0, e);
}

template <int M, int W, bool XG>
__global__ __launch_bounds__(64 * W, M == 8 ? 4 : 2) void k_colstep(ColStepArgs A) {
  __shared__ ColStepSmem<W> sm;
  // (the host launches fewer than 2^31 workgroups)
  const uint32_t ncg = (uint32_t)((A.batch + 63) / 64), nt = (uint32_t)A.ntiles;
  const uint32_t band = blockIdx.x / (kColBand * nt), g0 = band * kColBand;
  const uint32_t width = ncg - g0 < kColBand ? ncg - g0 : kColBand;
  const uint32_t rest = blockIdx.x - g0 * nt, tile = rest / width;
  colstep_tile<M, W, XG, false>(A, sm, tile, g0 + (rest - tile * width), A.st[0] & 1);
}

// After a pass: the tiles it has left, and NaN for the systems it has marked.  Nothing to do after
// nearly every pass, so a few workgroups.
template <int M, int W, bool XG>
__global__ __launch_bounds__(64 * W) void k_colstep_fix(ColStepArgs A) {
  __shared__ ColStepSmem<W> sm;
  const int e = A.st[1], ask[2] = {A.st[2], A.st[3]};
  if (ask[e]) {
    const int64_t ncg = (A.batch + 63) / 64;
    for (int64_t gt = blockIdx.x; gt < A.lk_n; gt += gridDim.x) {
      const int64_t tile = gt / ncg, cg = gt - tile * ncg;
      if (!A.done[gt]) {
        colstep_tile<M, W, XG, true>(A, sm, (uint32_t)tile, (uint32_t)cg, e);
      } else {
        const int64_t sys = cg * 64 + (threadIdx.x & 63);
        if (sys < A.batch && A.bad[(int64_t)e * A.batch + sys]) {
          const double nan = __builtin_nan("");
          for (int64_t r = tile * M * W + (threadIdx.x >> 6); r < (tile + 1) * M * W && r < A.n;
               r += W)
            A.out[sys + r * A.es] = mk(nan, nan);
        }
      }
      __syncthreads();
    }
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) A.st[0] = e ^ 1;
}

}  // namespace nsd
