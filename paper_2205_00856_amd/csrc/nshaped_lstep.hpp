// The field part of a partial-wave step in one pass (gfx950, FP64 complex): at every radial point
// r_s the Crank-Nicolson step in l with the coupling E r_s C, C_{l,l+1} = (l+1)/sqrt((2l+1)(2l+3)).
//
// T = 1 + i sigma C (sigma = tau E r) has a real off-diagonal times i and no other diagonal, so with
// y_l = (-i)^l u_l and psi_l = (-i)^l f_l the system is real,
//     u_l - sigma C_{l-1,l} u_{l-1} + sigma C_{l,l+1} u_{l+1}
//         = f_l + sigma C_{l-1,l} f_{l-1} - sigma C_{l,l+1} f_{l+1},
// with a complex right-hand side: the pivots 1 + sigma^2 C^2 / pivot and all multipliers are real
// numbers, and a row keeps 6 registers (D and its reciprocal pivot) instead of the 12 of complex
// reduced rows.  The first row of a block has its right-hand side split like its diagonal: the term
// of f_{l-1} is in the D slot of the block before.
//
// As in k_cols, a wavefront's lanes take 64 neighbouring systems (radial points), wavefront w the
// rows w M .. of each, and the joint lines of a system are eliminated in its lane by wavefront 0.
// The couplings C of the rows are computed once per workgroup, a row per thread.
//
// Bound by memory: 64 waves of 65536 points (134 MB a step) 49.8 us with the complex column kernel
// -> 24.6 us.  16 rows per lane need more than 128 registers.
#pragma once
#include "nshaped_kernels.hpp"

namespace nsd {

constexpr int kLRows = 8;   // rows per lane
constexpr int kLWaves = 8;  // most wavefronts of a workgroup (64 partial waves)

struct LStepArgs {
  const cd* in;
  cd* out;
  int64_t n, batch;  // partial waves; radial points (also the stride of a row)
  int64_t l0;
  double s0;  // tau E dr: sigma of system s is s0 (s + 1)
  int* status;
};

struct LBlk {
  double UA, UC, DB, DA;
  cd UD, DD;
};

// i^q z
__device__ __forceinline__ cd irot(int q, cd z) {
  switch (q & 3) {
    case 0: return z;
    case 1: return mk(-z.y, z.x);
    case 2: return mk(-z.x, -z.y);
  }
  return mk(z.y, -z.x);
}

template <int M>
__global__ __launch_bounds__(64 * kLWaves, 4) void k_lstep(LStepArgs A) {
  __shared__ LBlk sb[kLWaves][64];
  __shared__ cd jpsi[kLWaves + 1][64];
  __shared__ double cl[kLWaves * M + 1];  // C between rows q - 1 and q of the system, 0 at its ends
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int W = blockDim.x >> 6;
  const int64_t c0 = (int64_t)blockIdx.x * 64;
  const bool live = c0 + lane < A.batch;
  const int off = live ? lane : (int)(A.batch - 1 - c0);
  const uint32_t ob16 = (uint32_t)off * 16;
  const int r0 = wave * M, n = (int)A.n;
  // the rows' powers of -i count from this block's first row (M is a multiple of 4)
  cd D[M], fM;  // f; that of the row after the block
#pragma unroll
  for (int j = 0; j < M; ++j)
    D[j] = col_at(A.in + c0, ob16, r0 + j < n ? r0 + j : n - 1, A.batch);
  fM = col_at(A.in + c0, ob16, r0 + M < n ? r0 + M : n - 1, A.batch);
  for (int q = threadIdx.x; q <= W * M; q += blockDim.x) {
    const double l = (double)(A.l0 + q - 1);
    cl[q] = q > 0 && q < n ? (l + 1.0) / sqrt((2.0 * l + 1.0) * (2.0 * l + 3.0)) : 0.0;
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < M; ++j) D[j] = csel(r0 + j < n, irot(j, D[j]), czero());
  fM = csel(r0 + M < n, irot(M, fM), czero());
  const double sg = A.s0 * (double)(c0 + off + 1);
  auto e = [&](int j) { return sg * cl[r0 + j]; };
  double g[M];
  LBlk b;
  {
    // the right-hand sides (couplings past the system's ends are zero)
    cd p = D[0];
    D[0] = rfma(-e(1), D[1], p);
#pragma unroll
    for (int i = 1; i < M; ++i) {
      const cd f = D[i];
      D[i] = rfma(e(i), p, rfma(-e(i + 1), i + 1 < M ? D[i + 1 < M ? i + 1 : i] : fM, f));
      p = f;
    }
    g[1] = 1.0;
    double beta = -e(1), P = -e(2), fb = beta;
    cd fd = D[1];
#pragma unroll
    for (int i = 2; i < M; ++i) {
      const double ei = e(i);
      g[i] = rcp_nr(fma(ei * ei, g[i - 1], 1.0));
      D[i] = rmul(g[i], rfma(ei, D[i - 1], D[i]));
      beta = ei * beta * g[i];
      fb = fma(P, beta, fb);
      fd = rfma(P, D[i], fd);
      P = -(e(i + 1) * g[i]) * P;
    }
    const double e1 = e(1), eM = e(M);
    b.UA = fma(-e1, fb, 1.0);
    b.UC = e1 * P;
    b.UD = rfma(-e1, fd, D[0]);
    b.DB = eM * beta;
    b.DA = eM * eM * g[M - 1];
    b.DD = rmul(eM, cadd(p, D[M - 1]));
  }
  sb[wave][lane] = b;
  __syncthreads();
  if (wave == 0) {
#pragma unroll 1
    for (int w = 1; w < W; ++w) {
      const LBlk o = sb[w][lane];
      const double ia = rcp_nr(b.DA + o.UA);
      const double B = b.DB * ia, C = o.UC * ia;
      const cd dl = rmul(ia, cadd(b.DD, o.UD));
      b.UA = fma(-b.UC, B, b.UA);
      b.UD = rfma(-b.UC, dl, b.UD);
      b.UC = -b.UC * C;
      b.DB = -o.DB * B;
      b.DA = fma(-o.DB, C, o.DA);
      b.DD = rfma(-o.DB, dl, o.DD);
      sb[w][lane].UA = B;
      sb[w][lane].UC = C;
      sb[w][lane].UD = dl;
    }
    // the row past the last block is past the system's end: nothing couples to it
    const cd pJ = rmul(rcp_nr(b.UA), b.UD);
    jpsi[0][lane] = pJ;
    jpsi[W][lane] = czero();
    cd y = czero();
#pragma unroll 1
    for (int w = W - 1; w >= 1; --w) {
      // the powers of -i count from each block's first row: the same for every block (M % 4 == 0)
      y = rfma(-sb[w][lane].UC, y, rfma(-sb[w][lane].UA, pJ, sb[w][lane].UD));
      jpsi[w][lane] = y;
    }
  }
  __syncthreads();
  const cd pJ = jpsi[wave][lane];
  const cd pM = jpsi[wave + 1][lane];
  bool bad = false;
  auto put = [&](int i, cd f) {
    const cd p = irot(-i, f);
    if (live && r0 + i < n) {
      col_at(A.out + c0, ob16, r0 + i, A.batch) = p;
      bad |= !cfinite(p);
    }
  };
  {
    double beta = -e(1);
    D[1] = rfma(-beta, pJ, D[1]);
#pragma unroll
    for (int i = 2; i < M; ++i) {
      beta = e(i) * beta * g[i];
      D[i] = rfma(-beta, pJ, D[i]);
    }
  }
  cd y = pM;
#pragma unroll
  for (int i = M - 1; i >= 1; --i) {
    y = rfma(-(e(i + 1) * g[i]), y, D[i]);
    put(i, y);
  }
  put(0, pJ);
  if (__any(bad) && lane == 0) atomicOr(A.status, 1);
}

}  // namespace nsd
