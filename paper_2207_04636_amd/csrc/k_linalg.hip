// Dense FP64 linear algebra of the ISDF set-up.
//
// * Cholesky factorisation of the fitting metric X_gg (Sec. 4.3 solves the
//   least-squares fit of Sec. 3.1, Eq. 11, with a Cholesky factorisation):
//   blocked right-looking, 64-column panels factored by one wave, the block column
//   below by substitution, the trailing matrix by the FP64 MFMA product.
// * Triangular solves with many right-hand sides (the N_g columns of X_gR, or
//   the N_chi columns when forming W): 64-row diagonal blocks by one wave per
//   16 right-hand sides, the rest by matrix products.
// * Pivoted Cholesky of an explicit Gram matrix.  QR with column pivoting of a
//   matrix M (Sec. 3.1, 4.3) picks as pivot k the column whose norm, after
//   projecting out the columns picked before, is largest.  That residual norm
//   squared is the updated diagonal of a Cholesky factorisation of M^T M with
//   the same pivot order, so the pivots are those of QRCP in exact arithmetic.
//   An explicit Gram matrix is updated after each panel of 32 steps; the per-atom
//   sets of the selection never form theirs.
#include <math.h>

#include <algorithm>
#include <type_traits>

#include "mfma.h"
#include "rps_internal.h"

namespace rps {
namespace {

constexpr int NB = 64;

// One wave factors the 64 x 64 block with row i in lane i's registers.  The kernel is one
// serial chain (a square root, a quotient and a rank-1 update per column); nothing but its
// latency counts, so no barrier stands in it: column j goes round through LDS and every
// lane updates its row with 64 - j independent products.  A workgroup of 256 with the block
// in LDS and three barriers per column took 99 us.
__global__ __launch_bounds__(64) void chol_panel_kernel(double* A, int64_t lda, int64_t k0, int32_t* status) {
  __shared__ __align__(16) double col[NB];
  const int lane = threadIdx.x;
  double* row = A + (k0 + lane) * lda + k0;
  double x[NB];               // entries past the diagonal are never stored
#pragma unroll
  for (int j = 0; j < NB; ++j) x[j] = row[j];
  auto columns = [&](auto jb) {          // columns 16 jb .. 16 jb + 15
    constexpr int J0 = 16 * decltype(jb)::value;
#pragma unroll
    for (int jj = 0; jj < 16; ++jj) {
      const int j = J0 + jj;
      double d = __shfl(x[j], j, 64);
      if (!(d > 0.0)) {
        if (lane == 0 && status[0] == 0) status[0] = (int32_t)(1 + k0 + j);
        d = 1.0;
      }
      const double piv = sqrt(d);
      x[j] = (lane == j) ? piv : x[j] / piv;
      col[lane] = x[j];
      __builtin_amdgcn_wave_barrier();
      double c[NB - J0];
#pragma unroll
      for (int u = 0; u < NB - J0; ++u) c[u] = col[J0 + u];
#pragma unroll
      for (int u = jj + 1; u < NB - J0; ++u) x[J0 + u] -= x[j] * c[u];
      // (done here: put off to their uses the products would keep every c alive)
#pragma unroll
      for (int u = jj + 1; u < NB - J0; ++u) asm volatile("" : "+v"(x[J0 + u]));
      __builtin_amdgcn_wave_barrier();
    }
  };
  columns(std::integral_constant<int, 0>{});
  columns(std::integral_constant<int, 1>{});
  columns(std::integral_constant<int, 2>{});
  columns(std::integral_constant<int, 3>{});
#pragma unroll
  for (int j = 0; j < NB; ++j)
    if (j <= lane) row[j] = x[j];
}

// Solve 64-vectors v against the 64x64 lower triangle L: TRANS = false: L x = v
// (forward), TRANS = true: L^T x = v (backward).  Vector v number t has component j at
// base[t*sv + j*sj].  A wave takes 16 vectors, component 16 b + 4 r + lane / 16 of vector
// lane % 16 in x[b][r]: this is at once the result and the operand layout of the FP64
// matrix instruction, so the six 16 x 16 blocks off the diagonal are matrix products on
// registers.  The four on it are substitutions: component i goes round by a lane
// permutation, every lane divides, and subtracts it from the components it holds.  What is
// left is the latency of 64 such steps; two waves per SIMD share it at 32768 vectors.
// (One vector per thread, each component a chain of products over those before it, was
// 2016 dependent operations at one wave per SIMD: 49 us there against 18 us now.)
constexpr int TRI = 64;       // vectors of a workgroup (four waves)
template <bool TRANS>
__global__ __launch_bounds__(256) void tri64_kernel(const double* __restrict__ Lg, int64_t ldl, double* base,
                                                   int64_t sv, int64_t sj, int64_t nvec) {
  __shared__ double S[NB][NB + 2];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int l16 = lane & 15, lq = lane >> 4;
  const int64_t t = (int64_t)blockIdx.x * TRI + 16 * w + l16;
  double* v = base + (t < nvec ? t : nvec - 1) * sv;
  d4_t x[4];
#pragma unroll
  for (int b = 0; b < 4; ++b)
#pragma unroll
    for (int r = 0; r < 4; ++r) x[b][r] = v[(16 * b + 4 * r + lq) * sj];
#pragma unroll
  for (int u = 0; u < NB * NB / 256; ++u) {
    const int e = tid + 256 * u, i = e / NB, j = e % NB;
    S[i][j] = Lg[(int64_t)i * ldl + j];          // (nothing reads its upper triangle)
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int b = TRANS ? 3 - q : q;             // block solved now
    const int o = 16 * b;
    double f[16][4];                             // factor of component i in component 4 r + lq of the block
#pragma unroll
    for (int i = 0; i < 16; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) f[i][r] = TRANS ? S[o + i][o + 4 * r + lq] : S[o + 4 * r + lq][o + i];
#pragma unroll
    for (int s = 0; s < 16; ++s) {
      const int i = TRANS ? 15 - s : s;
      const double xi = __shfl(x[b][i >> 2], (i & 3) * 16 + l16, 64) / S[o + i][o + i];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int c = 4 * r + lq;
        if (c == i) x[b][r] = xi;
        else if (TRANS ? c < i : c > i) x[b][r] -= f[i][r] * xi;
      }
    }
    // the blocks still to be solved minus this one's contribution
#pragma unroll
    for (int p = q + 1; p < 4; ++p) {
      const int m = TRANS ? 3 - p : p;
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const double a = TRANS ? S[o + 4 * k + lq][16 * m + l16] : S[16 * m + l16][o + 4 * k + lq];
        x[m] = mfma_f64(-a, x[b][k], x[m]);
      }
    }
  }
  if (t >= nvec) return;
#pragma unroll
  for (int b = 0; b < 4; ++b)
#pragma unroll
    for (int r = 0; r < 4; ++r) v[(16 * b + 4 * r + lq) * sj] = x[b][r];
}

// ---------------- pivoted Cholesky
// The pivot of a step is the largest residual diagonal, ties to the lowest index; an
// index that is taken (-inf) or not a number never wins.  No winner: index -1.
struct PcBest {
  double v;
  int32_t i;
};
__device__ __forceinline__ PcBest pc_pick(PcBest a, PcBest b) {
  const bool take = (b.i >= 0) && (a.i < 0 || b.v > a.v || (b.v == a.v && b.i < a.i));
  return take ? b : a;
}
__device__ __forceinline__ PcBest pc_of(double d, int32_t j) { return PcBest{d, (d > -INFINITY) ? j : -1}; }
__device__ __forceinline__ PcBest pc_wave(PcBest b) {
  for (int off = 32; off > 0; off >>= 1) {
    const PcBest o{__shfl_xor(b.v, off, 64), __shfl_xor(b.i, off, 64)};
    b = pc_pick(b, o);
  }
  return b;
}
// over the 256 threads of a workgroup (every thread gets the result)
__device__ __forceinline__ PcBest pc_block256(PcBest b, PcBest* red) {
  b = pc_wave(b);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = b;
  __syncthreads();
  return pc_pick(pc_pick(red[0], red[1]), pc_pick(red[2], red[3]));
}

// One pivot step of every set in one launch (blockIdx.y = set, 256 candidates per
// workgroup).  Each workgroup first reduces the block maxima that the previous step left,
// so a step is one launch: column k of the factor
//   L[j][k] = (G[p][j] - sum_{t=kb}^{k-1} L[j][t] L[p][t]) / sqrt(d_p),
// the residual diagonal d_j -= L[j][k]^2, and the block maxima of the new diagonal.
// k < 0 forms the diagonal and its block maxima only.
//   FACT: G is never formed; G[p][j] = (a_p . a_j)(b_p . b_j) comes from the sketch
//         products (PcArgs::AB, one column per candidate), L holds one column of the set
//         after another.  A step reads 2p + k values per candidate: an atom's Gram matrix
//         has |kappa|^2 (512 MB for a set of 8000) and was formed for 50-odd of its rows.
//   else: one set with an explicit Gram matrix, updated by the caller after each panel;
//         L row-major.
// Bound by the launch and two dependent reads of a step: at 8 atoms of 8000 candidates
// and 62 pivots each, 63 launches of 11 us (0.7 ms) take the place of 992 launches of
// 4-5 us, 16 Gram products and 8 updates (14 ms in all).
template <bool FACT>
__global__ __launch_bounds__(256) void pchol_step_kernel(PcArgs a, int64_t k, int64_t kb) {
  extern __shared__ double sh[];       // L[p][kb..k), then a_p and b_p
  __shared__ PcBest red[4];
  const PcSet it = FACT ? a.sets[blockIdx.y] : PcSet{0, a.n, a.k, 0};
  const int64_t n = it.n;
  const int nb = (int)((n + 255) / 256);
  if ((int)blockIdx.x >= nb || k >= it.k) return;      // uniform over the workgroup
  const int tid = threadIdx.x;
  const int64_t j = (int64_t)blockIdx.x * 256 + tid;
  double* diag = a.diag + it.row0;
  const int64_t slot = (int64_t)blockIdx.y * a.nbmax;
  const int64_t half = (int64_t)gridDim.y * a.nbmax;
  double d = -INFINITY;
  if (k < 0) {
    if (j < n) {
      if constexpr (FACT) {
        double x = 0.0, y = 0.0;
        for (int q = 0; q < a.p; ++q) {
          const double u = a.AB[q * a.ldab + it.row0 + j], v = a.AB[(a.p + q) * a.ldab + it.row0 + j];
          x += u * u;
          y += v * v;
        }
        d = x * y;
      } else {
        d = a.G[j * a.ld + j];
      }
      diag[j] = d;
    }
  } else {
    const double* bv = a.bv + ((k + 1) & 1) * half + slot;
    const int32_t* bi = a.bi + ((k + 1) & 1) * half + slot;
    PcBest b{0.0, -1};
    for (int e = tid; e < nb; e += 256) b = pc_pick(b, PcBest{bv[e], bi[e]});
    b = pc_block256(b, red);
    const int64_t p = (b.i >= 0) ? b.i : 0;
    const double dp = (b.i >= 0) ? b.v : 0.0;
    if (blockIdx.x == 0 && tid == 0) a.piv[it.pofs + k] = p;
    const int nt = (int)(k - kb);
    double* Ls = a.L + (FACT ? it.row0 * a.ldl : 0);
    for (int t = tid; t < nt; t += 256) sh[t] = FACT ? Ls[(kb + t) * n + p] : Ls[p * a.ldl + kb + t];
    if constexpr (FACT)
      for (int q = tid; q < 2 * a.p; q += 256) sh[nt + q] = a.AB[q * a.ldab + it.row0 + p];
    __syncthreads();
    if (j < n) {
      d = diag[j];
      double l = 0.0;
      if (!(d == -INFINITY && j != p)) {       // else already selected: its residual is zero
        double s;
        if constexpr (FACT) {
          double x = 0.0, y = 0.0;
          for (int q = 0; q < a.p; ++q) {
            x += a.AB[q * a.ldab + it.row0 + j] * sh[nt + q];
            y += a.AB[(a.p + q) * a.ldab + it.row0 + j] * sh[nt + a.p + q];
          }
          s = x * y;
          for (int t = 0; t < nt; ++t) s -= Ls[(kb + t) * n + j] * sh[t];
        } else {
          s = a.G[p * a.ld + j];
          for (int t = 0; t < nt; ++t) s -= Ls[j * a.ldl + kb + t] * sh[t];
        }
        if (dp > 0.0) l = s / sqrt(dp);
        d = (j == p) ? -INFINITY : d - l * l;
        diag[j] = d;
      }
      if constexpr (FACT) Ls[k * n + j] = l;
      else Ls[j * a.ldl + k] = l;
    }
  }
  const PcBest m = pc_block256(pc_of(d, (int32_t)j), red);
  if (tid == 0) {
    const int64_t o = (k & 1) * half + slot + blockIdx.x;      // k = -1 and odd steps share a half
    a.bv[o] = m.v;
    a.bi[o] = m.i;
  }
}

// A panel of up to 32 pivot steps of one set of at most 1024 candidates in one workgroup,
// thread j holding candidate j's residual and panel row of L in registers (the same sums in
// the same order as the step kernel).  A step costs two barriers and one read of a row of G:
// 416 pivots of 496 candidates took two launches and 8.9 us a pivot, here 2.2 us.
constexpr int PCP = 32;
__global__ __launch_bounds__(1024) void pchol_panel_kernel(const double* __restrict__ G, int n, int64_t ld,
                                                          double* __restrict__ L, int64_t ldl, int64_t kb,
                                                          int steps, double* __restrict__ diag,
                                                          int64_t* __restrict__ piv) {
  __shared__ PcBest red[16];
  __shared__ double lp[PCP];
  const int j = threadIdx.x;
  const bool live = j < n;
  double d = live ? (kb == 0 ? G[(int64_t)j * ld + j] : diag[j]) : -INFINITY;
  double l[PCP];
#pragma unroll
  for (int kk = 0; kk < PCP; ++kk) {
    l[kk] = 0.0;
    if (kk < steps) {      // uniform
      PcBest b = pc_wave(pc_of(d, j));
      if ((j & 63) == 0) red[j >> 6] = b;
      __syncthreads();
      b = red[j & 15];
      for (int off = 8; off > 0; off >>= 1) {
        const PcBest o{__shfl_xor(b.v, off, 64), __shfl_xor(b.i, off, 64)};
        b = pc_pick(b, o);
      }
      const int p = (b.i >= 0) ? b.i : 0;
      const double dp = (b.i >= 0) ? b.v : 0.0;
      double s = live ? G[(int64_t)p * ld + j] : 0.0;
      if (j == p) {
#pragma unroll
        for (int t = 0; t < kk; ++t) lp[t] = l[t];
        piv[kb + kk] = p;
      }
      __syncthreads();
      if (live) {
        if (!(d == -INFINITY && j != p)) {
#pragma unroll
          for (int t = 0; t < kk; ++t) s -= l[t] * lp[t];
          if (dp > 0.0) l[kk] = s / sqrt(dp);
          d = (j == p) ? -INFINITY : d - l[kk] * l[kk];
        }
        L[(int64_t)j * ldl + kb + kk] = l[kk];
      }
    }
  }
  if (live) diag[j] = d;
}

inline unsigned nblk(int64_t n, int b) { return (unsigned)((n + b - 1) / b); }

}  // namespace

hipError_t cholesky_lower(double* A, int64_t n, int64_t lda, int32_t* status, hipStream_t s) {
  hipError_t e = hipMemsetAsync(status, 0, sizeof(int32_t), s);
  if (e != hipSuccess) return e;
  for (int64_t k0 = 0; k0 < n; k0 += NB) {
    hipLaunchKernelGGL(chol_panel_kernel, dim3(1), dim3(64), 0, s, A, lda, k0, status);
    const int64_t rest = n - k0 - NB;
    if (rest <= 0) break;
    // A21 <- A21 L11^-T : each row x solves L11 x = a
    hipLaunchKernelGGL(tri64_kernel<false>, dim3(nblk(rest, TRI)), dim3(256), 0, s,
                       A + k0 * lda + k0, lda, A + (k0 + NB) * lda + k0, lda, (int64_t)1, rest);
    Gemm g;
    g.M = rest; g.N = rest; g.K = NB;
    g.A = A + (k0 + NB) * lda + k0; g.lda = lda;
    g.B = A + (k0 + NB) * lda + k0; g.ldb = lda; g.transB = true;
    g.C = A + (k0 + NB) * lda + k0 + NB; g.ldc = lda;
    g.alpha = -1.0; g.beta = 1.0; g.lower_only = true;
    e = gemm_f64(g, s);
    if (e != hipSuccess) return e;
  }
  return hipGetLastError();
}

// Two-level blocked solve.  Outer blocks of NB2 rows: the block is solved 64 rows
// at a time (the 64 x 64 triangle in LDS, 16 right-hand sides per wave, and
// rank-64 updates confined to the block's rows), then the rest of B takes one
// rank-NB2 update.  The updates that sweep all of B are therefore NB2 deep, so B
// streams through HBM n / NB2 times instead of n / 64 times.
hipError_t tri_solve_lower(const double* L, int64_t n, int64_t ldl, double* B, int64_t ncols,
                           int64_t ldb, bool trans, hipStream_t s) {
  constexpr int64_t NB2 = 512;
  if (n % NB != 0) return hipErrorInvalidValue;
  const int64_t nout = (n + NB2 - 1) / NB2;
  auto update = [&](int64_t r0, int64_t r1, int64_t k0, int64_t kb) -> hipError_t {
    // rows [r0, r1) of B minus the contribution of the solved rows [k0, k0 + kb)
    if (r1 <= r0) return hipSuccess;
    Gemm g;
    g.M = r1 - r0; g.N = ncols; g.K = kb;
    g.B = B + k0 * ldb; g.ldb = ldb;
    g.C = B + r0 * ldb; g.ldc = ldb;
    g.alpha = -1.0; g.beta = 1.0;
    if (!trans) { g.A = L + r0 * ldl + k0; g.lda = ldl; }                     // L[r0:r1, k0:k0+kb]
    else { g.A = L + k0 * ldl + r0; g.lda = ldl; g.transA = true; }           // L[k0:k0+kb, r0:r1]^T
    return gemm_f64(g, s);
  };
  for (int64_t oq = 0; oq < nout; ++oq) {
    const int64_t ob = trans ? (nout - 1 - oq) : oq;
    const int64_t o0 = ob * NB2, o1 = (o0 + NB2 < n) ? o0 + NB2 : n;
    const int64_t nin = (o1 - o0) / NB;
    for (int64_t q = 0; q < nin; ++q) {
      const int64_t k0 = o0 + (trans ? (nin - 1 - q) : q) * NB;
      if (!trans)
        hipLaunchKernelGGL(tri64_kernel<false>, dim3(nblk(ncols, TRI)), dim3(256), 0, s,
                           L + k0 * ldl + k0, ldl, B + k0 * ldb, (int64_t)1, ldb, ncols);
      else
        hipLaunchKernelGGL(tri64_kernel<true>, dim3(nblk(ncols, TRI)), dim3(256), 0, s,
                           L + k0 * ldl + k0, ldl, B + k0 * ldb, (int64_t)1, ldb, ncols);
      const hipError_t e = trans ? update(o0, k0, k0, NB) : update(k0 + NB, o1, k0, NB);
      if (e != hipSuccess) return e;
    }
    const hipError_t e = trans ? update(0, o0, o0, o1 - o0) : update(o1, n, o0, o1 - o0);
    if (e != hipSuccess) return e;
  }
  return hipGetLastError();
}

int64_t pivoted_cholesky_work(int64_t n) { return n + 4 * ((n + 255) / 256); }

hipError_t pivoted_cholesky(double* G, int64_t n, int64_t ld, int64_t k, int64_t* piv,
                            double* Lbuf, double* work, hipStream_t s) {
  constexpr int64_t PB = PCP;
  if (n > INT32_MAX) return hipErrorInvalidValue;
  const bool one = n <= 1024;     // the candidates fit one workgroup
  PcArgs a{};
  a.n = n; a.k = k; a.nbmax = (n + 255) / 256;
  a.G = G; a.ld = ld; a.L = Lbuf; a.ldl = k; a.diag = work; a.piv = piv;
  a.bv = work + n;
  a.bi = reinterpret_cast<int32_t*>(work + n + 2 * a.nbmax);
  const dim3 grid((unsigned)a.nbmax, 1u);
  if (!one) hipLaunchKernelGGL(pchol_step_kernel<false>, grid, dim3(256), 0, s, a, (int64_t)-1, (int64_t)0);
  for (int64_t kb = 0; kb < k; kb += PB) {
    const int64_t ke = (kb + PB < k) ? kb + PB : k;
    if (one) {
      hipLaunchKernelGGL(pchol_panel_kernel, dim3(1), dim3(1024), 0, s, G, (int)n, ld, Lbuf, k, kb, (int)(ke - kb),
                         work, piv);
    } else {
      for (int64_t kk = kb; kk < ke; ++kk)
        hipLaunchKernelGGL(pchol_step_kernel<false>, grid, dim3(256), (size_t)PB * 8, s, a, kk, kb);
    }
    if (ke < k) {   // G -= L[:, kb:ke] L[:, kb:ke]^T
      Gemm g;
      g.M = n; g.N = n; g.K = ke - kb;
      g.A = Lbuf + kb; g.lda = k;
      g.B = Lbuf + kb; g.ldb = k; g.transB = true;
      g.C = G; g.ldc = ld; g.alpha = -1.0; g.beta = 1.0;
      hipError_t e = gemm_f64(g, s);
      if (e != hipSuccess) return e;
    }
  }
  return hipGetLastError();
}

hipError_t pivoted_cholesky_sets(const PcArgs& a, int nsets, int64_t kmax, hipStream_t s) {
  if (nsets <= 0 || kmax <= 0) return hipSuccess;
  if (nsets > 65535 || kmax + 2 * a.p > kPcSetsMax) return hipErrorInvalidValue;
  const dim3 grid((unsigned)a.nbmax, (unsigned)nsets);
  for (int64_t k = -1; k < kmax; ++k)
    hipLaunchKernelGGL(pchol_step_kernel<true>, grid, dim3(256), (size_t)(std::max<int64_t>(k, 0) + 2 * a.p) * 8, s, a,
                       k, (int64_t)0);
  return hipGetLastError();
}

}  // namespace rps
