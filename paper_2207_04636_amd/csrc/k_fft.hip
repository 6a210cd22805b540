// Coulomb potential of the fitting functions, V[g, :] = Vc chi_g (Sec. 3.2;
// the Coulomb operator is diagonal on the plane waves, Sec. 2.2 Eq. 7-8,
// with the G = 0 term removed, Sec. 4.5):
//     Vc f = IDFT( k(G) / N_g * DFT(f) ),  k(G) = 4 pi / |G|^2,  k(0) = 0.
//
// Two real rows f, h are transformed together as the complex row f + i h
// (split storage: the real parts stay in row 2c, the imaginary parts in row
// 2c + 1), which works because Vc is real: Vc(f + i h) = Vc f + i Vc h.
//
// The 3-D transform is separable: one pass per axis, each pass moving some pencils of
// one axis into LDS and applying the length-L transform there in FP64 (axes up to 256
// points): a self-sorting mixed-radix FFT (radices 4, 2, 3, 5) when L has no other prime
// factor, else the DFT by direct summation.  Passes:
// forward along axis 2, forward along axis 1, [forward along axis 0, multiply
// by k/N_g, inverse along axis 0] in one kernel, inverse along axis 1, inverse
// along axis 2.  The set-up transforms all fitting functions, the Coulomb build one row
// pair (the density).
//
// Bound by LDS traffic and latency, not by arithmetic, so a stage is compiled per radix
// (plain additions where the roots of unity are 1 and i), the pencil of a thread is fixed
// (one address computation per thread, no division per element), and the roots come from
// a table that the caller keeps.  The previous kernel took the radix, the pencil and the
// position of every element from run-time divisions and summed every butterfly over a
// table: 416 rows of 40^3 took 2.1 ms, the Coulomb build's pair of 48^3 49 us.
#include <math.h>

#include "mfma.h"
#include "rps_internal.h"

namespace rps {
namespace {

constexpr int LMAX = 256;    // longest supported axis

// y[o] = sum_r x[r] exp(sg 2 pi i r o / R), in place
template <int R>
__device__ __forceinline__ void butterfly(double (&xr)[R], double (&xi)[R], double sg) {
  if constexpr (R == 2) {
    const double ar = xr[0], ai = xi[0];
    xr[0] = ar + xr[1]; xi[0] = ai + xi[1];
    xr[1] = ar - xr[1]; xi[1] = ai - xi[1];
  } else if constexpr (R == 3) {
    const double tr = xr[1] + xr[2], ti = xi[1] + xi[2];
    const double h = sg * 0.86602540378443864676;          // sin(2 pi / 3)
    const double dr = h * (xr[1] - xr[2]), di = h * (xi[1] - xi[2]);
    const double mr = xr[0] - 0.5 * tr, mi = xi[0] - 0.5 * ti;
    xr[0] += tr; xi[0] += ti;
    xr[1] = mr - di; xi[1] = mi + dr;
    xr[2] = mr + di; xi[2] = mi - dr;
  } else if constexpr (R == 4) {
    const double ar = xr[0] + xr[2], ai = xi[0] + xi[2], br = xr[0] - xr[2], bi = xi[0] - xi[2];
    const double cr = xr[1] + xr[3], ci = xi[1] + xi[3];
    const double dr = sg * (xr[1] - xr[3]), di = sg * (xi[1] - xi[3]);
    xr[0] = ar + cr; xi[0] = ai + ci;
    xr[1] = br - di; xi[1] = bi + dr;
    xr[2] = ar - cr; xi[2] = ai - ci;
    xr[3] = br + di; xi[3] = bi - dr;
  } else {
    static_assert(R == 5, "radices 2, 3, 4, 5");
    constexpr double c1 = 0.30901699437494742410, c2 = -0.80901699437494742410;   // cos(2 pi / 5), cos(4 pi / 5)
    const double s1 = sg * 0.95105651629515357212, s2 = sg * 0.58778525229247312917;   // sin of the same
    const double ar = xr[1] + xr[4], ai = xi[1] + xi[4], br = xr[1] - xr[4], bi = xi[1] - xi[4];
    const double cr = xr[2] + xr[3], ci = xi[2] + xi[3], dr = xr[2] - xr[3], di = xi[2] - xi[3];
    const double pr = xr[0] + c1 * ar + c2 * cr, pi = xi[0] + c1 * ai + c2 * ci;
    const double qr = xr[0] + c2 * ar + c1 * cr, qi = xi[0] + c2 * ai + c1 * ci;
    const double ur = s1 * br + s2 * dr, ui = s1 * bi + s2 * di;
    const double vr = s2 * br - s1 * dr, vi = s2 * bi - s1 * di;
    xr[0] += ar + cr; xi[0] += ai + ci;
    xr[1] = pr - ui; xi[1] = pi + ur;
    xr[4] = pr + ui; xi[4] = pi - ur;
    xr[2] = qr - vi; xi[2] = qi + vr;
    xr[3] = qr + vi; xi[3] = qi - vr;
  }
}

// One Stockham stage of radix R after sub-transforms of length ns: butterfly j (< L / R)
// takes the R points j + r L / R, turns them by exp(sg 2 pi i r (j mod ns) / (ns R)),
// applies the R-point transform and writes point r' to (j / ns) ns R + (j mod ns) + r' ns.
// The elements of a pencil lie st apart.  wr, wi: exp(2 pi i m / L), ns R divides L.
template <int R>
__device__ __forceinline__ void stage_point(const double* sr, const double* si, double* dr, double* di, int st, int L,
                                            int ns, int j, const double* wr, const double* wi, double sg) {
  const int nb = L / R, ts = nb / ns;
  const int jd = (j * ((65536 + ns - 1) / ns)) >> 16;        // j / ns for j, ns <= 256
  const int k = j - jd * ns;
  double xr[R], xi[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    xr[r] = sr[(j + r * nb) * st];
    xi[r] = si[(j + r * nb) * st];
  }
  if (ns > 1) {
#pragma unroll
    for (int r = 1; r < R; ++r) {
      const double c = wr[r * k * ts], w = sg * wi[r * k * ts];
      const double a = xr[r], b = xi[r];
      xr[r] = a * c - b * w;
      xi[r] = a * w + b * c;
    }
  }
  butterfly<R>(xr, xi, sg);
  const int d0 = jd * ns * R + k;
#pragma unroll
  for (int o = 0; o < R; ++o) {
    dr[(d0 + o * ns) * st] = xr[o];
    di[(d0 + o * ns) * st] = xi[o];
  }
}

// A stage for the PEN pencils of an axis workgroup: thread t works on pencil t mod PEN.
template <int R, int PEN, int NT>
__device__ __forceinline__ void stage(const double* sr, const double* si, double* dr, double* di, int L, int ns,
                                      const double* wr, const double* wi, double sg, int tid) {
  for (int j = tid / PEN; j < L / R; j += NT / PEN) stage_point<R>(sr, si, dr, di, 1, L, ns, j, wr, wi, sg);
}

// A stage for npen pencils, sp apart, of a plane (elements st apart): consecutive threads
// take consecutive pencils.
template <int R, int NT>
__device__ __forceinline__ void plane_stage(const double* sr, const double* si, double* dr, double* di, int npen,
                                            int sp, int st, int L, int ns, const double* wr, const double* wi,
                                            double sg, int tid) {
  const int nb = L / R;
  const float rn = 1.0f / (float)npen;
  for (int e = tid; e < npen * nb; e += NT) {
    const int j = (int)(((float)e + 0.5f) * rn), o = (e - j * npen) * sp;
    stage_point<R>(sr + o, si + o, dr + o, di + o, st, L, ns, j, wr, wi, sg);
  }
}

__host__ __device__ __forceinline__ bool smooth235(int L) {
  while (L % 2 == 0) L /= 2;
  while (L % 3 == 0) L /= 3;
  while (L % 5 == 0) L /= 5;
  return L == 1;
}

// Both inner axes of one plane (L1 x L2, contiguous) of a row pair in LDS, forward (axis 2,
// then axis 1) or inverse (axis 1, then axis 2): three launches for a Poisson solve instead
// of five, and three passes over the rows.  A latency chain for the Coulomb build's one
// pair (48 planes of 48 x 48: two launches of 7 us became one), bandwidth for the set-up.
// LDS pitch L2 + 1 (or + 2 to make it odd) spreads rows and columns over the banks.
constexpr int PLANE_NT = 512;
__host__ __device__ __forceinline__ int plane_pitch(int L2) { return L2 | 1; }
inline size_t plane_lds(int L1, int L2) {
  return ((size_t)4 * L1 * plane_pitch(L2) + 2 * (L1 + L2)) * sizeof(double);
}
template <bool INV>
__global__ __launch_bounds__(PLANE_NT) void dft_plane_kernel(double* __restrict__ V, int64_t ld, int L1, int L2,
                                                            const double* __restrict__ tw1,
                                                            const double* __restrict__ tw2) {
  extern __shared__ double sm[];
  const int tid = threadIdx.x, P = plane_pitch(L2), n = L1 * L2, half = L1 * P;
  double* w1 = sm + 4 * half;            // cosines and sines of axis 1, then of axis 2
  double* w2 = w1 + 2 * L1;
  double* re = V + (int64_t)(2 * blockIdx.y) * ld + (int64_t)blockIdx.x * n;
  double* im = re + ld;
  const float r2 = 1.0f / (float)L2;
  for (int m = tid; m < 2 * L1; m += PLANE_NT) w1[m] = tw1[m];
  for (int m = tid; m < 2 * L2; m += PLANE_NT) w2[m] = tw2[m];
  for (int e = tid; e < n; e += PLANE_NT) {
    const int i = (int)(((float)e + 0.5f) * r2);
    sm[i * P + e - i * L2] = re[e];
    sm[half + i * P + e - i * L2] = im[e];
  }
  __syncthreads();
  const double sg = INV ? 1.0 : -1.0;
  int cur = 0;                           // buffer: re at 2 cur half, im at (2 cur + 1) half
#pragma unroll
  for (int pass = 0; pass < 2; ++pass) {
    const bool inner = INV ? (pass == 1) : (pass == 0);      // along axis 2
    const int L = inner ? L2 : L1, npen = inner ? L1 : L2, sp = inner ? P : 1, st = inner ? 1 : P;
    const double *wr = inner ? w2 : w1, *wi = wr + L;
    int ns = 1, left = L;
    while (left > 1) {
      const int R = (left % 4 == 0) ? 4 : (left % 2 == 0) ? 2 : (left % 3 == 0) ? 3 : 5;
      const double *sr = sm + 2 * cur * half, *si = sr + half;
      double *dr = sm + 2 * (cur ^ 1) * half, *di = dr + half;
      if (R == 4) plane_stage<4, PLANE_NT>(sr, si, dr, di, npen, sp, st, L, ns, wr, wi, sg, tid);
      else if (R == 2) plane_stage<2, PLANE_NT>(sr, si, dr, di, npen, sp, st, L, ns, wr, wi, sg, tid);
      else if (R == 3) plane_stage<3, PLANE_NT>(sr, si, dr, di, npen, sp, st, L, ns, wr, wi, sg, tid);
      else plane_stage<5, PLANE_NT>(sr, si, dr, di, npen, sp, st, L, ns, wr, wi, sg, tid);
      __syncthreads();
      cur ^= 1;
      ns *= R;
      left /= R;
    }
  }
  const double* out = sm + 2 * cur * half;
  for (int e = tid; e < n; e += PLANE_NT) {
    const int i = (int)(((float)e + 0.5f) * r2);
    re[e] = out[i * P + e - i * L2];
    im[e] = out[half + i * P + e - i * L2];
  }
}

// Pencil p (of outer*inner) starts at o*L*inner + i with o = p / inner, i = p % inner;
// element j of it is at start + j*inner.  PEN pencils and NT threads per workgroup: 16 and
// 256 for the set-up's many rows, 4 and 64 when a single row pair would leave most CUs
// idle.  LM is the longest axis the LDS arrays hold: 128, or 256 with at most 8 pencils.
// The LDS pitch LM + 64 / PEN puts the pencils' words of a wave on all banks alike.
// tw: exp(2 pi i m / L), m < L, as cosines then sines.
template <int MODE, int PEN, int NT, int LM>   // 0: forward, 1: inverse, 2: forward, multiply by kern, inverse
__global__ __launch_bounds__(NT) void dft_axis_kernel(double* __restrict__ V, int64_t ld, int L,
                                                      int64_t inner, int64_t npencil,
                                                      const double* __restrict__ kern,
                                                      const double* __restrict__ tw) {
  constexpr int PITCH = LM + 64 / PEN;
  __shared__ double br[2][PEN * PITCH], bi[2][PEN * PITCH];
  __shared__ double wr[LM], wi[LM];
  const int tid = threadIdx.x;
  double* re = V + (int64_t)(2 * blockIdx.y) * ld;
  double* im = re + ld;
  const int64_t p0 = (int64_t)blockIdx.x * PEN;
  const bool contiguous = (inner == 1);
  // this thread's pencil in the transform, and in the transfers of a strided axis
  const int q = tid % PEN, j0 = tid / PEN;
  const int64_t p = p0 + q;
  const int64_t at = (p / inner) * (int64_t)L * inner + p % inner;
  const bool live = p < npencil;
  const int nel = (int)((npencil - p0 < PEN) ? npencil - p0 : PEN) * L;    // elements of a contiguous axis
  const float rL = 1.0f / (float)L;
  for (int m = tid; m < L; m += NT) {
    wr[m] = tw[m];
    wi[m] = tw[L + m];
  }
  if (contiguous) {
    for (int e = tid; e < PEN * L; e += NT) {
      const int qq = (int)(((float)e + 0.5f) * rL), j = e - qq * L;
      br[0][qq * PITCH + j] = (e < nel) ? re[p0 * L + e] : 0.0;
      bi[0][qq * PITCH + j] = (e < nel) ? im[p0 * L + e] : 0.0;
    }
  } else {
    for (int j = j0; j < L; j += NT / PEN) {
      br[0][q * PITCH + j] = live ? re[at + j * inner] : 0.0;
      bi[0][q * PITCH + j] = live ? im[at + j * inner] : 0.0;
    }
  }
  __syncthreads();
  constexpr int PASSES = (MODE == 2) ? 2 : 1;
  int cur = 0;
  // lengths whose factors are all 2, 3 and 5 take the fast transform
  const bool fast = smooth235(L);
#pragma unroll
  for (int pass = 0; pass < PASSES; ++pass) {
    // out[k] = sum_j x[j] exp(sg * 2 pi i j k / L), sg = -1 forward, +1 inverse
    const double sg = (MODE == 1 || pass == 1) ? 1.0 : -1.0;
    if (fast) {
      int ns = 1, left = L;
      while (left > 1) {
        const int R = (left % 4 == 0) ? 4 : (left % 2 == 0) ? 2 : (left % 3 == 0) ? 3 : 5;
        const double *sr = &br[cur][q * PITCH], *si = &bi[cur][q * PITCH];
        double *dr = &br[cur ^ 1][q * PITCH], *di = &bi[cur ^ 1][q * PITCH];
        if (R == 4) stage<4, PEN, NT>(sr, si, dr, di, L, ns, wr, wi, sg, tid);
        else if (R == 2) stage<2, PEN, NT>(sr, si, dr, di, L, ns, wr, wi, sg, tid);
        else if (R == 3) stage<3, PEN, NT>(sr, si, dr, di, L, ns, wr, wi, sg, tid);
        else stage<5, PEN, NT>(sr, si, dr, di, L, ns, wr, wi, sg, tid);
        __syncthreads();
        cur ^= 1;
        ns *= R;
        left /= R;
      }
    } else {
      for (int k = j0; k < L; k += NT / PEN) {
        double sr = 0.0, si = 0.0;
        int m = 0;
        for (int j = 0; j < L; ++j) {
          const double c = wr[m], s = sg * wi[m];
          const double a = br[cur][q * PITCH + j], b = bi[cur][q * PITCH + j];
          sr += a * c - b * s;
          si += a * s + b * c;
          m += k;
          if (m >= L) m -= L;
        }
        br[cur ^ 1][q * PITCH + k] = sr;
        bi[cur ^ 1][q * PITCH + k] = si;
      }
      __syncthreads();
      cur ^= 1;
    }
    if (MODE == 2 && pass == 0) {
      for (int j = j0; j < L; j += NT / PEN) {
        const double kv = live ? kern[at + j * inner] : 0.0;
        br[cur][q * PITCH + j] *= kv;
        bi[cur][q * PITCH + j] *= kv;
      }
      __syncthreads();
    }
  }
  if (contiguous) {
    for (int e = tid; e < nel; e += NT) {
      const int qq = (int)(((float)e + 0.5f) * rL), j = e - qq * L;
      re[p0 * L + e] = br[cur][qq * PITCH + j];
      im[p0 * L + e] = bi[cur][qq * PITCH + j];
    }
  } else if (live) {
    for (int j = j0; j < L; j += NT / PEN) {
      re[at + j * inner] = br[cur][q * PITCH + j];
      im[at + j * inner] = bi[cur][q * PITCH + j];
    }
  }
}

template <int PEN, int NT, int LM>
void go(double* V, int64_t ld, int L, int64_t inner, int64_t np, const double* kern, const double* tw,
        int64_t npairs, int mode, hipStream_t s) {
  dim3 grid((unsigned)((np + PEN - 1) / PEN), (unsigned)npairs);
  if (mode == 0)
    hipLaunchKernelGGL((dft_axis_kernel<0, PEN, NT, LM>), grid, dim3(NT), 0, s, V, ld, L, inner, np, kern, tw);
  else if (mode == 1)
    hipLaunchKernelGGL((dft_axis_kernel<1, PEN, NT, LM>), grid, dim3(NT), 0, s, V, ld, L, inner, np, kern, tw);
  else
    hipLaunchKernelGGL((dft_axis_kernel<2, PEN, NT, LM>), grid, dim3(NT), 0, s, V, ld, L, inner, np, kern, tw);
}

}  // namespace

int64_t poisson_table_size(const int mesh[3]) {
  return (int64_t)mesh[0] * mesh[1] * mesh[2] + 2 * ((int64_t)mesh[0] + mesh[1] + mesh[2]);
}

void poisson_roots(const int mesh[3], double* out) {
  for (int a = 0; a < 3; ++a) {
    const int L = mesh[a];
    for (int m = 0; m < L; ++m) {
      const long double t = 2.0L * 3.14159265358979323846264338327950288L * m / L;
      out[m] = (double)cosl(t);
      out[L + m] = (double)sinl(t);
    }
    out += 2 * L;
  }
}

hipError_t poisson_rows(double* V, int64_t nrows, int64_t ld, const int mesh[3],
                        const double* kern, hipStream_t s) {
  if (nrows % 2 != 0) return hipErrorInvalidValue;
  for (int a = 0; a < 3; ++a)
    if (mesh[a] > LMAX || mesh[a] < 1) return hipErrorInvalidValue;
  const int64_t ng = (int64_t)mesh[0] * mesh[1] * mesh[2];
  const int64_t npairs = nrows / 2;
  const int64_t inner[3] = {(int64_t)mesh[1] * mesh[2], (int64_t)mesh[2], 1};
  const double* tw[3] = {kern + ng, kern + ng + 2 * mesh[0], kern + ng + 2 * (mesh[0] + mesh[1])};
  // grid.y <= 65535 pairs per launch
  for (int64_t c0 = 0; c0 < npairs; c0 += 65535) {
    const int64_t cn = (npairs - c0 < 65535) ? npairs - c0 : 65535;
    double* Vc = V + 2 * c0 * ld;
    auto launch = [&](int axis, int mode) {
      const int L = mesh[axis];
      const int64_t np = ng / L;
      if (L > 128) {
        go<8, 256, 256>(Vc, ld, L, inner[axis], np, kern, tw[axis], cn, mode, s);
      } else if ((np + 15) / 16 * cn >= 1024) {
        go<16, 256, 128>(Vc, ld, L, inner[axis], np, kern, tw[axis], cn, mode, s);
      } else {
        go<4, 64, 128>(Vc, ld, L, inner[axis], np, kern, tw[axis], cn, mode, s);
      }
    };
    // a plane of up to about 5000 points fits in LDS; the direct sum of other lengths stays
    // with the axis kernel
    const size_t lds = plane_lds(mesh[1], mesh[2]);
    if (lds <= 160 * 1024 && smooth235(mesh[1]) && smooth235(mesh[2])) {
      const dim3 grid((unsigned)mesh[0], (unsigned)cn);
      hipError_t e = hipFuncSetAttribute((const void*)dft_plane_kernel<false>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
      if (e == hipSuccess)
        e = hipFuncSetAttribute((const void*)dft_plane_kernel<true>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
      if (e != hipSuccess) return e;
      hipLaunchKernelGGL(dft_plane_kernel<false>, grid, dim3(PLANE_NT), lds, s, Vc, ld, mesh[1], mesh[2], tw[1], tw[2]);
      launch(0, 2);
      hipLaunchKernelGGL(dft_plane_kernel<true>, grid, dim3(PLANE_NT), lds, s, Vc, ld, mesh[1], mesh[2], tw[1], tw[2]);
    } else {
      launch(2, 0);
      launch(1, 0);
      launch(0, 2);
      launch(1, 1);
      launch(2, 1);
    }
  }
  return hipGetLastError();
}

}  // namespace rps
