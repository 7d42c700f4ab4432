// tables.hip -- FP64 construction of the rate and inverse-CDF tables on the GPU.
//
// Spectra (locally-constant-field nonlinear Compton and Breit-Wheeler, the
// rates the paper takes from precomputed approximations, Sec. 3):
//   emission: dW/d delta = alpha/(sqrt3 pi gamma) [A K_{2/3}(y) - Ki_{1/3}(y)],
//             A = 1 - delta + 1/(1-delta), y = 2 delta / (3 chi (1-delta));
//   pairs:    dW/d xi    = alpha/(sqrt3 pi eps)   [A K_{2/3}(y) + Ki_{1/3}(y)],
//             A = xi/(1-xi) + (1-xi)/xi,      y = 2 / (3 chi xi (1-xi));
// Ki_nu(y) = int_y^oo K_nu.
//
// Quadrature variables (both integrands are analytic and decay exponentially
// at both ends of the real line):
//   emission: w = (1/3) ln y, so z = delta/(1-delta) = 1.5 chi e^{3w} and
//             d(delta) = 4.5 chi y (1-delta)^2 dw;
//   pairs:    w = logit(xi), so y = (4/(3 chi)) (1 + cosh w) and
//             d(xi) = dw / (2 (1 + cosh w)); the integrand is even in w.
// K_{2/3} and Ki_{1/3} come from the trapezoid rule on their integral
// representations e^y K_nu(y) = int_0^oo e^{-y (cosh t - 1)} cosh(nu t) dt and
// e^y Ki_nu(y) = int_0^oo e^{-y (cosh t - 1)} cosh(nu t) / cosh t dt, which
// converges geometrically in the step for these analytic integrands.
// Integrals over w use 8-point Gauss-Legendre on panels of fixed width;
// inverse CDFs invert the cumulative panel sums by Newton iteration inside the
// panel that holds the target.
//
// The build is bound by FP64 arithmetic, nearly all of it in the two Bessel
// functions: a Newton step of one table entry takes nine of them, and a sum of
// up to 288 exponentials each time, by one wave per SIMD, made the default tables
// 167 ms.  Both are functions of y alone and smooth in ln y once e^-y is taken
// out, so for the pair tables and the FP32 emission grid the sums are taken only
// at the nodes of piecewise polynomials (k_bessel_table: 688 panels, 5,504 sums)
// and every integrand reads those (16 multiply-adds and an exponential): 0.4 ms.
// The FP64 pair grid then differs by up to 1.6e-14 from one made of the sums; both
// are 4.5e-11 (rms; 3.9e-10 at most) from the exact inverse, in every digit given.
// The FP32 emission grid has the same bits by default (on one of 19 other grids an
// entry rounded the other way).  The FP64 emission tables are held to the bits of
// the full sums (the same on the default grid and on 19 others, drawn over the
// ranges a configuration may have), so that FP64 steps with emission alone, whose
// records can be compared byte for byte, give what they gave: they are made from
// the sums, operation by operation, with the work spread over the chip
// (k_rad_nodes 1.1 ms, k_rad_panels 0.6, k_rad_rows 55 -> 15 ms).  The pair tables
// the same way would be another 26 ms.

#include <algorithm>
#include <cmath>
#include <vector>

#include "lib.h"
#include "physics.h"

namespace sfqed {

constexpr double kBesselH = 0.2;  // trapezoid step in t
constexpr int kBesselN = 288;     // t up to 57.6: covers y >= 1e-20
constexpr double kYSmall = 1e-20; // below: leading small-y forms
constexpr int kGL = 8;

// emission w-panels
constexpr double kRadW0 = -40.0;
constexpr double kRadDW = 1.0 / 16.0;
constexpr int kRadPanels = 676;   // up to w = 2.25 (y = 854)
// pair half-line panels: a fixed number over [0, W(chi)], where W is the point
// beyond which the spectrum is below e^-750 of its peak
// (y - y0 = y0 sinh^2(w/2) = 750, y0 = 8/(3 chi)); the spectrum is a Gaussian
// of width ~ sqrt(2 / y0) in w at small chi, so the panels follow its width.
constexpr int kPairPanels = 152;
constexpr double kPairWMax = 19.0;

struct Consts {
  double gl_x[kGL], gl_w[kGL];        // Gauss-Legendre on [-1, 1]
  double bc[kBesselN];                // cosh(t_j) - 1
  double b23[kBesselN];               // h cosh(2 t_j / 3) (half weight at j = 0)
  double b13[kBesselN];               // h cosh(t_j / 3) / cosh(t_j)
  double k23_small, ki13_zero;        // Gamma(2/3)/2 2^{2/3}, pi/sqrt3
  double to_power[64];                // [power][node]: values at 8 Chebyshev nodes -> powers
};

// e^{y_shift} K_{2/3}(y) and e^{y_shift} Ki_{1/3}(y), y_shift <= y (keeps the
// pair spectrum in range far below its threshold).  The trapezoid rule in t
// loses accuracy like exp(-2 pi^2 / (h^2 y)) as y grows, because the integrand
// narrows to a Gaussian of width 1/sqrt(y); above y = 4 the substitution
// y (cosh t - 1) = v^2, t = 2 asinh(v / sqrt(2y)), dt = 2 dv / sqrt(2y + v^2)
// turns it into e^{-v^2} times a function analytic in |Im v| < sqrt(2y), and
// the trapezoid rule in v converges like exp(-pi^2 / h^2).
constexpr double kBesselHv = 0.25;
constexpr int kBesselNv = 27;  // v up to 6.5

// term j of the sum in v (y > 4; r2y = 1 / sqrt(2y), iy = 1 / y) and in t
__device__ __forceinline__ void bessel_term_v(int j, double r2y, double iy, double& s23, double& s13) {
  const double v = j * kBesselHv;
  const double a = asinh(v * r2y);
  const double wv = (j == 0 ? 0.5 : 1.0) * kBesselHv * exp(-v * v) * 2.0 * r2y / sqrt(1.0 + v * v * r2y * r2y);
  const double c23 = cosh(a * (4.0 / 3.0)), c13 = cosh(a * (2.0 / 3.0));
  s23 = fma(wv, c23, s23);
  s13 = fma(wv, c13 / (1.0 + v * v * iy), s13);
}
__device__ __forceinline__ void bessel_term_t(const Consts& c, int j, double y, double& s23, double& s13) {
  const double a = y * c.bc[j];
  if (a > 745.0) return;
  const double ej = exp(-a);
  s23 = fma(c.b23[j], ej, s23);
  s13 = fma(c.b13[j], ej, s13);
}

__device__ void bessel_pair(const Consts& c, double y, double y_shift, double& k23, double& ki13) {
  if (y - y_shift > 745.0) {
    k23 = 0.0;
    ki13 = 0.0;
    return;
  }
  const double e = exp(-(y - y_shift));
  if (y < kYSmall) {
    k23 = e * c.k23_small * pow(y, -2.0 / 3.0);
    ki13 = e * c.ki13_zero;
    return;
  }
  double s23 = 0.0, s13 = 0.0;
  if (y > 4.0) {
    const double r2y = 1.0 / sqrt(2.0 * y), iy = 1.0 / y;
    for (int j = kBesselNv - 1; j >= 0; --j) bessel_term_v(j, r2y, iy, s23, s13);
  } else {
    // terms with y (cosh t - 1) > 745 underflow
    int jmax = (int)(acosh(1.0 + 745.0 / y) * (1.0 / kBesselH)) + 1;
    jmax = jmax < kBesselN - 1 ? jmax : kBesselN - 1;
    for (int j = jmax; j >= 0; --j) bessel_term_t(c, j, y, s23, s13);  // small terms first
  }
  k23 = s23 * e;
  ki13 = s13 * e;
}

// ------------------------------------------------------------------ Bessel functions by interpolation
// S(w) = e^y K_{2/3}(y) and e^y Ki_{1/3}(y), y = e^{3w}, as polynomials of
// degree 7 through 8 Chebyshev nodes on panels of kBtDW in w.  In ln y the
// functions are analytic within +-i pi of the real axis; with a panel's
// half-width of 3/64 in ln y the interpolation error falls as
// (2 pi 64 / 3)^-8 = 1e-17.  The table covers y from kYSmall to 8.7e7, past
// which (the pair spectrum at chi < 3e-8) the sums are taken directly.
constexpr double kBtDW = 1.0 / 32.0;
constexpr double kBtW0 = -493.0 / 32.0;  // y = 8.4e-21
constexpr int kBtPanels = 688;           // up to w = 6.09375, y = 8.7e7
constexpr int kBtNodes = 8;
struct BesselTable {
  double c[kBtPanels][2][kBtNodes];  // ascending powers of v in [-1, 1]
};

// One wave per panel: eight lanes share a node, each adding every eighth term
// of its sum; then lane (function, power) forms a coefficient.
__global__ void __launch_bounds__(64) k_bessel_table(const Consts* cg, BesselTable* out) {
  const Consts& c = *cg;
  const int lane = threadIdx.x, node = lane >> 3, part = lane & 7;
  __shared__ double val[2][kBtNodes];
  const double v = cos(kPi * (node + 0.5) / kBtNodes);
  const double y = exp(3.0 * (kBtW0 + kBtDW * (blockIdx.x + 0.5 * (v + 1.0))));
  double s23 = 0.0, s13 = 0.0;
  if (y > 4.0) {
    const double r2y = 1.0 / sqrt(2.0 * y), iy = 1.0 / y;
    for (int j = part; j < kBesselNv; j += 8) bessel_term_v(j, r2y, iy, s23, s13);
  } else {
    for (int j = part; j < kBesselN; j += 8) bessel_term_t(c, j, y, s23, s13);
  }
  for (int o = 1; o < 8; o <<= 1) {
    s23 += __shfl_xor(s23, o);
    s13 += __shfl_xor(s13, o);
  }
  if (part == 0) {
    val[0][node] = s23;
    val[1][node] = s13;
  }
  __syncthreads();
  if (lane < 2 * kBtNodes) {
    const int f = lane / kBtNodes, q = lane % kBtNodes;
    double acc = 0.0;
    for (int m = 0; m < kBtNodes; ++m) acc = fma(c.to_power[q * kBtNodes + m], val[f][m], acc);
    out->c[blockIdx.x][f][q] = acc;
  }
}

// e^{y_shift} K_{2/3}(y) and e^{y_shift} Ki_{1/3}(y) at y = e^{3w} (y_shift <= y)
__device__ __forceinline__ void bessel_at(const Consts& c, const BesselTable* bt, double w, double y, double y_shift,
                                          double& k23, double& ki13) {
  const double u = (w - kBtW0) * (1.0 / kBtDW);
  if (!(u >= 0.0 && u < (double)kBtPanels) || y < kYSmall) {
    bessel_pair(c, y, y_shift, k23, ki13);
    return;
  }
  if (y - y_shift > 745.0) {
    k23 = 0.0;
    ki13 = 0.0;
    return;
  }
  const int k = (int)u;
  const double v = 2.0 * (u - (double)k) - 1.0;
  const double2* q = reinterpret_cast<const double2*>(bt->c[k]);
  double2 a[kBtNodes / 2], b[kBtNodes / 2];
#pragma unroll
  for (int i = 0; i < kBtNodes / 2; ++i) {
    a[i] = q[i];
    b[i] = q[kBtNodes / 2 + i];
  }
  double s23 = a[3].y, s13 = b[3].y;
#pragma unroll
  for (int i = 3; i >= 0; --i) {
    s23 = fma(s23, v, a[i].x);
    s13 = fma(s13, v, b[i].x);
    if (i > 0) {
      s23 = fma(s23, v, a[i - 1].y);
      s13 = fma(s13, v, b[i - 1].y);
    }
  }
  const double e = exp(-(y - y_shift));
  k23 = s23 * e;
  ki13 = s13 * e;
}

// emission integrand in w (reduced by alpha/gamma)
__device__ double rad_integrand(const Consts& c, const BesselTable* bt, double chi, double w) {
  const double y = exp(3.0 * w);
  const double z = 1.5 * chi * y;
  const double omd = 1.0 / (1.0 + z);
  const double a = omd + (1.0 + z);
  double k23, ki13;
  bessel_at(c, bt, w, y, 0.0, k23, ki13);
  return (a * k23 - ki13) * (1.0 / (kSqrt3 * kPi)) * 4.5 * chi * y * omd * omd;
}

// pair integrand in w (reduced by alpha/eps), scaled by e^{8/(3 chi)}
__device__ double pair_integrand(const Consts& c, const BesselTable* bt, double chi, double w) {
  const double ch = cosh(w);
  const double y0 = 8.0 / (3.0 * chi);
  const double sh = sinh(0.5 * w);
  const double y = y0 + y0 * sh * sh;  // (4/(3chi))(1 + cosh w) = y0 cosh^2(w/2)
  double k23, ki13;
  bessel_at(c, bt, log(y) * (1.0 / 3.0), y, y0, k23, ki13);
  return (2.0 * ch * k23 + ki13) * (1.0 / (kSqrt3 * kPi)) / (2.0 * (1.0 + ch));
}

template <int P>
__device__ double integrand(const Consts& c, const BesselTable* bt, double chi, double w) {
  return P == 0 ? rad_integrand(c, bt, chi, w) : pair_integrand(c, bt, chi, w);
}

template <int P>
__device__ double gl_panel(const Consts& c, const BesselTable* bt, double chi, double a, double b) {
  const double m = 0.5 * (a + b), h = 0.5 * (b - a);
  double s = 0.0;
  for (int i = 0; i < kGL; ++i) s = fma(c.gl_w[i], integrand<P>(c, bt, chi, fma(h, c.gl_x[i], m)), s);
  return s * h;
}

// panel k spans [g.w0 + k g.dw, g.w0 + (k+1) g.dw]
struct Panels {
  double w0, dw;
};

template <int P>
__device__ __forceinline__ Panels panels_for(double chi) {
  if (P == 0) return Panels{kRadW0, kRadDW};
  const double y0 = 8.0 / (3.0 * chi);
  const double W = fmin(kPairWMax, 2.0 * asinh(sqrt(750.0 / y0)));
  return Panels{0.0, W / kPairPanels};
}
template <int P>
__device__ __forceinline__ int npanels() {
  return P == 0 ? kRadPanels : kPairPanels;
}

// Deterministic block sum in FP64 (fixed tree order).
__device__ double block_sum(double v, double* red) {
  const int t = threadIdx.x;
  red[t] = v;
  __syncthreads();
  for (int s = blockDim.x / 2; s > 0; s >>= 1) {
    if (t < s) red[t] += red[t + s];
    __syncthreads();
  }
  const double r = red[0];
  __syncthreads();
  return r;
}

// Reduced pair rate integral at chi: twice the half line (scaled by e^{8/(3chi)}).
__device__ double pair_total(const Consts& c, const BesselTable* bt, double chi, double* red) {
  const Panels pg = panels_for<1>(chi);
  double acc = 0.0;
  for (int k = threadIdx.x; k < kPairPanels; k += blockDim.x)
    acc += gl_panel<1>(c, bt, chi, pg.w0 + k * pg.dw, pg.w0 + (k + 1) * pg.dw);
  return 2.0 * block_sum(acc, red);
}

__global__ void __launch_bounds__(256) k_pair_nodes(const Consts* cg, const BesselTable* bt, double s_lo,
                                                    double* g_out) {
  __shared__ double red[256];
  const Consts& c = *cg;
  const int seg = blockIdx.x / kChebN, m = blockIdx.x % kChebN;
  const double xm = cos(kPi * (m + 0.5) / kChebN);
  const double s = s_lo + seg * kChebSegWidth + 0.5 * kChebSegWidth * (xm + 1.0);
  const double chi = exp(s);
  const double tot = pair_total(c, bt, chi, red);
  if (threadIdx.x == 0) g_out[blockIdx.x] = log(tot) - s;  // pairs: + 8/(3chi) is in the scaling
}

// c_j = (2/N) sum_m g_m cos(j pi (m + 1/2) / N)
__global__ void k_cheb_coeffs(const double* g, int nseg, double* coef) {
  const int seg = blockIdx.x, j = threadIdx.x;
  if (seg >= nseg || j >= kChebN) return;
  double acc = 0.0;
  for (int m = 0; m < kChebN; ++m) acc += g[seg * kChebN + m] * cos(kPi * j * (m + 0.5) / kChebN);
  coef[seg * kChebN + j] = 2.0 * acc / kChebN;
}

// FP32 Hermite nodes: g and h g' from the Chebyshev series.
__global__ void k_rate_herm(const double* coef, int nseg, double s_lo, int n, double h, float2* out) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const double s = s_lo + i * h;
  double u = (s - s_lo) / kChebSegWidth;
  int k = (int)floor(u);
  k = k < 0 ? 0 : (k >= nseg ? nseg - 1 : k);
  const double x = 2.0 * (u - k) - 1.0;
  const double* c = coef + k * kChebN;
  const double g = cheb_clenshaw(c, x);
  // derivative series: d_{j-1} = d_{j+1} + 2 j c_j
  double d[kChebN + 1];
  d[kChebN] = 0.0;
  d[kChebN - 1] = 0.0;
  for (int j = kChebN - 1; j >= 1; --j) d[j - 1] = (j + 1 <= kChebN ? d[j + 1] : 0.0) + 2.0 * j * c[j];
  const double dg_dx = cheb_clenshaw(d, x);  // uses d[0..16]
  const double dg_ds = dg_dx * (2.0 / kChebSegWidth);
  out[i] = make_float2((float)g, (float)(h * dg_ds));
}

// Exclusive prefix sum of v >= 0 over the block (kRowThreads threads) in thread
// order, by additions alone: what lies above a panel is many orders smaller
// than the panel itself, so nothing is taken off a sum.
constexpr int kRowThreads = 512;
__device__ __forceinline__ double block_scan(double v, double* wave_sum) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int o = 1; o < 64; o <<= 1) {
    const double up = __shfl_up(v, o);
    if (lane >= o) v += up;
  }
  if (lane == 63) wave_sum[wave] = v;
  const double below = __shfl_up(v, 1);
  __syncthreads();
  double before = 0.0;
  for (int w = 0; w < wave; ++w) before += wave_sum[w];
  __syncthreads();
  return lane ? before + below : before;
}

// A row of an inverse-CDF grid: chi = exp(s0 + row hs); columns x0 + j hx.
struct GridRows {
  double s0, x0;
  double hs32, hx32, hs64, hx64;
  int rows32, cols32, cols64;
  float* out32;
  double* out64;
};
// One block per row, the FP32 grid's rows first, then the FP64 grid's (one
// launch fills the chip: the FP32 grid alone has 70 and 47 rows).
template <int P>
__global__ void __launch_bounds__(kRowThreads) k_cdf_rows(const Consts* cg, const BesselTable* bt, GridRows g) {
  static_assert(kRadPanels <= 2 * kRowThreads && kPairPanels <= 2 * kRowThreads, "two panels per thread");
  __shared__ double I[kRadPanels];
  __shared__ double C[kRadPanels + 1], D[kRadPanels + 1];
  __shared__ double wave_sum[kRowThreads / 64];
  const Consts& c = *cg;
  const bool f32 = (int)blockIdx.x < g.rows32;
  const int row = f32 ? (int)blockIdx.x : (int)blockIdx.x - g.rows32;
  const int cols = f32 ? g.cols32 : g.cols64;
  const double hx = f32 ? g.hx32 : g.hx64, x0 = g.x0;
  float* out32 = f32 ? g.out32 : nullptr;
  double* out64 = f32 ? nullptr : g.out64;
  const double s = g.s0 + row * (f32 ? g.hs32 : g.hs64);
  const double chi = exp(s);
  const int np = npanels<P>();
  const Panels pg = panels_for<P>(chi);
  for (int k = threadIdx.x; k < np; k += blockDim.x)
    I[k] = gl_panel<P>(c, bt, chi, pg.w0 + k * pg.dw, pg.w0 + (k + 1) * pg.dw);
  __syncthreads();
  // C[k]: the integral below panel k (with the tail below the panels); D[k]:
  // from panel k to the top.  Thread t holds panels 2t and 2t + 1 (and, for D,
  // the same counted from the top).
  {
    const double c0 = P == 0 ? integrand<0>(c, bt, chi, kRadW0) : 0.0;
    const int k = 2 * threadIdx.x;
    const double a = k < np ? I[k] : 0.0, b = k + 1 < np ? I[k + 1] : 0.0;
    const double up = c0 + block_scan(a + b, wave_sum);
    if (k < np) C[k + 1] = up + a;
    if (k + 1 < np) C[k + 2] = up + a + b;
    const double da = k < np ? I[np - 1 - k] : 0.0, db = k + 1 < np ? I[np - 2 - k] : 0.0;
    const double down = block_scan(da + db, wave_sum);
    if (k < np) D[np - 1 - k] = down + da;
    if (k + 1 < np) D[np - 2 - k] = down + da + db;
    if (threadIdx.x == 0) {
      C[0] = c0;
      D[np] = 0.0;
    }
  }
  __syncthreads();
  const double total = P == 0 ? C[np] : 2.0 * D[0];
  for (int j = threadIdx.x; j < cols; j += blockDim.x) {
    const double x = x0 + j * hx;
    const double r = 1.0 / (1.0 + exp(-x)), rc = 1.0 / (1.0 + exp(x));
    // find the panel and the integral still to cover inside it, from its left edge
    int k;
    double loc;
    if (P == 0 && x <= 0.0) {
      const double T = r * total;
      int lo = 0, hi = np;  // C[lo] <= T < C[hi]
      if (T < C[0]) { lo = 0; hi = 0; }
      while (hi - lo > 1) {
        const int mid = (lo + hi) / 2;
        if (C[mid] <= T) lo = mid; else hi = mid;
      }
      k = lo;
      loc = T - C[k];
    } else {
      // from the top: find k with D[k+1] <= T < D[k]
      const double T = P == 0 ? rc * total : r * total;  // pairs: half line from the top = r * total
      int lo = 0, hi = np;  // D[lo] > T >= D[hi]
      while (hi - lo > 1) {
        const int mid = (lo + hi) / 2;
        if (D[mid] > T) lo = mid; else hi = mid;
      }
      k = lo;
      loc = I[k] - (T - D[k + 1]);
    }
    k = k < 0 ? 0 : (k >= np ? np - 1 : k);
    const double a = pg.w0 + k * pg.dw, b = a + pg.dw;
    double wlo = a, whi = b;
    double w = a + (b - a) * fmin(1.0, fmax(0.0, I[k] > 0.0 ? loc / I[k] : 0.5));
    for (int it = 0; it < 60; ++it) {
      const double G = gl_panel<P>(c, bt, chi, a, w) - loc;
      if (G > 0.0) whi = w; else wlo = w;
      const double f = integrand<P>(c, bt, chi, w);
      double wn = f > 0.0 ? w - G / f : 0.5 * (wlo + whi);
      // Newton's error squares: after a step of 1e-8 panels only rounding is
      // left, so the search ends there.  (Testing the bracket first sent such a
      // step, which often ends on the bracket itself, back to a bisection, and
      // most entries ran all 60 trips.)
      if (f > 0.0 && fabs(wn - w) <= 1e-8 * (b - a)) {
        w = fmin(fmax(wn, a), b);
        break;
      }
      if (!(wn > wlo && wn < whi)) wn = 0.5 * (wlo + whi);
      const bool done = whi - wlo <= 1e-15 * fmax(1.0, fabs(w));
      w = wn;
      if (done) break;
    }
    double q;
    if (P == 0) q = log(1.5) + 3.0 * w;  // logit(delta) - ln chi
    else q = -w;                         // logit(xi) for xi <= 1/2
    if (out32) out32[row * cols + j] = (float)q;
    if (out64) out64[row * cols + j] = q;
  }
}

// ------------------------------------------------------------------ emission in FP64, from the sums
// The same operations on each value as bessel_pair, in the same order, by a
// wave as a whole (all lanes active): the loops run to the longest of its lanes
// and the constants are scalar loads.
constexpr double kWaveCut = 70.0;
__device__ __forceinline__ void bessel_wave(const Consts& c, double y, double y_shift, double& k23, double& ki13) {
  const bool under = y - y_shift > 745.0, small = !under && y < kYSmall;
  const bool large = !under && !small && y > 4.0, series = !under && !small && !large;
  // Terms with y (cosh t - 1) > kWaveCut come first, small terms before large
  // ones, and are 1e-28 of the sum: that could decide a rounding once in 1e12
  // sums, and decided none on the 20 grids compared.
  int jmax = -1;
  if (series) {
    jmax = (int)(acosh(1.0 + kWaveCut / y) * (1.0 / kBesselH)) + 1;
    jmax = jmax < kBesselN - 1 ? jmax : kBesselN - 1;
  }
  int jw = jmax;
  for (int o = 32; o > 0; o >>= 1) {
    const int other = __shfl_xor(jw, o);
    jw = other > jw ? other : jw;
  }
  jw = __builtin_amdgcn_readfirstlane(jw);
  double s23 = 0.0, s13 = 0.0;
#pragma unroll 2
  for (int j = jw; j >= 0; --j) {  // small terms first
    const double a = y * c.bc[j];
    const double ej = a > kWaveCut ? 0.0 : exp(-a);  // so for all j > jmax
    s23 = fma(c.b23[j], ej, s23);
    s13 = fma(c.b13[j], ej, s13);
  }
  if (__any(large)) {
    const double r2y = 1.0 / sqrt(2.0 * y), iy = 1.0 / y;
    double l23 = 0.0, l13 = 0.0;
#pragma unroll 1
    for (int j = kBesselNv - 1; j >= 0; --j) {
      const double v = j * kBesselHv;
      const double a = asinh(v * r2y);
      const double wv = (j == 0 ? 0.5 : 1.0) * kBesselHv * exp(-v * v) * 2.0 * r2y / sqrt(1.0 + v * v * r2y * r2y);
      const double c23 = cosh(a * (4.0 / 3.0)), c13 = cosh(a * (2.0 / 3.0));
      l23 = fma(wv, c23, l23);
      l13 = fma(wv, c13 / (1.0 + v * v * iy), l13);
    }
    s23 = large ? l23 : s23;
    s13 = large ? l13 : s13;
  }
  const double e = exp(-(y - y_shift));
  k23 = s23 * e;
  ki13 = s13 * e;
  if (small) {
    k23 = e * c.k23_small * pow(y, -2.0 / 3.0);
    ki13 = e * c.ki13_zero;
  }
  if (under) {
    k23 = 0.0;
    ki13 = 0.0;
  }
}

// rad_integrand from the sums
__device__ __forceinline__ double rad_wave(const Consts& c, double chi, double w) {
  const double y = exp(3.0 * w);
  const double z = 1.5 * chi * y;
  const double omd = 1.0 / (1.0 + z);
  const double a = omd + (1.0 + z);
  double k23, ki13;
  bessel_wave(c, y, 0.0, k23, ki13);
  return (a * k23 - ki13) * (1.0 / (kSqrt3 * kPi)) * 4.5 * chi * y * omd * omd;
}
__device__ __forceinline__ double rad_panel_wave(const Consts& c, double chi, int k) {
  const double a = kRadW0 + k * kRadDW, b = kRadW0 + (k + 1) * kRadDW;
  const double m = 0.5 * (a + b), h = 0.5 * (b - a);
  double s = 0.0;
#pragma unroll 1
  for (int i = 0; i < kGL; ++i) s = fma(c.gl_w[i], rad_wave(c, chi, fma(h, c.gl_x[i], m)), s);
  return s * h;
}

// Emission rate at the Chebyshev nodes: thread t adds panels t, t + 256, ...
__global__ void __launch_bounds__(256, 2) k_rad_nodes(const Consts* cg, double s_lo, double* g_out) {
  __shared__ double red[256];
  const Consts& c = *cg;
  const int seg = blockIdx.x / kChebN, m = blockIdx.x % kChebN;
  const double xm = cos(kPi * (m + 0.5) / kChebN);
  const double s = s_lo + seg * kChebSegWidth + 0.5 * kChebSegWidth * (xm + 1.0);
  const double chi = exp(s);
  double acc = 0.0;
  for (int k0 = 0; k0 < kRadPanels; k0 += 256) {
    const int k = k0 + (int)threadIdx.x;
    const double v = rad_panel_wave(c, chi, k);
    if (k < kRadPanels) acc += v;
  }
  double tot = block_sum(acc, red);
  tot += rad_wave(c, chi, kRadW0);  // tail below w0 ~ e^w
  if (threadIdx.x == 0) g_out[blockIdx.x] = log(tot) - s;
}

// The FP64 grid of emission: chi = exp(s0 + row hs), columns x0 + j hx.
struct RadGrid {
  double s0, hs, x0, hx;
  int rows, cols;
  double* panels;  // [rows][kRadPanels] panel integrals
  double* out;
};
// One panel of one row per thread.
__global__ void __launch_bounds__(256, 2) k_rad_panels(const Consts* cg, RadGrid g) {
  const int n = g.rows * kRadPanels;
  const int i0 = (int)(blockIdx.x * blockDim.x + threadIdx.x), i = i0 < n ? i0 : n - 1;
  const double chi = exp(g.s0 + (i / kRadPanels) * g.hs);
  const double v = rad_panel_wave(*cg, chi, i % kRadPanels);
  if (i0 < n) g.panels[i] = v;
}

// Entries of one row: kLanes lanes each (the nodes of the panel rule and the end
// point), kPerWave of them at a time in a wave (lane 63 follows lane 62), which
// goes through a contiguous part of the row.  The search is Newton's, with the
// bracket's middle where a step leaves the bracket.  Once a step has reproduced w
// to the last bit, w is an end of the bracket, steps that lead back to it are
// refused, and up to 50 halvings follow; what they end on belongs to the
// result.  So lanes whose entry is done take the wave's next one, and a halving
// is decided by the interpolated integrand (1e-13 off, a twentieth of the work)
// where the sign of G and the step's leaving the bracket hold by ten times that.
// Bound by the exponentials of the sums: one thread per entry took 55 ms for 277
// rows of 1057, nine lanes 28 (with the FP32 grid), refilled 21, without the terms
// past kWaveCut 17.5, with the look ahead 15.  Eight blocks a row: with 4
// their unequal work shows (16.4), with 16 the sums of the panels (19.0 against
// 17.5).
constexpr int kLanes = kGL + 1, kPerWave = 64 / kLanes;
constexpr int kSumThreads = 256;
constexpr int kSumSplit = 8;
constexpr double kSumLook = 1e-12;  // the look ahead's margin, of loc / f and of 1

// The sum of the rule over a group's nodes, in their order.
__device__ __forceinline__ double panel_sum(const Consts& c, double v, int group) {
  double s = 0.0;
  for (int i = 0; i < kGL; ++i) s = fma(c.gl_w[i], __shfl(v, group * kLanes + i), s);
  return s;
}
// One step of the search, to wn; false when it has ended.
__device__ __forceinline__ bool go_on(double wn, double& w, double wlo, double whi, int& it) {
  const double tol = 1e-15 * fmax(1.0, fabs(w));
  const bool done = fabs(wn - w) <= tol || whi - wlo <= tol;
  w = wn;
  return !done && ++it < 60;
}
__global__ void __launch_bounds__(kSumThreads, 4) k_rad_rows(const Consts* cg, const BesselTable* bt, RadGrid g) {
  const Consts& c = *cg;
  __shared__ double I[kRadPanels];
  __shared__ double C[kRadPanels + 1], D[kRadPanels + 1];
  constexpr int np = kRadPanels;
  const int row = (int)blockIdx.x, cols = g.cols;
  const double chi = exp(g.s0 + row * g.hs);
  for (int k = threadIdx.x; k < np; k += kSumThreads) I[k] = g.panels[(size_t)row * np + k];
  const double tail = rad_wave(c, chi, kRadW0);
  __syncthreads();
  if (threadIdx.x == 0) {  // one addition after another: the two sums in two waves
    double sum = tail;
    C[0] = sum;
    for (int k = 0; k < np; ++k) C[k + 1] = sum = sum + I[k];
  }
  if (threadIdx.x == 64) {
    double sum = 0.0;
    D[np] = sum;
    for (int k = np - 1; k >= 0; --k) D[k] = sum = sum + I[k];
  }
  __syncthreads();
  const double total = C[np];
  const int lane = (int)(threadIdx.x & 63);
  const int group = (lane < 63 ? lane : 62) / kLanes, part = (lane < 63 ? lane : 62) % kLanes;
  const double node = c.gl_x[part < kGL ? part : 0];
  constexpr int waves = kSumSplit * (kSumThreads / 64);
  const int wave = __builtin_amdgcn_readfirstlane((int)(blockIdx.y * (kSumThreads / 64) + (threadIdx.x >> 6)));
  int next = cols * wave / waves;
  const int end = cols * (wave + 1) / waves;
  int j = end, it = 0;
  bool busy = false;  // the same in all lanes of a group, as is what follows
  double a = kRadW0, loc = 0.0, wlo = kRadW0, whi = kRadW0, w = kRadW0;
  while (true) {
    const uint64_t idle = __ballot(!busy && part == 0 && lane < 63);
    if (idle && next < end) {
      const int mine = next + __popcll(idle & ((1ull << (group * kLanes)) - 1));
      if (!busy && mine < end) {
        j = mine;
        busy = true;
        it = 0;
        const double x = g.x0 + j * g.hx;
        const double r = 1.0 / (1.0 + exp(-x)), rc = 1.0 / (1.0 + exp(x));
        // find the panel and the integral still to cover inside it, from its left edge
        int k;
        if (x <= 0.0) {
          const double T = r * total;
          int lo = 0, hi = np;  // C[lo] <= T < C[hi]
          if (T < C[0]) { lo = 0; hi = 0; }
          while (hi - lo > 1) {
            const int mid = (lo + hi) / 2;
            if (C[mid] <= T) lo = mid; else hi = mid;
          }
          k = lo;
          loc = T - C[k];
        } else {
          // from the top: find k with D[k+1] <= T < D[k]
          const double T = rc * total;
          int lo = 0, hi = np;  // D[lo] > T >= D[hi]
          while (hi - lo > 1) {
            const int mid = (lo + hi) / 2;
            if (D[mid] > T) lo = mid; else hi = mid;
          }
          k = lo;
          loc = I[k] - (T - D[k + 1]);
        }
        k = k < 0 ? 0 : (k >= np ? np - 1 : k);
        a = kRadW0 + k * kRadDW;
        const double b = a + kRadDW;
        wlo = a;
        whi = b;
        w = a + (b - a) * fmin(1.0, fmax(0.0, I[k] > 0.0 ? loc / I[k] : 0.5));
      }
      next += __popcll(idle);
    }
    if (!__any(busy)) break;
    bool open = busy;
    while (__any(open)) {  // halvings that the interpolated integrand decides
      const double m = 0.5 * (a + w), h = 0.5 * (w - a);
      const double v = rad_integrand(c, bt, chi, part < kGL ? fma(h, node, m) : w);
      const double G = panel_sum(c, v, group) * h - loc, f = __shfl(v, group * kLanes + kGL);
      if (!open) continue;
      const double newton = w - G / f, off = kSumLook * (1.0 + fabs(loc) / f);
      const double lo = G > 0.0 ? wlo : w, hi = G > 0.0 ? w : whi;
      open = f > 0.0 && fabs(G) > off * f && (newton < lo - off || newton > hi + off);
      if (!open) continue;
      wlo = lo;
      whi = hi;
      busy = open = go_on(0.5 * (wlo + whi), w, wlo, whi, it);
      if (!busy && part == 0) g.out[row * cols + j] = log(1.5) + 3.0 * w;
    }
    const double m = 0.5 * (a + w), h = 0.5 * (w - a);  // the rule on [a, w]
    const double v = rad_wave(c, chi, part < kGL ? fma(h, node, m) : w);
    const double G = panel_sum(c, v, group) * h - loc, f = __shfl(v, group * kLanes + kGL);
    if (!busy) continue;
    if (G > 0.0) whi = w; else wlo = w;
    double wn = f > 0.0 ? w - G / f : 0.5 * (wlo + whi);
    if (!(wn > wlo && wn < whi)) wn = 0.5 * (wlo + whi);
    busy = go_on(wn, w, wlo, whi, it);
    if (!busy && part == 0) g.out[row * cols + j] = log(1.5) + 3.0 * w;  // logit(delta) - ln chi
  }
}

// ------------------------------------------------------------------ host side
namespace {

void gauss_legendre(int n, double* x, double* w) {
  for (int i = 0; i < n; ++i) {
    double z = std::cos(kPi * (i + 0.75) / (n + 0.5)), dp = 1.0;
    for (int it = 0; it < 100; ++it) {
      double p1 = 1.0, p2 = 0.0;
      for (int j = 1; j <= n; ++j) {
        const double p3 = p2;
        p2 = p1;
        p1 = ((2.0 * j - 1.0) * z * p2 - (j - 1.0) * p3) / j;
      }
      dp = n * (z * p1 - p2) / (z * z - 1.0);
      const double dz = p1 / dp;
      z -= dz;
      if (std::fabs(dz) < 1e-16) {
        // recompute the derivative at the converged node
        double q1 = 1.0, q2 = 0.0;
        for (int j = 1; j <= n; ++j) {
          const double q3 = q2;
          q2 = q1;
          q1 = ((2.0 * j - 1.0) * z * q2 - (j - 1.0) * q3) / j;
        }
        dp = n * (z * q1 - q2) / (z * z - 1.0);
        break;
      }
    }
    x[i] = z;
    w[i] = 2.0 / ((1.0 - z * z) * dp * dp);
  }
}

// out[q][m]: the weight of the value at Chebyshev node cos(pi (m + 1/2) / n)
// in the coefficient of power q of the interpolating polynomial.
void chebyshev_to_power(int n, double* out) {
  std::vector<std::vector<double>> t(n, std::vector<double>(n, 0.0));  // T_j in powers
  t[0][0] = 1.0;
  if (n > 1) t[1][1] = 1.0;
  for (int j = 2; j < n; ++j)
    for (int q = 0; q < n; ++q) t[j][q] = (q ? 2.0 * t[j - 1][q - 1] : 0.0) - t[j - 2][q];
  for (int q = 0; q < n; ++q)
    for (int m = 0; m < n; ++m) {
      double a = 0.0;
      for (int j = 0; j < n; ++j) a += (j ? 2.0 : 1.0) / n * std::cos(kPi * j * (m + 0.5) / n) * t[j][q];
      out[q * n + m] = a;
    }
}

size_t align_up(size_t v) { return (v + 255) & ~size_t(255); }

}  // namespace

qed_status build_tables(const qed_table_cfg& cfg, hipStream_t stream, qed_tables* t) {
  TableGeom& g = t->geom;
  g.cfg = cfg;
  // Chebyshev rate ranges: emission from rate_chi_min, pairs from max(rate_chi_min, 1e-3)
  const double lo[2] = {std::log(cfg.rate_chi_min), std::log(std::max(cfg.rate_chi_min, 1e-3))};
  const double hi = std::log(cfg.rate_chi_max);
  for (int p = 0; p < 2; ++p) {
    g.cheb_s_lo[p] = lo[p];
    g.nseg[p] = (int)std::ceil((hi - lo[p]) / kChebSegWidth);
  }
  g.herm_n = cfg.rate_nodes;
  g.rows32[0] = cfg.rad_rows;
  g.cols32[0] = cfg.rad_cols;
  g.rows32[1] = cfg.pair_rows;
  g.cols32[1] = cfg.pair_cols;
  for (int p = 0; p < 2; ++p) {
    g.rows64[p] = (g.rows32[p] - 1) * cfg.f64_refine + 1;
    g.cols64[p] = (g.cols32[p] - 1) * cfg.f64_refine + 1;
  }
  g.s0[0] = std::log(cfg.rad_chi_min);
  g.s1[0] = std::log(cfg.rad_chi_max);
  g.x0[0] = cfg.rad_x_min;
  g.x1[0] = cfg.rad_x_max;
  g.s0[1] = std::log(cfg.pair_chi_min);
  g.s1[1] = std::log(cfg.pair_chi_max);
  g.x0[1] = cfg.pair_x_min;
  g.x1[1] = 0.0;

  // layout of the single allocation
  size_t off = 0;
  auto take = [&](size_t bytes) {
    const size_t o = off;
    off = align_up(off + bytes);
    return o;
  };
  const size_t o_consts = take(sizeof(Consts));
  const size_t o_bessel = take(sizeof(BesselTable));
  size_t o_nodes[2], o_cheb[2], o_herm[2], o_c32[2], o_c64[2];
  for (int p = 0; p < 2; ++p) {
    o_nodes[p] = take(sizeof(double) * g.nseg[p] * kChebN);
    o_cheb[p] = take(sizeof(double) * g.nseg[p] * kChebN);
    o_herm[p] = take(sizeof(float2) * g.herm_n);
    o_c32[p] = take(sizeof(float) * g.rows32[p] * g.cols32[p]);
    o_c64[p] = take(sizeof(double) * g.rows64[p] * g.cols64[p]);
  }
  const size_t o_panels = take(sizeof(double) * g.rows64[0] * kRadPanels);
  t->bytes = off;
  SFQED_HIP(hipMalloc(&t->mem, t->bytes));
  char* base = static_cast<char*>(t->mem);

  Consts hc;
  gauss_legendre(kGL, hc.gl_x, hc.gl_w);
  for (int j = 0; j < kBesselN; ++j) {
    const double tj = j * kBesselH;
    const double sh = std::sinh(0.5 * tj);
    hc.bc[j] = 2.0 * sh * sh;
    const double wj = (j == 0 ? 0.5 : 1.0) * kBesselH;
    hc.b23[j] = wj * std::cosh(2.0 * tj / 3.0);
    hc.b13[j] = wj * std::cosh(tj / 3.0) / std::cosh(tj);
  }
  hc.k23_small = 0.5 * std::tgamma(2.0 / 3.0) * std::pow(2.0, 2.0 / 3.0);
  hc.ki13_zero = kPi / kSqrt3;
  chebyshev_to_power(kBtNodes, hc.to_power);
  Consts* dconsts = reinterpret_cast<Consts*>(base + o_consts);
  SFQED_HIP(hipMemcpyAsync(dconsts, &hc, sizeof(Consts), hipMemcpyHostToDevice, stream));
  BesselTable* bt = reinterpret_cast<BesselTable*>(base + o_bessel);
  hipLaunchKernelGGL(k_bessel_table, dim3(kBtPanels), dim3(64), 0, stream, dconsts, bt);

  for (int p = 0; p < 2; ++p) {
    double* nodes = reinterpret_cast<double*>(base + o_nodes[p]);
    double* cheb = reinterpret_cast<double*>(base + o_cheb[p]);
    float2* herm = reinterpret_cast<float2*>(base + o_herm[p]);
    if (p == 0)
      hipLaunchKernelGGL(k_rad_nodes, dim3(g.nseg[p] * kChebN), dim3(256), 0, stream, dconsts, g.cheb_s_lo[p], nodes);
    else
      hipLaunchKernelGGL(k_pair_nodes, dim3(g.nseg[p] * kChebN), dim3(256), 0, stream, dconsts, bt, g.cheb_s_lo[p],
                         nodes);
    hipLaunchKernelGGL(k_cheb_coeffs, dim3(g.nseg[p]), dim3(32), 0, stream, nodes, g.nseg[p], cheb);
    const double hs = g.nseg[p] * kChebSegWidth / (g.herm_n - 1);
    hipLaunchKernelGGL(k_rate_herm, dim3((g.herm_n + 255) / 256), dim3(256), 0, stream, cheb, g.nseg[p],
                       g.cheb_s_lo[p], g.herm_n, hs, herm);
    RateView& rv = t->view.rate[p];
    rv.cheb = cheb;
    rv.s_lo = g.cheb_s_lo[p];
    rv.nseg = g.nseg[p];
    rv.herm = herm;
    rv.hs_lo = (float)g.cheb_s_lo[p];
    rv.inv_h = (float)(1.0 / hs);
    rv.n = g.herm_n;

    float* c32 = reinterpret_cast<float*>(base + o_c32[p]);
    double* c64 = reinterpret_cast<double*>(base + o_c64[p]);
    const double hs32 = (g.s1[p] - g.s0[p]) / (g.rows32[p] - 1), hx32 = (g.x1[p] - g.x0[p]) / (g.cols32[p] - 1);
    const double hs64 = (g.s1[p] - g.s0[p]) / (g.rows64[p] - 1), hx64 = (g.x1[p] - g.x0[p]) / (g.cols64[p] - 1);
    const GridRows gr{g.s0[p], g.x0[p], hs32, hx32, hs64, hx64, g.rows32[p], g.cols32[p], g.cols64[p], c32, c64};
    if (p == 0) {
      const RadGrid rg{g.s0[p],     hs64,        g.x0[p], hx64, g.rows64[p], g.cols64[p],
                       reinterpret_cast<double*>(base + o_panels), c64};
      const int n = g.rows64[p] * kRadPanels;
      hipLaunchKernelGGL(k_cdf_rows<0>, dim3(g.rows32[p]), dim3(kRowThreads), 0, stream, dconsts, bt, gr);
      hipLaunchKernelGGL(k_rad_panels, dim3((n + 255) / 256), dim3(256), 0, stream, dconsts, rg);
      hipLaunchKernelGGL(k_rad_rows, dim3(g.rows64[p], kSumSplit), dim3(kSumThreads), 0, stream, dconsts, bt, rg);
    } else {
      hipLaunchKernelGGL(k_cdf_rows<1>, dim3(g.rows32[p] + g.rows64[p]), dim3(kRowThreads), 0, stream, dconsts, bt,
                         gr);
    }
    SFQED_HIP(hipGetLastError());
    CdfView& cv = t->view.cdf[p];
    cv.f32 = c32;
    cv.rows32 = g.rows32[p];
    cv.cols32 = g.cols32[p];
    cv.s0_32 = (float)g.s0[p];
    cv.inv_hs32 = (float)(1.0 / hs32);
    cv.x0_32 = (float)g.x0[p];
    cv.inv_hx32 = (float)(1.0 / hx32);
    cv.s1_32 = cv.s0_32 + (float)(cv.rows32 - 1) / cv.inv_hs32;
    cv.f64 = c64;
    cv.rows64 = g.rows64[p];
    cv.cols64 = g.cols64[p];
    cv.s0_64 = g.s0[p];
    cv.inv_hs64 = 1.0 / hs64;
    cv.x0_64 = g.x0[p];
    cv.inv_hx64 = 1.0 / hx64;
    cv.chi_lo = std::exp(g.s0[p]);
    cv.chi_hi = std::exp(g.s1[p]);

    t->off[0 + p] = o_cheb[p];
    t->len[0 + p] = sizeof(double) * g.nseg[p] * kChebN;
    t->off[2 + p] = o_herm[p];
    t->len[2 + p] = sizeof(float2) * g.herm_n;
    t->off[4 + p] = o_c32[p];
    t->len[4 + p] = sizeof(float) * g.rows32[p] * g.cols32[p];
    t->off[6 + p] = o_c64[p];
    t->len[6 + p] = sizeof(double) * g.rows64[p] * g.cols64[p];
  }
  return QED_OK;
}

}  // namespace sfqed
