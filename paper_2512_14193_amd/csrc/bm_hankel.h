// Device evaluation of H0^(1), H1^(1), J0, J1 (principal branch), FP64, at the
// arguments z = k r of an assembly: one wavenumber k, real r > 0, in the sector
// |arg z| <= 1/2 + small margin (wavenumbers with Re k > 0, |Im k| <= Re k / 2).
//
//   |z| < 3         power series (DLMF 10.2.2, 10.8.1): J from its Taylor series,
//                   Y0 and Y1 from the logarithmic series with harmonic numbers.
//   real z >= 3     the normalised function F_nu(1/z) of
//                   H_nu = sqrt(2/(pi z)) e^{i(z - nu pi/2 - pi/4)} F_nu, from its
//                   Chebyshev series in t = 1/z on [0, 1/3] (degree 26, generated
//                   from 40-digit values by gen_hankel_cheb.py): about one ulp.
//   complex z, |z| >= 3   the same on the ray: with k = |k| e^{i th}, F_nu is a smooth
//                   function of the real t = 1/|z|, so a small kernel (hankel_ray_kernel)
//                   forms, per wavenumber, the Chebyshev series of F_nu - 1 for H^(1)
//                   and for H^(2)(z) = conj(H^(1)(conj z)), J = (H^(1) + H^(2))/2, from
//                   the Laplace-type integral (the integral behind the asymptotic
//                   expansion, DLMF 10.17)
//                     F_nu = 1 / Gamma(nu + 1/2) int_0^inf e^{-u} u^{nu-1/2} (1 + iu/(2z))^{nu-1/2} du,
//                   u = s^2, trapezoid rule; its nearest singularity sits at s^2 = 2iz.
//                   Likewise the power series is then a polynomial in the real r^2.
//
// Assembly at complex wavenumbers, N = 1024: 80 us, against 372 us with two 32-node
// integrals per pair and wavenumber; the wide domain at N = 4000: 389 against 786 us.
// The loops keep a few coefficients of each series at a time (scalar loads) and are not
// unrolled whole, which takes the assembly from 248 registers and one wavefront per SIMD
// to 148 and three: real wavenumbers N = 2048 275 -> 106 us, N = 8192 4.09 -> 1.45 ms.
// The blocks' error against long double values is that of the integral or smaller
// (2e-16 to 5e-15 of a block over the sector and below it).
//
// Wide domain: wavenumbers in the lower half plane beyond the sector
// (Im k < -Re k / 2), where the complex resonances and fictitious eigenvalues of
// Sec. 5.3 lie.  There the singularity s^2 = 2iz of the integral approaches the
// integration path, so the power series is used instead, for |z| < 6 with 26 terms
// (the last term is below 1e-26 of the largest); in the lower half plane J and Y grow
// like H^(1), so the series loses at most a factor e^{|z| - |Im z|} <= 30 to
// cancellation.  Larger |z| is outside the supported domain: the caller flags it.
// Up to BM_WIDE_LOCAL_MAX_N nodes each workgroup of the assembly makes the tables of the
// series for itself, in LDS, about 2 us of each: the kernel that makes them once takes
// 11 us (17 before the factorials became compile-time constants), and its tables arrive
// cold.  Assembly with tables made by each workgroup and made
// once (both formulations alike): N = 128 25 and 41 us, 512 30 and 46, 1024 51 and 62,
// 1200 62 and 69, 1400 74 and 78, 1600 88 and 88, 2048 134 and 125, 4000 478 and 390 (LDS
// reads, which the scalar loads spare).
#pragma once

#include "bm_internal.h"

#include "bm_hankel_cheb.h"

struct bm_hk4 {
  cplx h0, h1, j0, j1;
};

// Factors of the series of real arguments: term k to k + 1 of J0 and of J1 / (z/2), and
// the harmonic sums H_k and H_k + H_{k+1}.  (Tables, so that the loops need not be
// unrolled whole: the assembly then runs with half the registers.)
#define HK_NR 18
struct hk_series_tab {
  double r[HK_NR][4];
};
constexpr hk_series_tab hk_series_make() {
  hk_series_tab t{};
  double hk = 0.0, hk1 = 1.0;
  for (int k = 0; k < HK_NR; ++k) {
    t.r[k][0] = 1.0 / ((k + 1.0) * (k + 1.0));
    t.r[k][1] = 1.0 / ((k + 1.0) * (k + 2.0));
    t.r[k][2] = hk;
    t.r[k][3] = hk + hk1;
    hk = hk1;
    hk1 += 1.0 / (k + 2.0);
  }
  return t;
}
__constant__ hk_series_tab hk_series = hk_series_make();

__device__ inline void bm_hankel_series(double x, bm_hk4 &o) {
  const cplx z = cmk(x, 0.0);
  const double mw = -0.25 * (x * x);  // -z^2/4
  double t0 = 1.0, t1 = 1.0, sj0 = 1.0, sj1 = 1.0, sy0 = 0.0, sy1 = 1.0;
#pragma unroll 3
  for (int k = 0; k + 1 < HK_NR; ++k) {
    const double x0 = t0 * mw, x1 = t1 * mw;
    sj0 = fma(x0, hk_series.r[k][0], sj0);
    sj1 = fma(x1, hk_series.r[k][1], sj1);
    t0 = x0 * hk_series.r[k][0];
    t1 = x1 * hk_series.r[k][1];
    sy0 = fma(t0, hk_series.r[k + 1][2], sy0);
    sy1 = fma(t1, hk_series.r[k + 1][3], sy1);
  }
  const cplx zh = cscale(z, 0.5);
  const cplx J0 = cmk(sj0, 0.0), J1 = cmul(zh, cmk(sj1, 0.0));
  cplx L = clog_d(zh);
  L.x += BM_EULER;
  const cplx Y0 = cscale(csub(cmul(L, J0), cmk(sy0, 0.0)), 2.0 / BM_PI);
  const cplx Y1 = cadd(cadd(cscale(crecip(z), -2.0 / BM_PI), cscale(cmul(L, J1), 2.0 / BM_PI)),
                       cscale(cmul(zh, cmk(sy1, 0.0)), -1.0 / BM_PI));
  o.j0 = J0;
  o.j1 = J1;
  o.h0 = cmk(J0.x - Y0.y, J0.y + Y0.x);
  o.h1 = cmk(J1.x - Y1.y, J1.y + Y1.x);
}

// H^(1)_0, H^(1)_1, J0, J1 at real x >= 3 from the Chebyshev series of F_0, F_1
// (Clenshaw's recurrence in u = 6/x - 1; the coefficients are the same for every
// lane, so they come from the scalar cache).
__device__ inline void bm_hankel_real(double x, bm_hk4 &o) {
  const double t = 1.0 / x;
  const double u = 6.0 * t - 1.0, u2 = 2.0 * u;
  double b1[4] = {0.0, 0.0, 0.0, 0.0}, b2[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 2
  for (int j = BM_HC_DEG; j >= 1; --j) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const double bn = fma(u2, b1[q], bm_hc[j][q] - b2[q]);
      b2[q] = b1[q];
      b1[q] = bn;
    }
  }
  double f[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) f[q] = fma(u, b1[q], bm_hc[0][q] - b2[q]);
  double sn, cs;
  sincos(x, &sn, &cs);
  // sqrt(2/(pi x)) e^{i(x - pi/4)} = sqrt(1/(pi x)) ((cos x + sin x) + i (sin x - cos x))
  const double a = sqrt(t / BM_PI);
  const cplx e = cmk(a * (cs + sn), a * (sn - cs));
  o.h0 = cmul(e, cmk(f[0], f[1]));
  o.h1 = cmul(cmk(e.y, -e.x), cmk(f[2], f[3]));  // extra e^{-i pi/2}
  o.j0 = cmk(o.h0.x, 0.0);
  o.j1 = cmk(o.h1.x, 0.0);
}

// H^(1)_0, H^(1)_1, J0, J1 at real x > 0
__device__ inline bm_hk4 bm_hankel01_real(double x) {
  bm_hk4 o;
  if (x * x < 9.0)
    bm_hankel_series(x, o);
  else
    bm_hankel_real(x, o);
  return o;
}

// How the Hankel values of an assembly are evaluated
enum {
  BM_DOM_SECTOR,      // wavenumbers in the sector
  BM_DOM_WIDE,        // the wide domain, tables made once
  BM_DOM_WIDE_LOCAL,  // the wide domain, tables made by each workgroup
};
#define BM_WIDE_LOCAL_MAX_N 1200
#define BM_WIDE_ZMAX 6.0  // largest |z| of the wide domain

// Tables of one wavenumber k = ak e^{i th}; every lane reads the same entries, so those
// made once (hankel_ray_kernel) come through the scalar cache.
#define HK_NS 26          // series terms (18 for |z| < 3)
#define HK_NC 28          // Chebyshev coefficients (those of degree 24 and beyond are below 1e-16)
struct hk_wave {
  double ak, th;   // |k|, arg k
  cplx k, ik;      // k, 1/k
  double scale, pad;    // the power of two P with P <= |k| < 2 P
  double ser[HK_NS][8];  // J0, J1 / (z/2), and the harmonic sums of Y0, Y1: coefficients in (P r)^2
};
struct hk_ray {
  hk_wave w;
  cplx sq1, sq2;          // sqrt(2/pi) e^{-i th/2 -+ i pi/4}
  double cheb[HK_NC][8];  // F_0 - 1, F_1 - 1 of H^(1) and of H^(2), in u = 6/|z| - 1
};
#define HK_RAY_DOUBLES (sizeof(hk_ray) / sizeof(double))

// The power series (NT terms) at r, az = |k| r.  W: the hk_wave, in constant memory or LDS
template <int NT, class W>
__device__ inline bm_hk4 hk_series_at(W T, double r, double rinv, double az) {
  bm_hk4 o;
  const double xr = T->scale * r, x = xr * xr;
  double s[8];
#pragma unroll
  for (int q = 0; q < 8; ++q) s[q] = T->ser[NT - 1][q];
#pragma unroll 2
  for (int m = NT - 2; m >= 0; --m)
#pragma unroll
    for (int q = 0; q < 8; ++q) s[q] = fma(s[q], x, T->ser[m][q]);
  const cplx zh = cmk(0.5 * T->k.x * r, 0.5 * T->k.y * r), zi = cmk(T->ik.x * rinv, T->ik.y * rinv);
  const cplx J0 = cmk(s[0], s[1]), J1 = cmul(zh, cmk(s[2], s[3]));
  const cplx L = cmk(log(0.5 * az) + BM_EULER, T->th);
  const cplx Y0 = cscale(csub(cmul(L, J0), cmk(s[4], s[5])), 2.0 / BM_PI);
  const cplx Y1 = cadd(cadd(cscale(zi, -2.0 / BM_PI), cscale(cmul(L, J1), 2.0 / BM_PI)),
                       cscale(cmul(zh, cmk(s[6], s[7])), -1.0 / BM_PI));
  o.j0 = J0;
  o.j1 = J1;
  o.h0 = cmk(J0.x - Y0.y, J0.y + Y0.x);
  o.h1 = cmk(J1.x - Y1.y, J1.y + Y1.x);
  return o;
}

// The wide domain; *bad is set when |z| >= BM_WIDE_ZMAX.
template <class W>
__device__ inline bm_hk4 bm_hankel01_wide(W T, double r, double rinv, bool *bad) {
  const double az = T->ak * r;
  if (!(az < BM_WIDE_ZMAX)) *bad = true;
  return hk_series_at<HK_NS>(T, r, rinv, az);
}

// The sector, from the tables made once
__device__ inline bm_hk4 bm_hankel01_ray(const hk_ray *T_, double r, double rinv) {
  typedef const __attribute__((address_space(4))) hk_ray *ray_ptr;  // (constant: scalar loads)
  const ray_ptr T = (ray_ptr)T_;
  const double az = T->w.ak * r;
  if (az < 3.0) return hk_series_at<18>(&T->w, r, rinv, az);
  bm_hk4 o;
  const double t = 1.0 / az, u = 6.0 * t - 1.0, u2 = 2.0 * u;
  double b1[8], b2[8];
#pragma unroll
  for (int q = 0; q < 8; ++q) b1[q] = b2[q] = 0.0;
#pragma unroll 3
  for (int j = HK_NC - 1; j >= 1; --j)
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const double bn = fma(u2, b1[q], T->cheb[j][q] - b2[q]);
      b2[q] = b1[q];
      b1[q] = bn;
    }
  double d[8];
#pragma unroll
  for (int q = 0; q < 8; ++q) d[q] = fma(u, b1[q], T->cheb[0][q] - b2[q]);
  double sn, cs;
  sincos(T->w.k.x * r, &sn, &cs);
  const double e1 = exp(-T->w.k.y * r), a = sqrt(t), a1 = a * e1, a2 = a / e1;
  const cplx p1 = cmul(cmk(T->sq1.x, T->sq1.y), cmk(a1 * cs, a1 * sn));
  const cplx p2 = cmul(cmk(T->sq2.x, T->sq2.y), cmk(a2 * cs, -a2 * sn));
  o.h0 = cadd(p1, cmul(p1, cmk(d[0], d[1])));
  const cplx h1 = cadd(p1, cmul(p1, cmk(d[2], d[3])));
  const cplx g0 = cadd(p2, cmul(p2, cmk(d[4], d[5])));
  const cplx g1 = cadd(p2, cmul(p2, cmk(d[6], d[7])));
  o.h1 = cmk(h1.y, -h1.x);                      // e^{-i pi/2}
  o.j0 = cscale(cadd(o.h0, g0), 0.5);
  o.j1 = cscale(cadd(o.h1, cmk(-g1.y, g1.x)), 0.5);  // e^{+i pi/2}
  return o;
}

// Sums and products to twice double precision, for the series' coefficients: rounded
// once, they leave the evaluation as exact as the recurrence of the terms was.
struct hk_dd {
  double h, l;
};
__device__ inline hk_dd dd_sum(double a, double b) {
  const double s = a + b, t = s - a;
  return {s, (a - (s - t)) + (b - t)};
}
__device__ inline hk_dd dd_add(hk_dd a, hk_dd b) {
  const hk_dd s = dd_sum(a.h, b.h);
  return dd_sum(s.h, s.l + (a.l + b.l));
}
__device__ inline hk_dd dd_mul(hk_dd a, hk_dd b) {
  const double p = a.h * b.h;
  return dd_sum(p, fma(a.h, b.h, -p) + (a.h * b.l + a.l * b.h));
}
struct hk_ddc {
  hk_dd x, y;
};
__device__ inline hk_ddc ddc_mul(hk_ddc a, hk_ddc b) {
  const hk_dd yy = dd_mul(a.y, b.y);
  return {dd_add(dd_mul(a.x, b.x), {-yy.h, -yy.l}), dd_add(dd_mul(a.x, b.y), dd_mul(a.y, b.x))};
}

// The factors of the series' coefficients, in the same precision: 1 / (m!)^2,
// 1 / (m! (m + 1)!), and these times the harmonic sums H_m and H_m + H_{m+1} (at compile
// time, where a product is split instead of fused).
struct hk_fact_tab {
  hk_dd r[HK_NS][4];
};
constexpr hk_dd ct_sum(double a, double b) {
  const double s = a + b, t = s - a;
  return {s, (a - (s - t)) + (b - t)};
}
constexpr hk_dd ct_prod(double a, double b) {
  const double ca = 134217729.0 * a, ah = ca - (ca - a), al = a - ah;
  const double cb = 134217729.0 * b, bh = cb - (cb - b), bl = b - bh;
  const double p = a * b;
  return {p, ((ah * bh - p) + ah * bl + al * bh) + al * bl};
}
constexpr hk_dd ct_add(hk_dd a, hk_dd b) {
  const hk_dd s = ct_sum(a.h, b.h);
  return ct_sum(s.h, s.l + (a.l + b.l));
}
constexpr hk_dd ct_mul(hk_dd a, hk_dd b) {
  const hk_dd p = ct_prod(a.h, b.h);
  return ct_sum(p.h, p.l + (a.h * b.l + a.l * b.h));
}
constexpr hk_dd ct_div(hk_dd a, double d) {  // d exact
  const double q = a.h / d;
  const hk_dd p = ct_prod(q, d);
  return ct_sum(q, (((a.h - p.h) - p.l) + a.l) / d);
}
constexpr hk_fact_tab hk_fact_make() {
  hk_fact_tab t{};
  hk_dd f = {1.0, 0.0}, h = {0.0, 0.0};
  for (int m = 0; m < HK_NS; ++m) {
    if (m > 0) {
      f = ct_div(f, (double)m * m);
      h = ct_add(h, ct_div({1.0, 0.0}, m));
    }
    t.r[m][0] = f;
    t.r[m][1] = ct_div(f, m + 1.0);
    t.r[m][2] = ct_mul(f, h);
    t.r[m][3] = ct_mul(t.r[m][1], ct_add(ct_add(h, h), ct_div({1.0, 0.0}, m + 1.0)));
  }
  return t;
}
__constant__ hk_fact_tab hk_fact = hk_fact_make();

// Item i of the tables of wavenumber k: term i of the series, or, for i = HK_NS, the rest.
__device__ inline void hk_wave_item(cplx k, int i, hk_wave *T) {
  // 1 / P for P = 2^floor(log2 |k|)
  const double ak = hypot(k.x, k.y), sc = __hiloint2double(0x7fe00000 - (__double2hiint(ak) & 0x7ff00000), 0);
  if (i < HK_NS) {
    // (-k^2 / 4 P^2)^i and its companions
    const double x = k.x * sc, y = k.y * sc;  // k / P, exact
    const hk_dd xx = dd_mul({x, 0.0}, {-0.25 * x, 0.0}), yy = dd_mul({y, 0.0}, {0.25 * y, 0.0});
    hk_ddc f = {dd_add(xx, yy), dd_mul({x, 0.0}, {-0.5 * y, 0.0})}, c = {{1.0, 0.0}, {0.0, 0.0}};
    for (int e = i; e > 0; e >>= 1) {
      if (e & 1) c = ddc_mul(c, f);
      f = ddc_mul(f, f);
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const hk_dd a = hk_fact.r[i][q];
      T->ser[i][2 * q] = dd_mul(c.x, a).h;
      T->ser[i][2 * q + 1] = dd_mul(c.y, a).h;
    }
  } else {
    T->ak = ak;
    T->scale = 1.0 / sc;
    T->th = atan2(k.y, k.x);
    T->k = k;
    T->ik = crecip(k);
  }
}

// The tables of two wavenumbers, one workgroup each.
#define HK_RAY_NT 1024
__global__ __launch_bounds__(HK_RAY_NT) void hankel_ray_kernel(cplx k0, cplx k1, hk_ray *out) {
  constexpr int M = 32;  // Chebyshev nodes
  static_assert(HK_NC <= M && HK_RAY_NT == 2 * M * 16, "16 threads per node and sign");
  __shared__ double D[8][M], C[4 * M];
  const cplx k = blockIdx.x ? k1 : k0;
  hk_ray *T = out + blockIdx.x;
  const int tid = threadIdx.x;
  const double ak = hypot(k.x, k.y), th = atan2(k.y, k.x), cth = k.x / ak, sth = k.y / ak;
  if (tid < 4 * M) C[tid] = cospi((double)tid / (2 * M));
  {
    // F_nu - 1 = int weight ((1 + i u / 2z)^{nu - 1/2} - 1) at node m, H^(1) (sg = 0) and,
    // conjugated, at conj z (sg = 1); the differences in a form without cancellation
    const int part = tid & 15, m = (tid >> 4) & (M - 1), sg = tid >> 9;
    const double t = (cospi((m + 0.5) / M) + 1.0) / 6.0;
    const double cx = 0.5 * t * (sg ? -sth : sth), cy = 0.5 * t * cth;  // i t e^{-i th} / 2
    const double h = 0.16, rsp = 1.0 / sqrt(BM_PI);
    cplx d0 = cmk(0, 0), d1 = cmk(0, 0);
    for (int q = 1 + part; q <= 40; q += 16) {
      const double s2 = (q * h) * (q * h), e = h * exp(-s2) * rsp;
      const cplx v = cmk(cx * s2, cy * s2), w = cmk(1.0 + v.x, v.y), rt = csqrt_d(w);
      const cplx f = cdiv(v, cmk(1.0 + rt.x, rt.y));  // sqrt(w) - 1
      const cplx f0 = cdiv(f, rt);                    // 1 - 1/sqrt(w)
      d0 = csub(d0, cscale(f0, 2.0 * e));
      d1 = cadd(d1, cscale(f, 4.0 * e * s2));
    }
#pragma unroll
    for (int x = 8; x > 0; x >>= 1) {
      d0 = cadd(d0, cmk(__shfl_xor(d0.x, x), __shfl_xor(d0.y, x)));
      d1 = cadd(d1, cmk(__shfl_xor(d1.x, x), __shfl_xor(d1.y, x)));
    }
    if (part == 0) {
      D[4 * sg][m] = d0.x;
      D[4 * sg + 1][m] = sg ? -d0.y : d0.y;
      D[4 * sg + 2][m] = d1.x;
      D[4 * sg + 3][m] = sg ? -d1.y : d1.y;
    }
  }
  __syncthreads();
  if (tid < 8 * HK_NC) {
    const int j = tid / 8, q = tid % 8;
    double s = 0.0;
    for (int m = 0; m < M; ++m) s = fma(D[q][m], C[(j * (2 * m + 1)) % (4 * M)], s);
    T->cheb[j][q] = s * ((j == 0) ? 1.0 : 2.0) / M;
  } else if (tid >= 512 && tid <= 512 + HK_NS) {
    hk_wave_item(k, tid - 512, &T->w);
  } else if (tid == 1023) {
    double sn, cs;
    const double c = sqrt(2.0 / BM_PI);
    sincos(-0.5 * th - 0.25 * BM_PI, &sn, &cs);
    T->sq1 = cmk(c * cs, c * sn);
    sincos(-0.5 * th + 0.25 * BM_PI, &sn, &cs);
    T->sq2 = cmk(c * cs, c * sn);
  }
}
