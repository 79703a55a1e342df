// The kernel (i/4) H0(x) = (-Y0(x) + i J0(x)) / 4 as one function (device code).
//
// J0 and Y0 from two library calls cost a few thousand instructions per
// argument; both come here from one evaluation:
//   x >= 8: H0 = sqrt(2 / (pi x)) (P + i Q) e^(i (x - pi/4)), P and x Q
//           polynomials in z = (8 / x)^2, and e^(-i pi/4) taken out exactly,
//           so that only x itself goes through the sine and cosine;
//   x <  8: J0 and Y0 - (2/pi) ln(x/2) J0 by Chebyshev series in
//           2 (x/8)^2 - 1 (Clenshaw's recurrence).
// The coefficients are the Chebyshev interpolants of these functions at 40
// points of the interval, in 50-digit arithmetic (P and Q then expanded in
// z), cut below 1e-17, and Taylor's for the sine and cosine on |r| <= 0.8.
// Errors are at most 5e-16 |H0| for a given x.
#pragma once
#include "common.hpp"

namespace lsh {
namespace hankel {

// coefficients, one table (offsets and lengths below)
__device__ __constant__ double kTab[79] = {
    // P
    1.00000000000000000e+00, -1.09863281249971941e-03, 2.73808836745900268e-05,
    -2.18391908729392621e-06, 3.62033687437910211e-07, -1.02396345780849386e-07,
    4.38296146730047331e-08, -2.54441195570637124e-08, 1.73322449552050808e-08,
    -1.16889128114482359e-08, 6.68673033316311648e-09, -2.83710310794116033e-09,
    7.65111846434127909e-10, -9.66658279850134740e-11,
    // x Q
    -1.25000000000000000e-01, 1.14440917968492372e-03, -5.54462893037581660e-05,
    6.59075259296131087e-06, -1.45312383009376205e-06, 5.12863259559859044e-07,
    -2.62099686259405769e-07, 1.74322061386304993e-07, -1.30387048026867915e-07,
    9.32000812531442303e-08, -5.52106906085186247e-08, 2.39318903883565696e-08,
    -6.54314178683960439e-09, 8.34362908565041545e-10,
    // sin(r) / r in r^2
    1.00000000000000000e+00, -1.66666666666666657e-01, 8.33333333333333322e-03,
    -1.98412698412698413e-04, 2.75573192239858925e-06, -2.50521083854417202e-08,
    1.60590438368216133e-10, -7.64716373181981641e-13,
    // cos(r) in r^2
    1.00000000000000000e+00, -5.00000000000000000e-01, 4.16666666666666644e-02,
    -1.38888888888888894e-03, 2.48015873015873016e-05, -2.75573192239858883e-07,
    2.08767569878681002e-09, -1.14707455977297245e-11, 4.77947733238738525e-14,
    // J0
    1.57727971474890122e-01, -8.72344235285222105e-03, 2.65178613203336799e-01,
    -3.70094993872649769e-01, 1.58067102332097253e-01, -3.48937694114088842e-02,
    4.81918006946760458e-03, -4.60626166206275038e-04, 3.24603288210050832e-05,
    -1.76194690776215074e-06, 7.60816359241878206e-08, -2.67925353055767280e-09,
    7.84869631447946477e-11, -1.94383468673701645e-12, 4.12532059563437413e-14,
    -7.58850812544754590e-16, 1.22185158739614113e-17,
    // Y0 - (2/pi) ln(x/2) J0
    3.64546980911604410e-02, -2.78323709407582498e-01, 2.96049999020714827e-01,
    9.82550840818786353e-02, -1.07551552806277831e-01, 3.17990740844145137e-02,
    -5.16139710581071508e-03, 5.49852532003901199e-04, -4.19969831494201336e-05,
    2.42903611079237928e-06, -1.10499697934729567e-07, 4.06651736597911041e-09,
    -1.23741488982898536e-10, 3.16857255289459451e-12, -6.92695603243100155e-14,
    1.30863086258766845e-15, -2.15862019869144822e-17};
constexpr int kP0 = 0, kPN = 14, kQ0 = 14, kQN = 14, kSin0 = 28, kSinN = 8, kCos0 = 36, kCosN = 9, kJ0 = 45,
              kJN = 17, kY0 = 62, kYN = 17;

// The table through a pointer that the compiler cannot see through: its loads
// stay scalar and inside the caller's loop.  As literals the 79 constants are
// kept in 158 vector registers across the loop, and every multiply-add needs
// a move besides.
typedef const double __attribute__((address_space(4)))* ctab;
__device__ __forceinline__ ctab table() {
  ctab c = (ctab)kTab;
  asm volatile("" : "+s"(c));
  return c;
}

template <int O, int N>
__device__ __forceinline__ double horner(ctab c, double z) {
  double v = c[O + N - 1];
#pragma unroll
  for (int k = N - 2; k >= 0; --k) v = fma(v, z, c[O + k]);
  return v;
}

template <int O, int N>
__device__ __forceinline__ double clenshaw(ctab c, double t) {
  double b1 = c[O + N - 1], b2 = 0.0;
#pragma unroll
  for (int k = N - 2; k > 0; --k) {
    const double b = fma(2.0 * t, b1, c[O + k] - b2);
    b2 = b1;
    b1 = b;
  }
  return fma(t, b1, c[O] - b2);
}

// the library's functions, out of line: their reduction of huge arguments
// would cost every kernel registers that the arguments of a grid never need
__device__ __attribute__((noinline)) inline double2 sincos_far(double x) {
  double sn, cs;
  sincos(x, &sn, &cs);
  return double2{sn, cs};
}

// sin(x) and cos(x) for x >= 8: less k pi/2, pi/2 in two parts (fused, so that
// the rest is exact to 1e-16 of itself while k is exact), and Taylor's
// polynomials
__device__ __forceinline__ void sincos_pos(ctab c, double x, double& sn, double& cs) {
  if (x < 1e12) {
    const double k = rint(x * 0.63661977236758134308);
    const double r = fma(-k, 6.12323399573676603587e-17, fma(-k, 1.57079632679489655800, x)), r2 = r * r;
    const double a = r * horner<kSin0, kSinN>(c, r2), b = horner<kCos0, kCosN>(c, r2);
    const int q = (int)(k - 4.0 * floor(0.25 * k));  // k mod 4
    const double u = (q & 1) ? b : a, v = (q & 1) ? a : b;
    sn = (q & 2) ? -u : u;
    cs = ((q + 1) & 2) ? -v : v;
  } else {
    const double2 t = sincos_far(x);
    sn = t.x;
    cs = t.y;
  }
}

}  // namespace hankel

// (i/4) H0(x) for x >= 0 (x = 0: the real part is +infinity; x = infinity: 0)
__device__ __forceinline__ z64 green_h0(double x) {
  using namespace hankel;
  const ctab c = table();
  if (x < 8.0) {
    const double t = x * x * (1.0 / 32.0) - 1.0;
    const double j = clenshaw<kJ0, kJN>(c, t);
    const double y = fma(0.63661977236758134308 * log(0.5 * x), j, clenshaw<kY0, kYN>(c, t));
    return mk(-0.25 * y, 0.25 * j);
  }
  const double rs = rsqrt(x), w = rs * rs, z = 64.0 * w * w;
  const double p = horner<kP0, kPN>(c, z), q = horner<kQ0, kQN>(c, z) * w;
  double sn, cs;
  sincos_pos(c, x, sn, cs);
  // H0 = (pi x)^(-1/2) (p + i q)(1 - i)(cs + i sn)
  const double a = 0.56418958354775628695 * 0.25 * rs;
  const double u = cs + sn, v = sn - cs;  // (1 - i)(cs + i sn) = u + i v
  const double re = fma(p, u, -q * v), im = fma(p, v, q * u);
  return x < __longlong_as_double(0x7FF0000000000000LL) || !(x == x) ? mk(-a * im, a * re) : mk(0.0, 0.0);
}

}  // namespace lsh
