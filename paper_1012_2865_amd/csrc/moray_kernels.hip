// HIP kernels of the adaptive ray tracer (gfx950).
//
// One radiative-transfer pass (section 3.1, steps 1-3 of Wise & Abel) is the
// launch sequence
//   reset -> prep (absorber column per cell, input checks, zeroed accumulators)
//   -> trace_level(l) for l = l0 .. l_reach -> finalize,
// on one stream. A ray splits at most once per level: every launch consumes
// the rays of HEALPix level l (children written by the previous launch plus
// the seed rays of trees that start at level l) and writes the children of
// level l+1 into the other half of a ping-pong queue, so no launch ever waits
// on work produced inside itself.
//
// Inside trace_level the grid is persistent: every wave keeps 64 rays in
// flight, one per lane, marches them cell by cell (Eq. trace), tests the split
// criterion at each cell exit (Eq. split), and deposits P (1 - e^-tau) of every
// energy group the ray carries into the cell's accumulators (Eqs. dtau, flux,
// kph): with one group the absorbed rate, with more the absorbed rate and its
// energy moment, summed over the groups (Eq. gamma). Deposits combine in a
// per-wave LDS table and reach the float64 accumulators in HBM as atomics only
// when evicted; per-tree ray statistics combine per wave. A wave whose rays have
// all ended or split takes the next from its share of the level, or from units of
// it claimed with one atomic each, after it has written the rays that split, one
// queue slot each, in the order of their pixels.
//
// What bounds it, on the 128^3 workload (16 sources, 4 groups; 4.1 ms): 580
// million steps in 9.95 million wave steps (58 of 64 lanes with a ray), each about
// 115 vector and 100 scalar instructions and ten of LDS: the vector units are busy
// 70% of the step loop, which is three quarters of the time; a tenth goes to ray
// starts (a chain of memory round trips of 17 thousand cycles each), the rest to
// the ends of the levels. Without its memory-side atomics a build was 2 to 4%
// faster, with its gathers all in cache 0 to 3%, without deposits 20%.
#include "moray_device.h"

#include <hip/hip_runtime.h>
#include <cfloat>
#include <cmath>
#include <cstdint>
#include <type_traits>

namespace moray {

// The active lanes where p holds, from its lane mask itself (an int predicate
// costs a select and a compare).
__device__ __forceinline__ unsigned long long wave_mask(bool p) { return __builtin_amdgcn_ballot_w64(p); }
// The lane's bit of a wave-uniform mask, the mask itself serving as the predicate.
__device__ __forceinline__ bool in_mask(unsigned long long m) { return __builtin_amdgcn_inverse_ballot_w64(m); }

// ---------------------------------------------------------------------------
// HEALPix nested pixel centre (Gorski et al. 2005), float64.
// Face f, in-face coordinates (ix, iy) from the even/odd bits of the in-face
// index; ring j = jr(f) Ns - ix - iy - 1; polar caps z = 1 - nr^2/(3 Ns^2),
// equatorial belt z = 2(2 Ns - j)/(3 Ns); azimuth (pi/2)(jp - (s+1)/2)/nr.
// z and sin(theta) come from exact integers; the azimuth is reduced to the
// first octant before sin/cos so multiples of pi/4 are exact.
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint32_t compact_even_bits(uint32_t x) {
  x &= 0x55555555u;
  x = (x | (x >> 1)) & 0x33333333u;
  x = (x | (x >> 2)) & 0x0F0F0F0Fu;
  x = (x | (x >> 4)) & 0x00FF00FFu;
  x = (x | (x >> 8)) & 0x0000FFFFu;
  return x;
}
__device__ __forceinline__ uint64_t compact_even_bits(uint64_t x) {
  x &= 0x5555555555555555ull;
  x = (x | (x >> 1)) & 0x3333333333333333ull;
  x = (x | (x >> 2)) & 0x0F0F0F0F0F0F0F0Full;
  x = (x | (x >> 4)) & 0x00FF00FF00FF00FFull;
  x = (x | (x >> 8)) & 0x0000FFFF0000FFFFull;
  x = (x | (x >> 16)) & 0x00000000FFFFFFFFull;
  return x;
}

// sin and cos of beta in [0, pi/4]: their Taylor series about 0 (coefficients
// 1/n!) through x^19 and x^20 in Horner form; the first omitted terms are
// below 1e-19 relative there, and the rounding of the evaluation stays within
// 1 ulp (0.67 ulp for sin, 0.87 for cos over 4e6 points against long double).
// Used instead of the general sincos, whose argument reduction for large
// arguments would set the trace kernel's register peak.
__device__ __forceinline__ void sincos_octant(double beta, double& s, double& c) {
  const double x2 = beta * beta;
  double ps = 1.0 / 121645100408832000.0;      // 1/19!
  ps = fma(ps, -x2, 1.0 / 355687428096000.0);  // 1/17!
  ps = fma(ps, -x2, 1.0 / 1307674368000.0);    // 1/15!
  ps = fma(ps, -x2, 1.0 / 6227020800.0);       // 1/13!
  ps = fma(ps, -x2, 1.0 / 39916800.0);         // 1/11!
  ps = fma(ps, -x2, 1.0 / 362880.0);           // 1/9!
  ps = fma(ps, -x2, 1.0 / 5040.0);             // 1/7!
  ps = fma(ps, -x2, 1.0 / 120.0);              // 1/5!
  ps = fma(ps, -x2, 1.0 / 6.0);                // 1/3!
  s = fma(beta * x2, -ps, beta);
  double pc = 1.0 / 2432902008176640000.0;     // 1/20!
  pc = fma(pc, -x2, 1.0 / 6402373705728000.0); // 1/18!
  pc = fma(pc, -x2, 1.0 / 20922789888000.0);   // 1/16!
  pc = fma(pc, -x2, 1.0 / 87178291200.0);      // 1/14!
  pc = fma(pc, -x2, 1.0 / 479001600.0);        // 1/12!
  pc = fma(pc, -x2, 1.0 / 3628800.0);          // 1/10!
  pc = fma(pc, -x2, 1.0 / 40320.0);            // 1/8!
  pc = fma(pc, -x2, 1.0 / 720.0);              // 1/6!
  pc = fma(pc, -x2, 1.0 / 24.0);               // 1/4!
  pc = fma(pc, -x2, 0.5);                      // 1/2!
  c = fma(x2, -pc, 1.0);
}

// 1/b, and a/b, of positive finite numbers far from the ends of the range: the
// hardware's estimate and two Newton steps, without the scaling and special cases
// of a general division (which take as many instructions again). The quotient's
// last step is Markstein's: for integers below 2^20 it is the rounded quotient,
// whose distance from a midpoint is then above 2^-75 of it.
__device__ __forceinline__ double reciprocal(double b) {
  double y = __builtin_amdgcn_rcp(b);
  y = fma(fma(-b, y, 1.0), y, y);
  return fma(fma(-b, y, 1.0), y, y);
}
__device__ __forceinline__ double ratio(double a, double b) {
  const double y = reciprocal(b), q = a * y;
  return fma(fma(-b, q, a), y, q);
}
// a/3 rounded (Markstein 1990)
__device__ __forceinline__ double third(double a) {
  const double q = a * (1.0 / 3.0);
  return fma(fma(-3.0, q, a), 1.0 / 3.0, q);
}

// I is the integer type of the ring arithmetic: every intermediate is below
// 16 Ns^2, so 32 bits hold it up to level 13. The polar and equatorial rings, the
// octants and the quarter turns differ by selects, not branches: the lanes of a
// wave straddle them, and a ray start is a tenth of a large level.
template <typename I>
__device__ __forceinline__ void healpix_dir_t(int level, uint64_t pix, double& vx, double& vy, double& vz) {
  using B = std::conditional_t<sizeof(I) == 4, uint32_t, uint64_t>;   // pixel numbers
  const I ns = (I)1 << level;
  const int face = (int)((B)pix >> (2 * level));
  const B ipf = (B)pix & (((B)1 << (2 * level)) - (B)1);
  const I ix = (I)compact_even_bits(ipf);
  const I iy = (I)compact_even_bits((B)(ipf >> 1));
  const int row = face >> 2;                              // 0 north, 1 equator, 2 south
  const I jr = (I)(row + 2) * ns - ix - iy - 1;
  const I jpf = 2 * (face & 3) + (row == 1 ? 0 : 1);
  const bool north = jr < ns, south = jr > 3 * ns, polar = north || south;
  const I nr = north ? jr : (south ? 4 * ns - jr : ns);
  const I m = 2 * (2 * ns - jr);
  // z = (3 Ns^2 - nr^2) / (3 Ns^2) in the caps, m / (3 Ns) between them, and
  // sin(theta) likewise
  const int scale = polar ? -2 * level : -level;
  double z = ldexp(third((double)(polar ? 3 * ns * ns - nr * nr : m)), scale);
  const double root = sqrt((double)(polar ? 6 * ns * ns - nr * nr : 9 * ns * ns - m * m));
  const double sth = ldexp(third(polar ? (double)nr * root : root), scale);
  z = south ? -z : z;
  const int kshift = polar ? 0 : (int)((jr - ns) & 1);
  I jp = (jpf * nr + ix - iy + 1 + kshift) >> 1;          // the numerator is always even
  jp -= jp > 4 * nr ? 4 * nr : 0;
  jp += jp < 1 ? 4 * nr : 0;
  const I num = 2 * jp - kshift - 1, den = 2 * nr;        // quarter turns: num / den, below 4
  const int q = (num >= den ? 1 : 0) + (num >= 2 * den ? 1 : 0) + (num >= 3 * den ? 1 : 0);
  const I rem = num - (I)q * den;
  const bool low = 2 * rem < den, diagonal = 2 * rem == den;
  const I mo = low ? rem : den - rem;
  double sb, cb;
  if constexpr (sizeof(I) == 4) sincos_octant(ratio((double)mo, (double)den) * (M_PI / 2.0), sb, cb);
  else sincos_octant(((double)mo / (double)den) * (M_PI / 2.0), sb, cb);
  sb = diagonal ? M_SQRT1_2 : sb;
  cb = diagonal ? M_SQRT1_2 : cb;
  const bool odd = (q & 1) != 0;
  const double cx = low != odd ? cb : sb, cy = low != odd ? sb : cb;
  vx = sth * (q == 1 || q == 2 ? -cx : cx);
  vy = sth * (q >= 2 ? -cy : cy);
  vz = z;
}

__device__ void healpix_dir(int level, uint64_t pix, double& vx, double& vy, double& vz) {
  if (level <= 13) healpix_dir_t<int32_t>(level, pix, vx, vy, vz);
  else healpix_dir_t<int64_t>(level, pix, vx, vy, vz);
}

// A point on a cell plane belongs to the upper cell when the direction
// component is >= 0, else to the lower one.
__device__ __forceinline__ int cell_rule(double x, double d) { return d >= 0.0 ? (int)floor(x) : (int)ceil(x) - 1; }
__device__ __forceinline__ int floor_half(int c) { return c >= 0 ? c / 2 : -((-c + 1) / 2); }

// One in-order counter covers a wave's vector loads, stores and atomics. A
// load still in flight where a rare path (a ray start, a grid change, the source's
// coordinate for the covering factor) rejoins the hot loop makes the compiler wait at the
// join for that counter to reach zero, which includes every deposit atomic
// issued since; those paths therefore finish their own loads before rejoining.
__device__ __forceinline__ void finish_vector_loads() { __builtin_amdgcn_s_waitcnt(0x0F70); }  // vmcnt(0) alone

// PHYS selects the optional physics some tree of the launch asks for:
// kPhysCover scales deposits by the covering factor (section 2.3), kPhysRadp
// adds the absorbed momentum E_ph dP / c n to three more sums per cell
// (radiation pressure, section 2.5.4), kPhysHalt halts every ray at its
// tree's radius r_halt (time-dependent rays, section 2.1 and section 3.1
// step 3j): the segment in that cell ends there and the ray, with the
// photons it still carries, goes to the halt list for the next step.
// kPhysThin applies the optically-thin approximation (section 2.4, Eq.
// optthin): a ray whose optical depth from its source stays below tau_thin
// through a cell removes no photons there, is split against min(1, phi_c)
// rays per cell face, and sets its tree's mark on the cell (a byte; the rate
// sigma P / (Omega_ray r_cell^2) is the same for every thin ray of a tree,
// so finalize adds it once per marked tree); in a cell that holds the source
// it adds its general deposit to the cell's second sum instead.
// PHYS = 0 is the plain trace.
constexpr int kPhysCover = 1, kPhysRadp = 2, kPhysHalt = 4, kPhysThin = 8;

// ---------------------------------------------------------------------------
// Geometry. Per axis a ray holds the distance t to the next cell plane (root
// cells); the nearest is the exit of the current cell, and stepping across it
// moves that axis to its next plane. The radius and every t are float64 in both
// precision modes: float64 vector adds, multiplies and fmas issue at the float32
// rate here, and one 64-bit value takes the place of a float pair and its
// error terms.
//
// An axis without a direction component never sets the exit: its t is kFar.
// ---------------------------------------------------------------------------
constexpr double kFar = 1e300;

// v_min_f64 and v_max_f64 alone (fmin and fmax would first quiet their operands,
// which are never NaN here)
__device__ __forceinline__ double min_f64(double x, double y) {
  double r;
  asm("v_min_f64 %0, %1, %2" : "=v"(r) : "v"(x), "v"(y));
  return r;
}
__device__ __forceinline__ double max_f64(double x, double y) {
  double r;
  asm("v_max_f64 %0, %1, %2" : "=v"(r) : "v"(x), "v"(y));
  return r;
}

// x = max(x, y) in the lanes of a mask (as a branch: two instructions more, and its wait)
__device__ __forceinline__ void max_where(double& x, double y, unsigned long long lanes) {
  unsigned long long all;
  asm volatile(
      "s_mov_b64 %[all], exec\n\t"
      "s_mov_b64 exec, %[lanes]\n\t"
      "v_max_f64 %[x], %[x], %[y]\n\t"
      "s_mov_b64 exec, %[all]"
      : [x] "+v"(x), [all] "=&s"(all)
      : [y] "v"(y), [lanes] "s"(lanes));
}

// n += 1 there
__device__ __forceinline__ void count_where(unsigned& n, unsigned long long lanes) {
  asm("v_addc_co_u32_e64 %0, vcc, 0, %0, %1" : "+v"(n) : "s"(lanes) : "vcc");
}

// The current cell's exit: distance, and which axis (neither flag: x). Ties go
// to the lowest axis.
struct Exit {
  double t;
  bool y, z;               // z overrides y
  __device__ int axis() const { return z ? 2 : (y ? 1 : 0); }
  template <typename T> __device__ T pick(T a, T b, T c) const { return z ? c : (y ? b : a); }
};

// Float64 mode: the definition's expressions, t = ((b - s) / d) / h for the
// plane coordinate b, so every decision equals the reference's. The quotient is
// rounded correctly without a division: with y = 1/d rounded and q = (b - s) y,
// q + (b - s - q d) y is the rounded quotient (Markstein 1990).
struct Geom64 {
  double d[3], inv[3];     // direction and its reciprocal
  double s[3];             // source in local cells
  double b[3];             // coordinate of the next plane
  double t[3];             // distance to it
  double r;                // radius
  double hinv;             // root cells per local cell
  int sgn[3];              // high word of the float64 +1 or -1 that moves b

  __device__ void set_dir(const double v[3]) {
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      d[k] = v[k];
      inv[k] = v[k] == 0.0 ? kFar : 1.0 / v[k];
      sgn[k] = v[k] > 0.0 ? 0x3ff00000 : (int)0xbff00000;
    }
  }
  __device__ bool up(int k) const { return d[k] > 0.0; }
  __device__ double quotient(int k, double bk) const {
    const double a = bk - s[k], q = a * inv[k];
    const double e = fma(-q, d[k], a);
    return fma(e, inv[k], q) * hinv;
  }
  __device__ void frame(const double sl[3], const int c[3], const int n[3], bool child, double& tbox) {
    hinv = child ? 0.5 : 1.0;
    tbox = __builtin_huge_val();
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      s[k] = sl[k];
      const bool none = d[k] == 0.0;
      if (none) sgn[k] = 0;                        // its plane does not move
      b[k] = (double)(c[k] + (d[k] > 0.0 || none ? 1 : 0));
      t[k] = none ? kFar : quotient(k, b[k]);
      const double face = none ? kFar : quotient(k, d[k] > 0.0 ? (double)n[k] : 0.0);
      tbox = face < tbox ? face : tbox;
    }
  }
  __device__ Exit exit() const {
    Exit e;
    const double m = min_f64(t[0], t[1]);
    e.y = t[1] < t[0];
    e.t = min_f64(m, t[2]);
    e.z = t[2] < m;
    return e;
  }
  __device__ void step(const Exit& e, const int (&st)[3], int sy, int sz, int& lin, uint32_t& yz) {
    const bool ax[3] = {!e.y && !e.z, e.y && !e.z, e.z};
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      b[k] += __hiloint2double(ax[k] ? sgn[k] : 0, 0);
      t[k] = quotient(k, b[k]);                    // (b - s) kFar and more without a component: far
    }
    lin += e.pick(st[0], st[1], st[2]);
    yz += (uint32_t)e.pick(0, sy, sz);
  }
  // a segment counts when it is longer than 0
  static __device__ bool positive(double dr, double) { return dr > 0.0; }
  __device__ double hloc() const { return 1.0 / hinv; }
  // coordinate of the current cell's centre (local cells), and the source's
  __device__ double centre(int k) const { return d[k] == 0.0 ? b[k] - 0.5 : (d[k] > 0.0 ? b[k] - 0.5 : b[k] + 0.5); }
};

// Mixed mode: the planes of an axis are equally spaced, so a step adds the
// spacing e = 1/|d| to that axis' t, against the plane coordinate, its
// difference from the source, the product and its error terms. A t that has been stepped N times is off by at most N/2 of its ulps;
// kResync steps, after which t is formed afresh, keep that below 2^-42 of t.
// Segments shorter than 2^-40 of their exit radius are plane ties (dr = 0 in
// exact arithmetic, or a length no float64 coordinate resolves) and are not
// counted.
constexpr unsigned kResync = 2048;
struct Geom32 {
  double t[3], e[3];       // distance to the next plane, spacing (0: no component along the axis)
  double r;
  double hinv;
  unsigned neg;            // bit k: the direction's component k is negative

  __device__ void set_dir(const double v[3]) {
    neg = 0u;
    hinv = 1.0;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      e[k] = v[k] == 0.0 ? 0.0 : reciprocal(fabs(v[k]));
      if (v[k] < 0.0) neg |= 1u << k;
    }
  }
  __device__ bool up(int k) const { return e[k] != 0.0 && !((neg >> k) & 1u); }
  __device__ void frame(const double sl[3], const int c[3], const int n[3], bool child, double& tbox) {
    hinv = child ? 0.5 : 1.0;
    tbox = __builtin_huge_val();
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      e[k] *= hinv;                                // set_dir precedes every frame
      const bool up_k = up(k), none = e[k] == 0.0;
      const double a = up_k ? (double)(c[k] + 1) - sl[k] : sl[k] - (double)c[k];
      t[k] = none ? kFar : a * e[k];
      const double face = none ? kFar : (up_k ? (double)n[k] - sl[k] : sl[k]) * e[k];
      tbox = face < tbox ? face : tbox;
    }
    // a step within a plane tie of the box's face is taken as leaving, so the
    // rounding of a stepped t never carries a ray past the face
    tbox -= tbox * 0x1p-40;
  }
  __device__ Exit exit() const {
    Exit x;
    const double m = min_f64(t[0], t[1]);
    x.y = t[1] < t[0];
    x.t = min_f64(m, t[2]);
    x.z = t[2] < m;
    return x;
  }
  // Across the exit face, in every lane of the wave (a lane without a ray steps
  // over values nothing reads): t, the cell index and its yz, axis by axis under
  // the axis' lane mask, which takes 8 vector instructions where selects take 18.
  __device__ void step(const Exit& x, const int (&st)[3], int sy, int sz, int& lin, uint32_t& yz) {
    const unsigned long long mz = wave_mask(x.z), my = wave_mask(x.y);
    unsigned long long all, m;
    asm volatile(
        "s_mov_b64 %[all], exec\n\t"
        "s_or_b64 %[m], %[my], %[mz]\n\t"
        "s_andn2_b64 exec, %[all], %[m]\n\t"
        "v_add_f64 %[t0], %[t0], %[e0]\n\t"
        "v_add_u32 %[lin], %[lin], %[s0]\n\t"
        "s_andn2_b64 exec, %[my], %[mz]\n\t"
        "v_add_f64 %[t1], %[t1], %[e1]\n\t"
        "v_add_u32 %[lin], %[lin], %[s1]\n\t"
        "v_add_u32 %[yz], %[yz], %[sy]\n\t"
        "s_mov_b64 exec, %[mz]\n\t"
        "v_add_f64 %[t2], %[t2], %[e2]\n\t"
        "v_add_u32 %[lin], %[lin], %[s2]\n\t"
        "v_add_u32 %[yz], %[yz], %[sz]\n\t"
        "s_mov_b64 exec, %[all]"
        : [t0] "+v"(t[0]), [t1] "+v"(t[1]), [t2] "+v"(t[2]), [lin] "+v"(lin), [yz] "+v"(yz), [all] "=&s"(all),
          [m] "=&s"(m)
        : [e0] "v"(e[0]), [e1] "v"(e[1]), [e2] "v"(e[2]), [s0] "v"(st[0]), [s1] "v"(st[1]), [s2] "v"(st[2]),
          [sy] "v"(sy), [sz] "v"(sz), [my] "s"(my), [mz] "s"(mz)
        : "scc");
  }
  static __device__ bool positive(double dr, double t) { return fma(t, -0x1p-40, dr) > 0.0; }
};

template <typename R> struct GeomOf;
template <> struct GeomOf<double> { using type = Geom64; };
template <> struct GeomOf<float> { using type = Geom32; };

// Photons removed in a segment of optical depth tau: dP = P (1 - e^-tau)
// (Eq. flux), P -= dP.
//
// Float64: 1 - e^-tau by Cody-Waite reduction x = -tau = k ln2 + r, |r| <= ln2/2,
// and the Taylor series of expm1(r) to r^13 (the first omitted term is below
// 1e-17 of r): e^x - 1 = 2^k expm1(r) + (2^k - 1). What r lost in rounding joins the
// square: r^2/2 + its loss. Against the platform's expm1 (262144 points a range,
// ulps rms and at most): tau 0.1 to 0.347 0.292 and 0.69 (0.292 and 0.97), 0.347 to
// 0.5 0.376 and 0.92 (0.440 and 1.12), 0.5 to 3 0.302 and 0.66 (0.304 and 0.73),
// elsewhere the same; without the loss 0.445 and 1.16. 64^3, 16 sources, 4 groups:
// 1.41 ms with the platform's, 1.33 ms with this.
__device__ __forceinline__ double absorb(double& P, double tau) {
  const double x = -fmin(tau, 745.0);                       // e^-745 is the smallest float64
  const double k = __builtin_rint(x * 1.4426950408889634);
  // ln 2 in two parts, the first with 32 bits so k times it is exact
  const double x1 = fma(-k, 0.69314718036912381649, x);
  const double r = fma(-k, 1.9082149292705877e-10, x1);
  const double loss = fma(-k, 1.9082149292705877e-10, x1 - r);
  double q = 1.0 / 6227020800.0;                            // 1/13!
  q = fma(q, r, 1.0 / 479001600.0);
  q = fma(q, r, 1.0 / 39916800.0);
  q = fma(q, r, 1.0 / 3628800.0);
  q = fma(q, r, 1.0 / 362880.0);
  q = fma(q, r, 1.0 / 40320.0);
  q = fma(q, r, 1.0 / 5040.0);
  q = fma(q, r, 1.0 / 720.0);
  q = fma(q, r, 1.0 / 120.0);
  q = fma(q, r, 1.0 / 24.0);
  q = fma(q, r, 1.0 / 6.0);
  q = fma(q, r, 0.5);
  q = fma(fma(r, r, loss + loss), q, r);
  const double p2 = ldexp(1.0, (int)k);
  const double dP = -P * fma(p2, q, p2 - 1.0);
  P -= dP;
  return dP;
}
// Float32, of y = tau / ln 2 (the factor is folded into the cross-section). Thin
// segments (y <= 1): 1 - 2^-y = y ln 2 - y^2 g(y), g of degree 4 fitted on [0, 1]
// to the least relative error of the sum (1.1e-8). The small part, at most 0.31 of
// the sum, is a float; the leading term and the sum are float64, so that little
// more than the rounding of y is left: 2.3e-8 to 2.6e-8 rms for tau of 1e-4 to
// 0.69 (with a float sum 3.4e-8 to 3.6e-8, with a float product y q(y) 4.3e-8 to 5.1e-8;
// the 128^3 workload takes 4.09, 4.11 and 4.10 ms). Thick ones: the transmitted part P 2^-y from
// the hardware exp2 (within 1.5 x 2^-24, and below 2^-126, where it gives 0, from
// 2^(64-y)), and the absorbed part as the float64 difference. dP + P_new = P to
// float64 rounding either way. Where no lane is thick, as in ionised gas and for
// the hardest photons everywhere, the wave takes the series alone.
__device__ __forceinline__ double absorb(double& P, float y) {
  float g = fmaf(y, -1.1519434e-4f, 1.2924776e-3f);
  g = fmaf(y, g, -9.5979832e-3f);
  g = fmaf(y, g, 5.5499703e-2f);
  g = fmaf(y, g, -2.4022619e-1f);
  const double f = fma((double)y, 0.69314718055994530942, (double)((y * y) * g));
  const bool thick = y > 1.0f;
  if (!wave_mask(thick)) {
    const double dP = P * f;
    P -= dP;
    return dP;
  }
  float e = __builtin_amdgcn_exp2f(-y);
  if (wave_mask(y > 126.0f)) e = y > 126.0f ? __builtin_amdgcn_exp2f(64.0f - y) * 0x1p-64f : e;
  const double a = P * (thick ? (double)e : f), rest = P - a;
  P = thick ? a : rest;
  return thick ? rest : a;
}
constexpr double kLog2e = 1.4426950408889634074;
// what the cross-section is multiplied by for absorb's argument
template <typename R> constexpr double kSigmaScale = sizeof(R) == 4 ? kLog2e : 1.0;

// A column or cross-section as R: a float no larger than half the largest, so that a
// column times a segment's length (below sqrt(3)) is finite and 0 times either is 0,
// not NaN (a lane without the group or the segment multiplies by 0). 1.7e38 cm^-2 is
// opaque to any cross-section above 1e-36 cm^2.
template <typename R> __device__ __forceinline__ R in_range(double x) {
  return sizeof(R) == 4 ? (R)fmin(x, 0.5 * (double)FLT_MAX) : (R)x;
}

constexpr unsigned kNoCut = 0xffffffffu;

// Per-lane ray state. A ray carries NG energy groups of its source: they share
// its geometry, and each has its own photon rate, cross-section and end. Only
// what the step reads is held; the rest of the ray's tree and grid is read from
// their tables by the rare paths (a ray start, a grid change).
template <typename R, int NG>
struct Ray {
  typename GeomOf<R>::type g;
  double rs, tbox;        // a step whose exit lies beyond rs splits the ray, at tbox or beyond leaves the grid
  int st[3];              // what crossing a plane of each axis adds to lin
  int lin;                // batch-wide cell index
  uint32_t yz;            // the local cell's j + 8 k
  int sy, sz;             // what crossing a y or z plane adds to it
  int q;                  // grid index
  bool root;              // it is the problem's root grid
  uint64_t pix;           // its pixel, or the one it descends to (see descend)
  int more;               // levels it has still to descend
  uint32_t tree;
  double P[NG], pmin[NG];
  bool alive[NG];         // groups the ray still carries
  unsigned cut[NG];       // of a group truncated in this flight, its segments (its P is what it had left); kNoCut: not
  uint32_t slot0;         // the ray's accumulator of cell lin is acc[slot0 + (lin << ashift)]
  uint32_t ashift;
  R sigma[NG];
  double eexc[NG];        // E - E_ion (moments only)
  R kap;                  // absorber column per root-cell length of the current cell
  unsigned segs;
  uint32_t stat0;
  double mscale;          // E_ph / c, 0 when the problem does not ask for the momentum
  double d[3];            // direction (the variants that need it at every step)
  double ad[3];           // its magnitudes per local cell (covering factor, mixed mode)
  double lpix;            // covering factor: width of the ray's pixel per unit radius, local cells; 0: not scaled
  double rhalt;           // time-dependent rays: radius where the tree's rays halt in this step
  // optically-thin approximation (section 2.4): while the ray is thin, the
  // absorber column it may still cross before its optical depth from the
  // source reaches tau_thin, rem = (tau_thin - tau) / sigma (units of kap x
  // radius), and the split radius of thin rays
  bool thin;
  double rem;
  double kap64;           // the current cell's column in float64 (the thin decision's optical depth)
  double rs_thin;
  long long mark_base;
  unsigned tsegs;         // the ray's thin segments
};

// Why an idle lane's ray goes on: with a new frame after it crossed into or out
// of a child grid along axis 0..2 (kCross + axis), or in the cell it is in
// (kResyncFrame), or as its own child (kChild, see descend). The step loop has no frame code of its own: it holds the
// whole state of every lane, and with the frame's temporaries on top overflows
// the register budget (spills in the loop took the 128^3 workload from 8 to
// 10.5 ms). Such a ray waits, idle, for the wave's next refill, where little else is live.
constexpr int kFresh = 0, kResyncFrame = 1, kChild = 2, kCross = 3;

template <typename R, int NG, int PHYS>
struct Tracer {
  static constexpr bool COVER = (PHYS & kPhysCover) != 0, RADP = (PHYS & kPhysRadp) != 0, THIN = (PHYS & kPhysThin) != 0;
  using L_t = Ray<R, NG>;
  const TraceArgs<R>& a;
  __device__ explicit Tracer(const TraceArgs<R>& args) : a(args) {}

  // Radius (root cells) beyond which an exit splits a ray of `level`: the
  // canonical test 12 * 4^l < (4 pi phi) u^2, u = t h the exit distance in local
  // cells, solved for t. The float64 mode moves it to the largest t that fails
  // the test as float64 evaluates it (which is monotonic in t), so that
  // comparing with it is the test.
  static __device__ double split_radius(double split_r, double four_pi_phi, int level, int level_max, bool child) {
    if (level >= level_max) return __builtin_huge_val();
    const double h = child ? 2.0 : 1.0;
    double rs = ldexp(split_r, child ? level - 1 : level);
    if constexpr (sizeof(R) == 8) {
      const double need = ldexp(12.0, 2 * level);
      auto test = [&](double t) { return need < four_pi_phi * ((t * h) * (t * h)); };
      for (int i = 0; i < 8 && test(rs); ++i) rs = __longlong_as_double(__double_as_longlong(rs) - 1);
      for (int i = 0; i < 8; ++i) {
        const double up = __longlong_as_double(__double_as_longlong(rs) + 1);
        if (test(up)) break;
        rs = up;
      }
    }
    return rs;
  }
  // Descend. The coarse levels hold few rays, each of which crosses few cells: a
  // launch per level for them is a chain of dependent loads on an idle device
  // (30 to 80 us a level, most of a small problem's solve). The seeds therefore
  // enter at a finer level, that of the launch: one lane per pixel of it, each of
  // which traces its pixel's ancestors from the seed level on, going on in place
  // as its own child where a ray splits. All descendants of a pixel trace it alike;
  // the first of them (low bits 0) owns it and alone deposits and counts. What the
  // others repeat costs lanes that would idle otherwise.
  __device__ int level_of(const TreeDev& S) const { return S.level_init + (a.gen - S.gen0); }   // of the launch
  __device__ int level_of(const TreeDev& S, const L_t& L) const { return level_of(S) - L.more; }
  static __device__ uint64_t pixel(const L_t& L) { return L.pix >> (2 * L.more); }
  static __device__ bool owner(const L_t& L) { return (L.pix & ((1ull << (2 * L.more)) - 1ull)) == 0ull; }

  // The ray's frame in grid q at local cell c: source in its cells, planes,
  // strides, split radius and cell index.
  __device__ void frame(L_t& L, const TreeDev& S, int q, const int c[3]) const {
    const bool child = q != S.root_grid;
    int n[3] = {S.rnx, S.rny, S.rnz};
    double sl[3] = {S.sx, S.sy, S.sz};
    long long off = S.rcell_off;
    if (child) {
      const GridDev& G = a.grids[q];
      n[0] = G.nx; n[1] = G.ny; n[2] = G.nz;
      sl[0] = 2.0 * (S.sx - (double)G.ox); sl[1] = 2.0 * (S.sy - (double)G.oy); sl[2] = 2.0 * (S.sz - (double)G.oz);
      off = G.cell_off;
    }
    L.q = q;
    L.root = !child;
    L.g.frame(sl, c, n, child, L.tbox);
    const int level = level_of(S, L);
    L.rs = split_radius(S.split_r, S.four_pi_phi_c, level, S.level_max, child);
    if constexpr (THIN) L.rs_thin = split_radius(S.split_r_thin, S.four_pi_phi_thin, level, S.level_max, child);
    if constexpr (COVER) {
      // sqrt(pi/3) 2^-l, the pixel's width at unit distance
      L.lpix = S.covering ? ldexp(1.0233267079464885, child ? 1 - level : -level) : 0.0;
      if constexpr (sizeof(R) == 4) {
#pragma unroll
        for (int k = 0; k < 3; ++k) L.ad[k] = child ? 2.0 * fabs(L.d[k]) : fabs(L.d[k]);
      }
    }
    const int sx = n[0], sxy = n[0] * n[1];
    L.st[0] = L.g.up(0) ? 1 : -1;
    L.st[1] = L.g.up(1) ? sx : -sx;
    L.st[2] = L.g.up(2) ? sxy : -sxy;
    L.lin = (int)off + c[0] + sx * (c[1] + n[1] * c[2]);
    L.yz = (uint32_t)c[1] + 8u * (uint32_t)c[2];
    L.sy = L.g.up(1) ? 1 : -1;
    L.sz = L.g.up(2) ? 8 : -8;
  }

  // Local cell of batch-wide index lin in grid q.
  __device__ void cell(const TreeDev& S, int q, int lin, int c[3]) const {
    int nx = S.rnx, ny = S.rny;
    long long off = S.rcell_off;
    if (q != S.root_grid) {
      const GridDev& G = a.grids[q];
      nx = G.nx; ny = G.ny;
      off = G.cell_off;
    }
    const unsigned local = (unsigned)(lin - (int)off);
    const unsigned row = local / (unsigned)nx;
    c[0] = (int)(local - row * (unsigned)nx);
    c[2] = (int)(row / (unsigned)ny);
    c[1] = (int)(row - (unsigned)c[2] * (unsigned)ny);
  }

  // From root cell c, covered by child grid `ch`, into the child's cell: along
  // the crossing axis it follows from the face, along the others from the
  // position x on the ray (direction v), kept among the two fine cells under the
  // root cell. ax = 3: from the position along every axis (a ray that starts).
  __device__ void into_child(int ch, int c[3], const double x[3], const double v[3], int ax) const {
    const GridDev& G = a.grids[ch];
    const int o[3] = {G.ox, G.oy, G.oz};
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const int lo = 2 * (c[k] - o[k]);
      const int at = min(max(cell_rule(2.0 * (x[k] - (double)o[k]), v[k]), lo), lo + 1);
      c[k] = k == ax ? lo + (v[k] < 0.0 ? 1 : 0) : at;
    }
  }

  // The leaf cell (grid q, local cell c) a ray goes on in after it crossed a
  // face of cell `from` of grid q along `ax`, out of a child grid or into a root
  // cell under one. Returns false when it left the root grid.
  __device__ bool cross(const TreeDev& S, int& q, int from, int ax, int c[3], const double x[3], const double v[3]) const {
    cell(S, q, from, c);
#pragma unroll
    for (int k = 0; k < 3; ++k) c[k] += k == ax ? (v[k] < 0.0 ? -1 : 1) : 0;
    if (q != S.root_grid) {
      const GridDev& G = a.grids[q];
      if ((unsigned)c[0] < (unsigned)G.nx && (unsigned)c[1] < (unsigned)G.ny && (unsigned)c[2] < (unsigned)G.nz)
        return true;                               // crossed within a plane tie of the child's face
      c[0] = G.ox + floor_half(c[0]); c[1] = G.oy + floor_half(c[1]); c[2] = G.oz + floor_half(c[2]);
      q = S.root_grid;
    }
    if ((unsigned)c[0] >= (unsigned)S.rnx || (unsigned)c[1] >= (unsigned)S.rny || (unsigned)c[2] >= (unsigned)S.rnz)
      return false;
    const R k = a.kappa[(int)S.rcell_off + c[0] + S.rnx * (c[1] + S.rny * c[2])];
    if (k < (R)0) {
      q = (int)(-k) - 1;
      into_child(q, c, x, v, ax);
    }
    return true;
  }

  // A ray starts in three steps:
  //   fetch  - its queue record (a child of a split ray), its halted record,
  //            or its tree and pixel (a seed); a ray that changes frames (see
  //            Again) has its state;
  //   tree   - the tree's constants;
  //   locate - direction, start cell and frame, and that cell's absorber column.
  __device__ void fetch_child(L_t& L, unsigned long long i, double& r64) const {
    const unsigned long long slot = i >> 2;
    L.tree = a.in.tree[slot];
    L.pix = 4ull * a.in.pix[slot] + (i & 3ull);
    L.more = 0;
    r64 = a.in.r[slot];
#pragma unroll
    for (int g = 0; g < NG; ++g) L.P[g] = 0.25 * a.in.P[g * a.in.pstride + slot];
  }
  __device__ void fetch_held(L_t& L, unsigned long long i, double& r64) const {
    const unsigned long long slot = a.held_order[a.held_first + i];
    L.tree = a.held.tree[slot];
    L.pix = a.held.pix[slot];
    L.more = 0;
    r64 = a.held.r[slot];
#pragma unroll
    for (int g = 0; g < NG; ++g) L.P[g] = a.held.P[g * a.held.pstride + slot];
  }
  __device__ void fetch_seed(L_t& L, unsigned long long i, double& r64) const {
    const unsigned long long npix = 12ull << (2 * a.seed_level);
    L.tree = (uint32_t)(a.seed_begin + i / npix);
    L.pix = i % npix;
    const TreeDev& S = a.trees[L.tree];
    L.more = a.gen - S.gen0;
    r64 = 0.0;
#pragma unroll
    for (int g = 0; g < NG; ++g) L.P[g] = S.P0[g];
  }

  __device__ void load_tree(L_t& L, const TreeDev& S) const {
    L.slot0 = (uint32_t)S.acc_slot;
    L.stat0 = S.stat0;
    L.ashift = S.acc_shift;
    if constexpr (RADP) L.mscale = S.mom_scale;
    if constexpr ((PHYS & kPhysHalt) != 0) L.rhalt = S.r_halt;
    if constexpr (THIN) L.mark_base = S.mark_base;
    const int level = level_of(S, L);
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      L.pmin[g] = ldexp(S.pmin0[g], -2 * (level - S.level_init));
      L.sigma[g] = in_range<R>(S.sigma64[g] * kSigmaScale<R>);
      L.eexc[g] = S.eexc[g];
    }
  }

  // Thin state of a fetched ray (before locate). A thin ray has removed no
  // photons, so its rate is its seed's, quartered per level; its queue
  // record holds -4 (1 + rem) in place of the rate, which reading a child
  // quarters like any rate. A seed is thin when its tree uses the
  // approximation. rem is capped at kRemMax (a zero cross-section), which
  // keeps every record finite.
  static constexpr double kRemMax = 1e300;
  __device__ void thin_start(L_t& L, const TreeDev& S, bool seed) const {
    L.tsegs = 0;
    if (seed) {
      L.thin = S.tau_thin > 0.0;
      const double r = S.tau_thin / S.sigma64[0];
      L.rem = r < kRemMax ? r : kRemMax;
    } else if (L.P[0] < 0.0) {
      L.thin = true;
      L.rem = -L.P[0] - 1.0;
      L.P[0] = ldexp(S.P0[0], -2 * (level_of(S) - S.level_init));   // a queue record: of the launch's level
    } else {
      L.thin = false;
    }
  }

  // Does the ray's current cell hold its source (inside or on its boundary)?
  // Only a cell within sqrt(3) local cells of the source can: nearer than 2
  // the test is taken exactly, on the source's float64 local coordinates.
  __device__ bool holds_source(const L_t& L) const {
    if (L.g.r >= 2.0 * L.g.hinv) return false;
    const TreeDev& S = a.trees[L.tree];
    double sl[3] = {S.sx, S.sy, S.sz};
    if (L.q != S.root_grid) {
      const GridDev& G = a.grids[L.q];
      sl[0] = 2.0 * (S.sx - (double)G.ox);
      sl[1] = 2.0 * (S.sy - (double)G.oy);
      sl[2] = 2.0 * (S.sz - (double)G.oz);
    }
    int c[3];
    cell(S, L.q, L.lin, c);
    bool in = true;
#pragma unroll
    for (int k = 0; k < 3; ++k) in = in && (double)c[k] <= sl[k] && sl[k] <= (double)c[k] + 1.0;
    return in;
  }

  // Start of a fetched ray (again = kFresh: in its leaf cell, the root cell
  // holding s + r d or where a child grid covers that the fine cell under it,
  // exact in floating point and kept in range regardless), or a new frame of one
  // in flight. Returns false when it is outside the root grid.
  __device__ bool locate(L_t& L, const TreeDev& S, double r64, int again, int from, int q) const {
    double v[3];
    healpix_dir(level_of(S, L), pixel(L), v[0], v[1], v[2]);
    L.g.set_dir(v);
    L.g.r = r64;
    if constexpr (RADP || (COVER && sizeof(R) == 4)) {
      L.d[0] = v[0]; L.d[1] = v[1]; L.d[2] = v[2];
    }
    const double x[3] = {__dadd_rn(S.sx, __dmul_rn(r64, v[0])), __dadd_rn(S.sy, __dmul_rn(r64, v[1])),
                         __dadd_rn(S.sz, __dmul_rn(r64, v[2]))};
    int c[3];
    if (again == kFresh || again == kChild) {
      L.segs = 0;
#pragma unroll
      for (int g = 0; g < NG; ++g) {
        // a record may hold fewer rates than NG: what it has in their place, which may be
        // anything, must not reach the step (it computes every group some lane carries)
        L.alive[g] = NG == 1 || (g < S.n_grp && L.P[g] >= 0.0);
        if constexpr (NG > 1) L.P[g] = L.alive[g] ? L.P[g] : -1.0;
        L.cut[g] = kNoCut;
      }
      q = S.root_grid;
      c[0] = cell_rule(x[0], v[0]); c[1] = cell_rule(x[1], v[1]); c[2] = cell_rule(x[2], v[2]);
      if ((unsigned)c[0] >= (unsigned)S.rnx || (unsigned)c[1] >= (unsigned)S.rny || (unsigned)c[2] >= (unsigned)S.rnz)
        return false;
      const R k = a.kappa[(int)S.rcell_off + c[0] + S.rnx * (c[1] + S.rny * c[2])];
      if (k < (R)0) {
        q = (int)(-k) - 1;
        into_child(q, c, x, v, 3);
      }
      L.kap = k;
    } else if (again == kResyncFrame) {
      cell(S, q, from, c);
    } else if (!cross(S, q, from, again - kCross, c, x, v)) {
      return false;
    }
    frame(L, S, q, c);
    // (a ray that starts in a root cell has it already)
    if ((again != kFresh && again != kChild) || q != S.root_grid) L.kap = a.kappa[L.lin];
    return true;
  }

  // Covering factor of the segment that starts at the current radius R_0 and
  // has chord dr (root cells), section 2.3: D_edge = 1/2 - max_i D_c,i is
  // the distance from the segment's midpoint to the nearest face of its cell,
  // L_pix = R_0 theta_pix the pixel's width at entry (theta_pix =
  // sqrt(4 pi / N_pix) = sqrt(pi/3) 2^-l), both in local cells, and
  // f_c = (1/2 + D_edge / L_pix)^2, at most 1 (1 also for R_0 = 0). The mixed
  // mode takes D_c,i from the distance left to the axis' next plane; along an
  // axis without a direction component it comes from the source's coordinate.
  __device__ double covering_factor(const L_t& L, double dr) const {
    const double r0 = L.g.r;
    double dmax = 0.0;
    if constexpr (sizeof(R) == 4) {
      const double rmid = r0 + 0.5 * dr;
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        double d;
        if (L.ad[k] == 0.0) {
          const TreeDev& S = a.trees[L.tree];
          const GridDev& G = a.grids[L.q];
          const double s = k == 0 ? S.sx : (k == 1 ? S.sy : S.sz);
          const double sl = L.q != S.root_grid ? 2.0 * (s - (double)(k == 0 ? G.ox : (k == 1 ? G.oy : G.oz))) : s;
          d = fabs(sl - floor(sl) - 0.5);
          finish_vector_loads();
        } else {
          d = fabs((L.g.t[k] - rmid) * L.ad[k] - 0.5);
        }
        dmax = d > dmax ? d : dmax;
      }
    } else {
      const double h = L.g.hloc();
      const double rmid = (r0 + 0.5 * dr) * h;
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        const double d = fabs(L.g.s[k] + rmid * L.g.d[k] - L.g.centre(k));
        dmax = d > dmax ? d : dmax;
      }
    }
    const double lpix = r0 * L.lpix;
    if (!(lpix > 0.0)) return 1.0;
    const double f = 0.5 + ratio(0.5 - dmax, lpix);
    return f * f >= 1.0 ? 1.0 : f * f;
  }
};

// Wave-uniform values in scalar registers: the first active lane's, lane 0's,
// and the wave's number in its block (which the compiler cannot tell is uniform).
__device__ __forceinline__ int uniform32(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ unsigned long long uniform64(unsigned long long v) {
  const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)v);
  const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)(v >> 32));
  return ((unsigned long long)hi << 32) | lo;
}
__device__ __forceinline__ unsigned long long lane0_64(unsigned long long v) {
  const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)v, 0);
  const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(v >> 32), 0);
  return ((unsigned long long)hi << 32) | lo;
}
// the lane's place among the lanes of a mask
__device__ __forceinline__ unsigned lane_rank(unsigned long long m, unsigned base) {
  return __builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, base));
}
__device__ __forceinline__ int wave_in_block() { return uniform32((int)(threadIdx.x / kWave)); }

// The order of a wave's lanes that its rays' order follows: lane l holds the ray
// of rank lane_pos(l). Neighbouring rays cross the same cells, and the LDS
// serialises a float64 atomic of lanes with one address at about 2.9 cycles a lane
// within each row of 16 (4 of 16 neighbours in one cell: 45 cycles an instruction;
// 4 lanes of different rows: 12). Dealing consecutive rays to the four rows in turn
// leaves each row a quarter of a cell's rays: 128^3, 16 sources, 4 groups 5.25 -> 4.80 ms, with
// radiation pressure (four sums a deposit) 11.8 -> 8.7 ms.
__device__ __forceinline__ int lane_pos(int lane) { return ((lane & 15) << 2) | (lane >> 4); }
// the lanes with p, bit lane_pos(l) for lane l (every lane calls)
__device__ __forceinline__ unsigned long long pos_mask(bool p) {
  const int i = (int)(threadIdx.x & (kWave - 1));
  return wave_mask(__builtin_amdgcn_ds_bpermute(((i >> 2) | ((i & 3) << 4)) << 2, p ? 1 : 0) != 0);
}
__device__ __forceinline__ unsigned long long bits_below(int pos) { return (1ull << pos) - 1ull; }

// Sums over the 64 lanes of a wave in which every lane is active (data-parallel
// primitives: row shifts inside 16 lanes, then the two row broadcasts; the last
// lane holds the total).
template <int CTRL, int ROWS>
__device__ __forceinline__ unsigned dpp_zero(unsigned x) {
  return (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, ROWS, 0xf, false);
}
template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_zero(double x) {
  const unsigned long long u = __double_as_longlong(x);
  const unsigned lo = dpp_zero<CTRL, ROWS>((unsigned)u), hi = dpp_zero<CTRL, ROWS>((unsigned)(u >> 32));
  return __longlong_as_double(((unsigned long long)hi << 32) | lo);
}
template <typename T>
__device__ __forceinline__ T wave_total(T x) {     // valid in the last lane
  x += dpp_zero<0x111, 0xf>(x);                    // row_shr:1
  x += dpp_zero<0x112, 0xf>(x);
  x += dpp_zero<0x114, 0xf>(x);
  x += dpp_zero<0x118, 0xf>(x);
  x += dpp_zero<0x142, 0xa>(x);                    // row_bcast:15 into rows 1 and 3
  x += dpp_zero<0x143, 0xc>(x);                    // row_bcast:31 into rows 2 and 3
  return x;
}

// Per-(tree, group) statistics of finished rays (segments, splits, escaped and
// truncated rays with their photon rates). The rays of a claim nearly always
// belong to one tree, so a wave keeps one tree's sums in LDS and adds them to
// the tree's global counters when it changes trees and at its end; a ray of
// another tree adds to the global counters directly. Ended rays are tallied
// when their lanes refill, all at once: the counts come from ballots and the
// rates from one reduction, so a ray end puts no atomic into the memory
// counter the next column gather waits on (a global atomic per ray end took
// the 128^3 workload, 16 sources and 4 groups, from 11.7 to 21 ms).
// kind: 0 escaped, 1 every group truncated, 2 split, 3 halted (its segments only:
// the photons it holds are summed where its record is written).
template <int NG, bool THIN>
struct WaveTally {
  static constexpr int kRows = 5;                  // segs, splits, n_esc, n_trunc, thin_segs
  unsigned long long* cnt;                         // [kRows][NG]
  double* sum;                                     // [2][NG]: esc_P, trunc_P
  uint32_t stat0;                                  // wave-uniform; kNoTree: none yet

  __device__ void init(int lane) {
    __shared__ unsigned long long scnt[kTraceBlock / kWave][kRows * NG];
    __shared__ double ssum[kTraceBlock / kWave][2 * NG];
    cnt = scnt[wave_in_block()];
    sum = ssum[wave_in_block()];
    stat0 = kNoTree;
    clear(lane);
  }
  __device__ void clear(int lane) {
    if (lane < kRows * NG) cnt[lane] = 0ull;
    if (lane < 2 * NG) sum[lane] = 0.0;
    __builtin_amdgcn_wave_barrier();
  }
  __device__ void flush(SgStats* stats, int lane) {
    __builtin_amdgcn_wave_barrier();
    if (stat0 != kNoTree && lane < NG) {
      SgStats& st = stats[stat0 + lane];
      if (cnt[lane]) atomicAdd(&st.segs, cnt[lane]);
      if (cnt[NG + lane]) atomicAdd(&st.splits, cnt[NG + lane]);
      if (cnt[2 * NG + lane]) {
        atomicAdd(&st.n_esc, cnt[2 * NG + lane]);
        unsafeAtomicAdd(&st.esc_P, sum[lane]);
      }
      if (cnt[3 * NG + lane]) {
        atomicAdd(&st.n_trunc, cnt[3 * NG + lane]);
        unsafeAtomicAdd(&st.trunc_P, sum[NG + lane]);
      }
      if (THIN && cnt[4 * NG + lane]) atomicAdd(&st.thin_segs, cnt[4 * NG + lane]);
    }
    __builtin_amdgcn_wave_barrier();
  }
  // the tree whose sums the wave keeps from now on (all lanes)
  __device__ void follow(SgStats* stats, uint32_t s0, int lane) {
    if (s0 == stat0) return;
    flush(stats, lane);
    clear(lane);
    stat0 = s0;
  }
  static __device__ void direct(SgStats& st, unsigned segs, unsigned tsegs, int kind, double P) {
    if (segs) atomicAdd(&st.segs, (unsigned long long)segs);
    if (THIN && tsegs) atomicAdd(&st.thin_segs, (unsigned long long)tsegs);
    if (kind == 2) {
      atomicAdd(&st.splits, 1ull);
    } else if (kind == 0) {
      atomicAdd(&st.n_esc, 1ull);
      unsafeAtomicAdd(&st.esc_P, P);
    } else if (kind == 1) {
      atomicAdd(&st.n_trunc, 1ull);
      unsafeAtomicAdd(&st.trunc_P, P);
    }
  }
  // every lane whose ray ended with `kind` >= 0 (all lanes): its groups, those
  // truncated in this flight and those that ended with the ray
  template <typename RAY>
  __device__ void ended(SgStats* stats, const RAY& L, int kind, int lane) {
    const bool over = kind >= 0, here = L.stat0 == stat0;
    // the segments of the rays of which a group is live, summed once for all
    // groups that are live in every one of them
    const unsigned long long ends = wave_mask(over), ours = wave_mask(here);
    const unsigned all = wave_total(over && here ? L.segs : 0u);
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      const unsigned long long live = ends & wave_mask(L.alive[g]), cut = ends & ~live & wave_mask(L.cut[g] != kNoCut);
      if (!(cut | live)) continue;
      const unsigned mine = in_mask(live) ? L.segs : L.cut[g];
      const unsigned segs = live == ends ? all : wave_total(in_mask((cut | live) & ours) ? mine : 0u);
      const unsigned tsegs = THIN ? wave_total(in_mask((cut | live) & ours) ? L.tsegs : 0u) : 0u;
      const unsigned long long split = wave_mask(kind == 2) & live & ours, out = wave_mask(kind == 0) & live & ours;
      const unsigned long long trunc = cut & ours;
      const double esc_P = out ? wave_total(in_mask(out) ? L.P[g] : 0.0) : 0.0;
      const double trunc_P = trunc ? wave_total(in_mask(trunc) ? L.P[g] : 0.0) : 0.0;
      if (lane == kWave - 1) {
        cnt[g] += segs;
        if (split) cnt[NG + g] += (unsigned)__popcll(split);
        if (out) {
          cnt[2 * NG + g] += (unsigned)__popcll(out);
          sum[g] += esc_P;
        }
        if (trunc) {
          cnt[3 * NG + g] += (unsigned)__popcll(trunc);
          sum[NG + g] += trunc_P;
        }
        if (THIN) cnt[4 * NG + g] += tsegs;
      }
      if (in_mask((cut | live) & ~ours))
        direct(stats[L.stat0 + g], mine, THIN ? L.tsegs : 0u, in_mask(cut) ? 1 : kind, L.P[g]);
    }
    __builtin_amdgcn_wave_barrier();
  }
};

// Every global store or atomic a wave issues stays outstanding in the same
// in-order counter as its loads, so the next gather of an absorber column
// may wait for it, and float64 atomics are performed at the memory side, one
// 64-byte request at a time: 2.4e10 requests a second, whether a request holds
// one sum or eight neighbouring ones. The trace therefore stages its writes in
// LDS and issues them in bulk: deposits combine in a per-wave cache of
// accumulator lines, evicted lines collect in a per-wave buffer drained eight
// at a time, and rays that split are written when their wave refills.

// Deposit combining: each wave keeps a direct-mapped cache of accumulator lines,
// eight consecutive float64 sums (64 bytes) each, in LDS. The rays of a wave
// come from one small patch of HEALPix pixels, so each cell of their cone
// receives several of their deposits a few steps apart, and the cells of a
// line (eight of one sum, four of two) are crossed one after the other by rays
// along x and side by side by the others. All of them add up in LDS; the line
// leaves with one request when another takes its entry or the launch ends.
// Against a table of single cells that is a third of the memory-side requests.
//
// A deposit is NS consecutive sums of one cell's record, which never straddles a
// line: the absorbed rate (1), the moments of rays with several groups (2:
// absorbed rate, energy), or the radiation-pressure record (4). `shift` says how
// many of them (2^shift) the lane's problem keeps (a batch may mix problems).
//
// kLines and kOut: what three blocks leave of a CU's 160 KB of LDS.
constexpr int kLineLog2 = 7, kLines = 1 << kLineLog2;
constexpr int kOut = 24;                       // evicted lines waiting for their atomics

// Entry of a line: 8 x 8 cells in y and z, two lines in x, so the lines a wave
// uses at about the same time, those of a compact patch of cells, never share an
// entry, and a line leaves when the wave has moved on by eight cells (a
// multiplicative hash of the line number put about one conflict into every step
// and as many requests on the memory side as a table of single cells). yz is the
// local cell's j + 8 k, whose low six bits differ between any two cells less than
// eight apart in y and z. Any value is correct: a line that is found
// under two entries is summed in both.
__device__ __forceinline__ uint32_t line_index(uint32_t slot, uint32_t yz) {
  static_assert(kLines == 128, "two lines of 64 cells");
  return ((slot << 3) & 64u) | (yz & 63u);
}
// Where sum j of entry h's line is kept (bytes): in 64 banks of 32 bits four entries side
// by side have their own, so those of different z are rotated against each other
// (radiation pressure 9.98 -> 8.67 ms).
__device__ __forceinline__ uint32_t line_place(uint32_t h, uint32_t j) { return (h << 6) | (((j << 3) ^ h) & 56u); }

template <bool CACHE, int NS>
struct DepositCache {
  static constexpr int kWaves = kTraceBlock / kWave;
  uint32_t* key;          // line numbers of all waves' entries; kNoSlot: empty
  double* val;            // [8] each
  uint32_t* okey;
  double* oval;           // [kOut][8] each
  uint2* moves;           // (entry, line) pairs of one call's evictions
  uint32_t first;         // the wave's first entry
  int ocount;             // wave-uniform

  __device__ void init(int lane) {
    if constexpr (CACHE) {
      __shared__ uint32_t skey[kWaves * kLines];
      __shared__ double sval[8 * kWaves * kLines];
      __shared__ uint32_t sokey[kWaves][kOut];
      __shared__ double soval[kWaves][8 * kOut];
      __shared__ uint2 smoves[kWaves * kWave];
      const int wv = wave_in_block();
      key = skey;
      val = sval;
      okey = sokey[wv];
      oval = soval[wv];
      moves = smoves;
      ocount = 0;
      // in a vector register: the step loop has scalar ones to spare for nothing
      first = (uint32_t)(threadIdx.x / kWave) * kLines;
      asm volatile("" : "+v"(first));
      for (int e = lane; e < kLines; e += kWave) key[first + e] = kNoSlot;
      for (int e = lane; e < 8 * kLines; e += kWave) val[8 * first + e] = 0.0;
      __builtin_amdgcn_wave_barrier();
    }
  }
  __device__ __forceinline__ double* at(uint32_t bytes) const { return (double*)((char*)val + bytes); }
  static __device__ __forceinline__ void add_line(double* acc, uint32_t line, int j, double v) {
    if (v != 0.0) unsafeAtomicAdd(&acc[((unsigned long long)line << 3) + j], v);
  }
  // eight lanes a line, eight lines an instruction
  __device__ void drain(double* acc, int lane) {
    if constexpr (CACHE) {
      __builtin_amdgcn_wave_barrier();
      static_assert(8 * kOut % kWave == 0, "whole waves of sums");
      double v[8 * kOut / kWave];
      uint32_t line[8 * kOut / kWave];
#pragma unroll
      for (int k = 0; k < 8 * kOut / kWave; ++k) {
        v[k] = oval[lane + k * kWave];
        line[k] = okey[(lane + k * kWave) >> 3];
      }
#pragma unroll
      for (int k = 0; k < 8 * kOut / kWave; ++k)
        if (lane + k * kWave < 8 * ocount) add_line(acc, line[k], lane & 7, v[k]);
      ocount = 0;
      __builtin_amdgcn_wave_barrier();
    }
  }
  // A deposit takes four calls, made by every lane of the wave (uniform control
  // flow), with the step's other work between them, so that no LDS round trip is
  // waited for where it is asked (issued and awaited in one place, three of them
  // took a fifth of the step).
  // probe: every lane that may deposit reads its entry's line, exchanges its own
  // in, and reads the entry again; the last read tells which line owns the
  // entry from now on (lanes of different lines race for it; the last one wins).
  // list: where the owner differs from the line before, the entry's sums belong to
  // that: the lane whose exchange returned it (the first in the race; a
  // lane that holds the old line itself can make it several) lists the entry.
  // add: eight lanes per listed entry exchange zeros in and get the old sums
  // (an entry listed twice gives zeros the second time); then the lanes
  // of the owning line add their deposits, and those of a losing line add theirs
  // to memory. The LDS operations of a wave are performed in order, so no wait
  // separates the exchanges from the adds.
  // keep: the old sums go to the buffer.
  // The phases are separated by wave barriers, which keep the compiler from merging them.
  struct Probe {
    uint32_t h, was, before, owner;
    unsigned long long moved;            // lanes that listed an entry
    int count;                           // entries whose sums are still to be kept
    uint2 listed;                        // the entry (x) and line the lane's eight move
    double old;                          // its sum
  };
  __device__ __forceinline__ Probe probe(uint32_t slot, uint32_t yz, unsigned long long has) const {
    Probe p;
    p.moved = 0;
    if constexpr (CACHE) {
      const uint32_t line = slot >> 3;
      p.h = first | line_index(slot, yz);
      // undefined in the other lanes, and not known to be: a constant there lets the
      // compiler compare at once, which waits for the reads
      asm("" : "=v"(p.was), "=v"(p.before), "=v"(p.owner));
      asm("" : "=v"(p.listed), "=v"(p.old));
      if (in_mask(has)) {
        p.was = __hip_atomic_load(&key[p.h], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        p.before = __hip_atomic_exchange(&key[p.h], line, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        p.owner = __hip_atomic_load(&key[p.h], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      }
      __builtin_amdgcn_wave_barrier();
    }
    return p;
  }
  __device__ __forceinline__ void list(Probe& p, unsigned long long has, int lane) const {
    if constexpr (CACHE) {
      p.moved = has & wave_mask(p.owner != p.was) & wave_mask(p.before == p.was) & wave_mask(p.was != kNoSlot);
      if (p.moved) {
        if (in_mask(p.moved)) moves[lane_rank(p.moved, first / (kLines / kWave))] = make_uint2(p.h, p.was);
        __builtin_amdgcn_wave_barrier();
        p.listed = moves[first / (kLines / kWave) + (lane >> 3)];   // past the listed ones: unused
        __builtin_amdgcn_wave_barrier();
      }
    }
  }
  // the sums of `count` listed entries (at most eight)
  __device__ __forceinline__ void take(double* acc, Probe& p, int count, int lane) {
    if (ocount + count > kOut) drain(acc, lane);
    p.count = count;
    if ((lane >> 3) < count)
      p.old = __hip_atomic_exchange(at(line_place(p.listed.x, lane)), 0.0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    __builtin_amdgcn_wave_barrier();
  }
  __device__ __forceinline__ void keep(const Probe& p, int lane) {
    if constexpr (CACHE) {
      if (p.moved) {
        const int i = lane >> 3;
        if (i < p.count) {
          oval[8 * ocount + lane] = p.old;
          if ((lane & 7) == 0) okey[ocount + i] = p.listed.y;
        }
        ocount += p.count;
        __builtin_amdgcn_wave_barrier();
      }
    }
  }
  // Without the cache: NS neighbouring lanes add the NS sums of one of their records at
  // a time, so that a record leaves with one request, not with one a sum (64^3 with a
  // nested grid, 6 sources, 4 groups 2.98 -> 1.69 ms; with radiation pressure 9.82 -> 2.52 ms).
  static __device__ __forceinline__ void add_records(double* acc, uint32_t slot, uint32_t shift, const double (&v)[NS],
                                                     unsigned long long has, int lane) {
    if constexpr (NS == 1) {
      if (in_mask(has)) unsafeAtomicAdd(&acc[slot], v[0]);
    } else {
      add_record_of<0>(acc, slot, shift, v, has, lane);
      add_record_of<1>(acc, slot, shift, v, has, lane);
      if constexpr (NS == 4) {
        add_record_of<2>(acc, slot, shift, v, has, lane);
        add_record_of<3>(acc, slot, shift, v, has, lane);
      }
    }
  }
  // the records of the lanes whose number is Q modulo NS (every lane calls)
  template <int Q>
  static __device__ __forceinline__ void add_record_of(double* acc, uint32_t slot, uint32_t shift, const double (&v)[NS],
                                                       unsigned long long has, int lane) {
    // quad permutation: each lane reads the Q-th of its NS lanes
    static constexpr int kFrom = NS == 4 ? Q * 0x55 : (Q | Q << 2 | (2 + Q) << 4 | (2 + Q) << 6);
    auto from = [](unsigned x) { return (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, kFrom, 0xf, 0xf, false); };
    const unsigned c = (unsigned)lane & (NS - 1u);
    double w = 0.0;
#pragma unroll
    for (unsigned k = 0; k < NS; ++k) {
      const unsigned long long u = __double_as_longlong(v[k]);
      const double x = __longlong_as_double(((unsigned long long)from((unsigned)(u >> 32)) << 32) | from((unsigned)u));
      w = k == c ? x : w;
    }
    // (All of them are read before any branch: a lane reads nothing from one that is not
    // active. And it reads how many sums there are, not the shift: folded into
    // v_lshrrev_b32_dpp, the permutation reached the number that is shifted.)
    const unsigned at = from(slot) + c, sums = from(1u << shift), owner = from(in_mask(has) ? 1u : 0u);
    if (owner != 0u && c < sums) unsafeAtomicAdd(&acc[at], w);
  }
  // v[c] belongs to the lane's problem where c < 2^shift
  __device__ __forceinline__ void add(double* acc, Probe& p, uint32_t slot, uint32_t shift, const double (&v)[NS],
                                      unsigned long long has, int lane) {
    auto to_memory = [&]() {
#pragma unroll
      for (int c = 0; c < NS; ++c)
        if (c == 0 || (c >> shift) == 0) unsafeAtomicAdd(&acc[slot + c], v[c]);
    };
    if constexpr (!CACHE) {
      add_records(acc, slot, shift, v, has, lane);
      return;
    }
    if (p.moved) {
      const int n = __popcll(p.moved);
      int i0 = 0;
      for (; i0 + 8 < n; i0 += 8) {
        take(acc, p, 8, lane);
        keep(p, lane);
        p.listed = moves[first / (kLines / kWave) + i0 + 8 + (lane >> 3)];
      }
      take(acc, p, n - i0, lane);
    }
    const unsigned long long mine = has & wave_mask(p.owner == slot >> 3);
    // (a record is aligned to its length, so its sums are places apart by XOR)
    const uint32_t place = line_place(p.h, slot);
    if (in_mask(mine)) {
#pragma unroll
      for (int c = 0; c < NS; ++c)
        if (c == 0 || (c >> shift) == 0)
          __hip_atomic_fetch_add(at(place ^ (8u * c)), v[c], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
    __builtin_amdgcn_wave_barrier();
    const unsigned long long lost = has & ~mine;
    if (lost) {
      if (in_mask(lost)) to_memory();
    }
  }
  __device__ void flush(double* acc, int lane) {
    if constexpr (CACHE) {
      drain(acc, lane);
      for (int j = lane; j < 8 * kLines; j += kWave) {
        const uint32_t h = first + (uint32_t)(j >> 3), line = key[h];
        if (line != kNoSlot) add_line(acc, line, j & 7, *at(line_place(h, j)));
      }
    }
  }
};

// The rays of a wave that split go to the wave's current segment of the next
// level's queue (its home segment at first) through blocks of slots it reserves
// with one atomic, in coalesced stores. They wait in their idle lanes until the
// wave refills and are written then, all at once and in the order they started (lane_pos): 64 rays that
// started as neighbouring pixels leave their children as neighbouring pixels,
// whatever order they split in, so that a wave's rays stay a compact patch of the
// sphere from level to level (written in the order of their splits, 16 or 32 at
// a time, every level spread a wave's rays over several times the area, and the
// deposit cache's lines with them). A slot holds the split ray; its four
// children are formed when they are claimed, a quarter of the bytes. A segment
// that is full sends the wave on to the next one, so the splits of a few
// neighbouring pixel ranges (the rays towards a grid's corners, say) can fill one
// segment without losing children while the queue has room elsewhere; only when
// every segment is full are children lost (an overflow, which the host answers
// by tracing in smaller chunks).
template <typename R, int NG, bool THIN>
struct SplitWriter {
  int wseg;                                     // segment of the wave's current reservation
  unsigned long long o_next, o_end;             // the wave's reserved slots of segment wseg

  __device__ void init(int home) {
    wseg = home;
    o_next = o_end = 0;
  }
  // the lanes with `split` (all lanes call)
  __device__ void write(const TraceArgs<R>& a, const Ray<R, NG>& L, bool split, int lane) {
    const unsigned long long mask = pos_mask(split);
    const int need = __popcll(mask);
    const int rank = __popcll(mask & bits_below(lane_pos(lane)));
    int done = 0;
    int full = 0;                                           // segments found full in this call
    while (done < need) {
      if (o_next >= o_end) {
        const unsigned long long want = (unsigned long long)(need - done);
        const unsigned long long grab = want > a.reserve ? want : a.reserve;
        unsigned long long fresh = 0;
        if (lane == 0) fresh = atomicAdd(&a.ctr->count[a.cout][wseg], grab);
        fresh = lane0_64(fresh);
        if (fresh >= a.seg_cap) {
          if (++full >= a.nseg) break;                      // every segment is full
          wseg = (wseg + 1) & (a.nseg - 1);
          continue;
        }
        o_next = fresh;
        o_end = fresh + grab < a.seg_cap ? fresh + grab : a.seg_cap;
      }
      const unsigned long long room = o_end - o_next;
      const int n = (unsigned long long)(need - done) < room ? need - done : (int)room;
      if (split && rank >= done && rank < done + n) {
        const unsigned long long slot = (unsigned long long)wseg * a.seg_cap + o_next + (unsigned)(rank - done);
        a.out.pix[slot] = L.pix;
        a.out.tree[slot] = L.tree;
        a.out.r[slot] = L.g.r;
        // a thin ray's record carries its remaining column as -4 (1 + rem), an ended group a negative rate
        if constexpr (THIN) {
          a.out.P[slot] = L.thin ? -4.0 * (1.0 + L.rem) : L.P[0];
        } else {
#pragma unroll
          for (int g = 0; g < NG; ++g) a.out.P[g * a.out.pstride + slot] = NG == 1 || L.alive[g] ? L.P[g] : -1.0;
        }
      }
      o_next += (unsigned long long)n;
      done += n;
    }
    if (done < need && lane == 0) atomicOr(&a.ctr->err, kErrOverflow);
  }
  // all lanes of the wave, at its end: the unused slots of its last
  // reservation become empty slots
  __device__ void close(const TraceArgs<R>& a, int lane) const {
    for (unsigned long long i = o_next + lane; i < o_end; i += kWave)
      a.out.tree[(unsigned long long)wseg * a.seg_cap + i] = kNoTree;
  }
};

// Time-dependent rays: the halted rays of a wave take consecutive records of its
// reserved block of the halt list, and of new blocks (one atomic per kHaltBlock
// records) once that is full: a counter every wave of the device shares is not
// touched at every halt. Written when the wave refills, like the split rays.
template <typename R, int NG>
struct HaltWriter {
  unsigned long long h_next, h_end, h_count;   // reserved records, rays halted in this launch
  double held;                                 // the lane's: photons they hold
  int place;                                   // of Counters::halted

  __device__ void init(int home) {
    h_next = h_end = h_count = 0;
    held = 0.0;
    place = home % kHaltSpread;
  }
  // the lanes with `halt` (all lanes call)
  __device__ void write(const TraceArgs<R>& a, const Ray<R, NG>& L, bool halt, int lane) {
    const unsigned long long hm = pos_mask(halt);
    if (!hm) return;
    const unsigned long long n = (unsigned long long)__popcll(hm);
    const unsigned long long room = h_end - h_next;
    unsigned long long nb = 0;
    if (n > room) {
      if (lane == 0) nb = atomicAdd(&a.ctr->halt_count, (unsigned long long)kHaltBlock);
      nb = lane0_64(nb);
    }
    if (halt) {
      const unsigned long long rank = (unsigned long long)__popcll(hm & bits_below(lane_pos(lane)));
      const unsigned long long i = rank < room ? h_next + rank : nb + (rank - room);
      if (i < a.halt_cap) {
        a.halt.pix[i] = L.pix >> (2 * L.more);
        a.halt.tree[i] = L.tree;
        a.halt.r[i] = L.g.r;
#pragma unroll
        for (int g = 0; g < NG; ++g) {
          const bool live = NG == 1 || L.alive[g];
          a.halt.P[g * a.halt.pstride + i] = live ? L.P[g] : -1.0;
          held += live ? L.P[g] : 0.0;
        }
        a.halt_lev[i] = a.gen - L.more;
        if (L.more) atomicAdd(&a.ctr->halted[a.gen - L.more][place].rays, 1ull);
      } else {
        atomicOr(&a.ctr->err, kErrOverflow);
      }
    }
    if (n > room) {
      h_next = nb + (n - room);
      h_end = nb + (unsigned long long)kHaltBlock;
    } else {
      h_next += n;
    }
    h_count += (unsigned long long)__popcll(wave_mask(halt && L.more == 0));
  }
  // the unfilled rest of the wave's last block: empty records (no photons,
  // a level above every real one); the level's count once per wave
  __device__ void close(const TraceArgs<R>& a, int lane) const {
    for (unsigned long long i = h_next + lane; i < h_end; i += kWave)
      if (i < a.halt_cap) {
        a.halt.pix[i] = 0;
        a.halt.tree[i] = 0;
        a.halt.r[i] = 0.0;
#pragma unroll
        for (int g = 0; g < NG; ++g) a.halt.P[g * a.halt.pstride + i] = 0.0;
        a.halt_lev[i] = kHaltHole;
      }
    const double sum = wave_total(held);
    if (lane == kWave - 1 && sum > 0.0) unsafeAtomicAdd(&a.ctr->halted[a.gen][place].P, sum);
    if (lane == 0 && h_count) atomicAdd(&a.ctr->halted[a.gen][place].rays, h_count);
  }
};

// Waves per SIMD the register budget is set for: three (at most 168 VGPRs),
// which the LDS of a block (four waves) also allows.
//
// NG: energy groups a ray carries (its tree's pack is at most that; the
// radiation-pressure and optically-thin variants carry one). With NG > 1 a
// deposit has two sums, the absorbed rate and its energy moment over the
// groups. Groups share all of the geometry, the split test and the deposit's
// LDS combining, so a step's cost per group is its optical depth, exponential
// and photon rate alone; a group no lane of the wave still carries is skipped.
// Traced one group per ray, the 128^3 workload (16 sources, 4 groups) made 895
// million steps in neutral gas and 2.3 billion in ionised gas; carrying the
// four groups together makes 580 million of either.
template <typename R, bool CACHE, int PHYS, int NG>
__global__ __launch_bounds__(kTraceBlock) __attribute__((amdgpu_waves_per_eu(sizeof(R) == 8 && NG > 2 ? 2 : 3)))
void trace_level_kernel(TraceArgs<R> a) {
  constexpr bool COVER = (PHYS & kPhysCover) != 0, RADP = (PHYS & kPhysRadp) != 0, HALT = (PHYS & kPhysHalt) != 0;
  constexpr bool THIN = (PHYS & kPhysThin) != 0;
  static_assert(!(THIN && (RADP || HALT)), "the optically-thin approximation is a single-pass option");
  static_assert(NG == 1 || !(THIN || RADP), "these variants carry one group per ray");
  constexpr int NS = RADP ? 4 : (NG > 1 ? 2 : 1);
  const int lane = threadIdx.x & (kWave - 1);
  const int pos = lane_pos(lane);
  if (__hip_atomic_load(&a.ctr->err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & kErrBadInput) return;   // set before this launch: the whole grid
  const int K = a.nseg;                      // a power of two
  const int kshift = __ffs(K) - 1;
  const unsigned long long npix = 12ull << (2 * a.seed_level);
  // rays of the launch that are not children: resumed ones (time-dependent rays), then seeds
  const unsigned long long n_held = HALT ? a.n_held : 0ull;
  const unsigned long long n_extra = n_held + (unsigned long long)(a.seed_end - a.seed_begin) * npix;
  Counters::Head* head_in = a.ctr->head[a.cin];
  // The level's rays in units of `span`: those of each segment's children, then
  // the others. A unit is the launch's setting; of a level that holds no more than
  // one for every wave of the launch each wave gets an equal share, in whole rays
  // per lane (ragged float64 1.10 -> 0.91 ms against units halved until they were
  // enough, of which some waves got two). Wave `rank`
  // of the launch starts with its share of the first `fixed` units (at most one),
  // which takes no atomic; the others are claimed one by one from K equal parts of
  // them. Claimed from the first ray on, the 3072 waves of a launch queued up at
  // the counters of a small level: 5 to 50 us of the 35 to 90 a level took (a
  // 32^3 source 173 -> 107 us, 20 steps of a 64^3 front 4.1 -> 3.1 ms).
  __shared__ struct Level {
    unsigned first[kSegMax], rays[kSegMax];  // of each segment: its first unit, its rays
    unsigned children, fixed, open, span;    // units of children; units dealt at the start; the others; rays of one
  } lev;                                     // (all waves store the same values)
  const unsigned waves = gridDim.x * (kTraceBlock / kWave);
  // the blocks of one XCD (every eighth) have consecutive ranks: their rays, and
  // those that split from them, stay on it
  const unsigned blk = (gridDim.x & 7u) ? blockIdx.x : (blockIdx.x & 7u) * (gridDim.x >> 3) + (blockIdx.x >> 3);
  const unsigned rank = blk * (kTraceBlock / kWave) + wave_in_block();
  unsigned u_next, u_end;                    // the units the wave has claimed
  {
    // (32 bits hold a segment: 64 of 2^30 slots would be terabytes)
    const unsigned rays = lane < K ? (unsigned)(4ull * min(a.ctr->count[a.cin][lane], a.seg_cap)) : 0u;
    unsigned long long all = rays;
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) {
      const unsigned lo = __shfl_xor((unsigned)all, o), hi = __shfl_xor((unsigned)(all >> 32), o);
      all += ((unsigned long long)hi << 32) | lo;
    }
    all = uniform64(all) + n_extra;
    if (all == 0) return;                    // a level no ray reached (the host launches all it may need)
    const unsigned span = unit_rays(all, (unsigned)a.chunk, waves);
    unsigned upto = (rays + span - 1) / span;
    const unsigned mine = upto;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
      const unsigned before = __shfl_up(upto, o);
      upto += lane >= o ? before : 0u;
    }
    const unsigned children = __builtin_amdgcn_readlane(upto, kWave - 1);
    const unsigned units = children + (unsigned)((n_extra + span - 1) / span);
    const unsigned fixed = min(units, waves);
    lev.first[lane] = upto - mine;
    lev.rays[lane] = rays;
    lev.children = children;
    lev.fixed = fixed;
    lev.open = units - fixed;
    lev.span = span;
    const double share = (double)fixed / (double)waves;
    u_next = uniform32((int)(share * (double)rank));
    u_end = rank + 1 == waves ? fixed : uniform32((int)(share * (double)(rank + 1)));
  }
  // the segment the wave writes its splits to first, and the part it claims from first
  const int home = (int)(((unsigned long long)rank * (unsigned)K) / waves);
  const Tracer<R, NG, PHYS> T(a);
  Ray<R, NG> L;
  int ended = -1;          // kind of the lane's ray that ended and is not yet tallied
  WaveTally<NG, THIN> tally;
  tally.init(lane);
  DepositCache<CACHE, NS> cache;
  cache.init(lane);
  SplitWriter<R, NG, THIN> splits;
  splits.init(home);
  bool active = false;
  int again = kFresh;      // an idle lane whose ray goes on in a new frame
  int from = 0;            // the cell it comes from
  unsigned steps = 0;      // of the wave since rays last started or changed grids in it
  L.stat0 = kNoTree;
  L.segs = 0;
  L.pix = 0;
  L.more = 0;
#pragma unroll
  for (int g = 0; g < NG; ++g) {
    L.alive[g] = false;
    L.P[g] = 0.0;
  }
  // the rays the wave takes next, [w_next, w_end): children, by their place in
  // the queue, or resumed rays and seeds
  unsigned long long w_next = 0, w_end = 0;
  bool w_child = false;
  int w_part = home;
  bool drained = false;
  HaltWriter<R, NG> halts;
  if constexpr (HALT) halts.init(home);
  // the step's column pointer, held in vector registers in the float kernels:
  // their scalar registers are full, and from there it was reloaded (a
  // kernel-argument load and lane reads of spilled scalars) at every step; the
  // float64 kernels have no vector registers to spare
  uint64_t kappa_v = (uint64_t)a.kappa;
  if constexpr (sizeof(R) == 4) asm volatile("" : "+v"(kappa_v));
  const __attribute__((address_space(1))) R* const kappa_step = (const __attribute__((address_space(1))) R*)kappa_v;
  // the float kernel with the optically-thin approximation gathers the
  // float64 columns instead (the same values before rounding to float), so
  // that its thin decisions see the optical depth the float64 path sees
  constexpr bool K64 = THIN && sizeof(R) == 4;
  uint64_t kappa64_v = (uint64_t)a.kappa64;
  if constexpr (K64) asm volatile("" : "+v"(kappa64_v));
  const __attribute__((address_space(1))) double* const kappa64_step =
      (const __attribute__((address_space(1))) double*)kappa64_v;

  for (;;) {
    // ---- refill: no lane has a ray in flight ----
    // Every lane whose ray does not go on first gets its queue slot or seed number
    // (from as many units as that takes), then all of them start in one pass; lanes
    // whose slot turns out empty wait for the next refill. A wave that refilled at 24
    // idle lanes kept the state of the others alive through this and wrote their
    // splits out of order: 1.8 to 3 times as long.
    if (wave_mask(ended >= 0)) {
      // (a lane that repeats another's ray reports nothing of it)
      const bool owns = Tracer<R, NG, PHYS>::owner(L);
      splits.write(a, L, ended == 2 && L.more == 0, lane);
      if constexpr (HALT) halts.write(a, L, ended == 3 && owns, lane);
      tally.ended(a.stats, L, owns ? ended : -1, lane);
      if (ended == 2 && L.more > 0) again = kChild;
      ended = -1;
    }
    const unsigned long long going = wave_mask(again != kFresh);
    if (drained && !going) break;
    {
      // no lane holds a ray but those going on, of which this is all that is live
      Ray<R, NG> keep;
      keep.pix = L.pix; keep.more = L.more; keep.tree = L.tree; keep.q = L.q; keep.segs = L.segs; keep.g.r = L.g.r;
#pragma unroll
      for (int g = 0; g < NG; ++g) {
        keep.P[g] = L.P[g];
        keep.alive[g] = L.alive[g];
        keep.cut[g] = L.cut[g];
      }
      if constexpr (THIN) {
        keep.thin = L.thin; keep.rem = L.rem; keep.tsegs = L.tsegs;
      }
      L = keep;
    }
    const unsigned long long crossed = wave_mask(again >= kChild);
    // the lanes that want a ray, in the order they get them (lane_pos)
    unsigned long long left = drained ? 0ull : pos_mask(again == kFresh);
    bool take = false, child = false;
    unsigned long long q = 0;
    while (left) {
      if (w_next >= w_end) {
        if (u_next >= u_end) {
          // Claim a unit: from the wave's current part while it has units
          // left; once it is used up, every lane reads one part's counter
          // (one round trip for all of them), the wave picks the first part
          // with units left after it, and claims there with one atomic; a claim
          // that finds the part used up in the meantime looks again. No
          // part with units left: the level is drained.
          const unsigned open = (unsigned)uniform32((int)lev.open);
          auto part = [&](unsigned p) { return (unsigned)(((unsigned long long)p * open) >> kshift); };
          auto claim = [&](int p) {
            const unsigned b0 = part((unsigned)p), size = part((unsigned)p + 1u) - b0;
            unsigned long long b = 0;
            if (lane == 0) b = atomicAdd(&head_in[p].n, 1ull);
            b = lane0_64(b);
            if (b >= size) return false;
            u_next = (unsigned)uniform32((int)lev.fixed) + b0 + (unsigned)b;
            u_end = u_next + 1u;
            return true;
          };
          bool got = false;
          while (open != 0) {
            // the current part first: one load while it lasts
            const unsigned long long seen =
                uniform64(__hip_atomic_load(&head_in[w_part].n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
            if (seen < part((unsigned)w_part + 1u) - part((unsigned)w_part) && (got = claim(w_part))) break;
            bool has = false;
            if (lane < K)
              has = __hip_atomic_load(&head_in[lane].n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) <
                    part((unsigned)lane + 1u) - part((unsigned)lane);
            const unsigned long long live = wave_mask(has);
            if (!live) break;
            const unsigned long long ahead = live & (~0ull << w_part);
            w_part = uniform32((int)__ffsll((long long)(ahead ? ahead : live)) - 1);
            if ((got = claim(w_part))) break;
          }
          if (!got) { drained = true; break; }
        }
        const unsigned children = (unsigned)uniform32((int)lev.children), span = (unsigned)uniform32((int)lev.span);
        const unsigned u = u_next++;
        w_child = u < children;
        if (w_child) {
          const int sg = __popcll(wave_mask(lane < K && lev.first[lane] <= u)) - 1;
          const unsigned in = (u - (unsigned)uniform32((int)lev.first[sg])) * span;
          const unsigned long long base = 4ull * (unsigned long long)sg * a.seg_cap;
          w_next = base + in;
          w_end = base + min(in + span, (unsigned)uniform32((int)lev.rays[sg]));
        } else {
          w_next = (unsigned long long)(u - children) * span;
          w_end = min(w_next + span, n_extra);
        }
      }
      const unsigned long long idx = w_next + __popcll(left & bits_below(pos));
      const bool mine = ((left >> pos) & 1ull) && idx < w_end;
      if (mine) {
        take = true;
        child = w_child;
        q = idx;
      }
      const unsigned long long got_mask = pos_mask(mine);
      w_next += __popcll(got_mask);
      left &= ~got_mask;
    }
    if (take || again != kFresh) {
      double r64 = L.g.r;
      if (take) {
        if (child) T.fetch_child(L, q, r64);
        else if (HALT && q < n_held) T.fetch_held(L, q, r64);
        else T.fetch_seed(L, q - n_held, r64);
      }
      if (again == kChild) {
        L.more -= 1;
        if constexpr (THIN) L.tsegs = 0;
#pragma unroll
        for (int g = 0; g < NG; ++g) L.P[g] = L.alive[g] ? 0.25 * L.P[g] : -1.0;
      }
      if (L.tree != kNoTree) {
        const TreeDev& S = a.trees[L.tree];
        T.load_tree(L, S);
        if constexpr (THIN) {
          if (take) T.thin_start(L, S, !child);
        }
        active = T.locate(L, S, r64, again, from, L.q);
        if (!active) ended = 0;            // outside the root grid: escaped
        else if constexpr (K64) L.kap64 = a.kappa64[L.lin];
        else if constexpr (THIN) L.kap64 = (double)L.kap;
        if constexpr (NG > 1) {
#pragma unroll
          for (int g = 0; g < NG; ++g) L.sigma[g] = L.alive[g] ? L.sigma[g] : (R)0;
        }
      }
      again = kFresh;
    }
    if (wave_mask(take) || crossed) steps = 0;
    // the tree of the first ray started is the one the wave's tally follows
    const unsigned long long started = wave_mask(active);
    if (started) tally.follow(a.stats, (uint32_t)__builtin_amdgcn_readlane((int)L.stat0, __ffsll((long long)started) - 1), lane);
    finish_vector_loads();
    // ---- step until the wave refills ----
    // Nothing but the step itself is in this loop: rays that split, end, halt or
    // change frames are marked and dealt with at the refill. What is known of the
    // lanes is kept as wave-uniform masks: a flag carried through the loop per
    // lane is merged with its old value under the execution mask, three scalar
    // instructions a flag and branch.
    unsigned long long run = wave_mask(active);               // lanes with a ray in flight
    unsigned long long at_split = 0, at_end = 0, at_out = 0, at_halt = 0, at_cross = 0;
    unsigned long long carries[NG];                           // lanes whose ray carries group g
#pragma unroll
    for (int g = 0; g < NG; ++g) carries[g] = wave_mask(active && L.alive[g]);
    const unsigned long long root = wave_mask(L.root), owners = wave_mask(active && Tracer<R, NG, PHYS>::owner(L));
    // Steps until the wave must look up: the steps since rays last started or
    // changed grids bound every active ray's own (a bound never reached by a correct trace:
    // cell indices move monotonically), and the mixed mode forms its distances afresh.
    unsigned todo = a.max_steps - steps;
    if constexpr (sizeof(R) == 4) todo = todo < kResync ? todo : kResync;
    const unsigned allowed = todo;
    while (run) {
      // ---- one cell: exit plane, split test, deposit, step ----
      // In every lane; those without a ray compute on values nothing reads.
      typename DepositCache<CACHE, NS>::Probe probe;
      uint32_t slot = NS > 1 || THIN ? L.slot0 + ((uint32_t)L.lin << L.ashift) : L.slot0 + (uint32_t)L.lin;
      // (with the optically-thin approximation only once it is known which rays
      // are thin here: those deposit nothing and would displace lines for it)
      const unsigned long long probed = run & owners;
      if constexpr (!THIN) probe = cache.probe(slot, L.yz, probed);
      const Exit x = L.g.exit();
      const int here = L.lin;                  // (used with the optically-thin approximation alone,
      const uint32_t yz = L.yz;                // whose step is not at its limit)
      const unsigned long long leave = wave_mask(x.t >= L.tbox);
      unsigned long long thin = 0;
      double tc64 = 0.0, rs = L.rs;
      if constexpr (THIN) {
        // optically thin in this cell: the optical depth on leaving it, in
        // float64, below tau_thin
        const double dr64 = x.t - L.g.r;
        tc64 = dr64 > 0.0 ? L.kap64 * dr64 : 0.0;
        const bool thin_here = L.thin && tc64 < L.rem;
        thin = wave_mask(thin_here);
        rs = thin_here ? L.rs_thin : rs;
      }
      const unsigned long long split = run & wave_mask(x.t > rs);
      at_split |= split;
      const unsigned long long go = run & ~split;
      // the segment in this cell, before the step moves the planes
      double dr = x.t - L.g.r, r_end = x.t;
      unsigned long long pos = go & wave_mask(L.g.positive(dr, x.t)), halt = 0;
      if constexpr (HALT) {
        // the ray reaches its halting radius inside this cell: the segment ends there
        const bool halts_here = x.t > L.rhalt;
        halt = go & wave_mask(halts_here);
        r_end = halts_here ? L.rhalt : r_end;
        dr = halts_here ? L.rhalt - L.g.r : dr;
        pos = (pos & ~halt) | (halt & wave_mask(dr > 0.0));
      }
      double fc = 1.0;
      if constexpr (COVER) {
        if (in_mask(pos) && L.lpix > 0.0) fc = T.covering_factor(L, dr);
      }
      unsigned long long own = 0;              // thin: the cell holds the source
      if constexpr (THIN) {
        bool o = false;
        if (in_mask(pos & thin)) o = T.holds_source(L);
        own = wave_mask(o);
      }
      // across the exit face; the next cell's column is gathered now, under the
      // deposit and its combining (a ray that leaves its grid reads cell 0 of the
      // batch, unused)
      L.g.step(x, L.st, L.sy, L.sz, L.lin, L.yz);
      R kpre = (R)0;
      double kpre64 = 0.0;
      R col = L.kap * (R)dr;
      col = in_mask(pos) ? col : (R)0;
      const unsigned next = in_mask(go & ~leave) ? (unsigned)L.lin : 0u;
      if constexpr (K64) {
        kpre64 = kappa64_step[next];
      } else {
        kpre = kappa_step[next];
      }
      const unsigned long long thinly = pos & thin, dep = ((pos & ~thinly) | (thinly & own)) & owners;
      if constexpr (THIN) {
        slot += in_mask(thinly) ? 1u : 0u;
        probe = cache.probe(slot, yz, dep);
      }
      cache.list(probe, THIN ? dep : probed, lane);
      // groups that fell below their cutoff here (not in a ray that halts here)
      const unsigned long long on = go & ~halt;
      auto cutoff = [&](int g) {
        const unsigned long long low = on & carries[g] & wave_mask(L.P[g] < L.pmin[g]);
        if (low) {
          if (in_mask(low)) {
            L.cut[g] = L.segs;
            L.sigma[g] = (R)0;
          }
          carries[g] &= ~low;
        }
      };
      double v[NS];                            // absorbed rate, then its energy moment or the momentum rate
#pragma unroll
      for (int c = 0; c < NS; ++c) v[c] = 0.0;
      count_where(L.segs, pos);
      if constexpr (THIN) {
        if (in_mask(thinly)) {
          // no photons removed
          double Pc = L.P[0];
          v[0] = absorb(Pc, col * L.sigma[0]);
          // the tree's mark on the cell: a plain byte store (every thin ray
          // of the tree that crosses the cell stores the same 1); a segment
          // shorter than 2^-40 of its exit radius (a ray through an edge or
          // a corner) does not cross the cell
          if (!in_mask(own) && dr > x.t * 0x1p-40) a.mark[L.mark_base + (long long)here] = 1;
          L.rem -= tc64;
          L.tsegs++;
        } else if (in_mask(pos)) {
          v[0] = absorb(L.P[0], col * L.sigma[0]);
          L.thin = false;
        }
        cutoff(0);
      } else {
#pragma unroll
        for (int g = 0; g < NG; ++g) {
          // a lane that does not go on has no column, one without the group no
          // cross-section: both absorb nothing
          if (NG == 1 || (go & carries[g])) {
            const double d = absorb(L.P[g], col * L.sigma[g]);
            v[0] = g == 0 ? d : v[0] + d;
            if constexpr (NG > 1) v[1] = g == 0 ? d * L.eexc[g] : fma(d, L.eexc[g], v[1]);
            cutoff(g);
          }
        }
      }
      if constexpr (RADP) {
        // the momentum rate along the ray, of the absorbed radiation itself, before
        // any covering-factor scaling (zero for a problem that does not ask for it)
        const double m = v[0] * L.mscale;
#pragma unroll
        for (int k = 0; k < 3; ++k) v[1 + k] = m * L.d[k];
      }
      if constexpr (COVER) {
        v[0] *= fc;
        if constexpr (NG > 1) v[1] *= fc;
      }
      max_where(L.g.r, r_end, go);
      unsigned long long any = 0;              // rays with a group left
#pragma unroll
      for (int g = 0; g < NG; ++g) any |= carries[g];
      at_halt |= halt;
      at_end |= on & ~any;
      run = on & any;
      cache.add(a.acc, probe, slot, THIN ? 0u : L.ashift, v, dep, lane);
      // the gather completes here, on every path: left in flight across the
      // loop's back edge it would make the compiler drain the whole counter
      if constexpr (K64) {
        asm volatile("" ::"v"(kpre64));
        kpre = (R)kpre64;
      } else {
        asm volatile("" ::"v"(kpre));
      }
      cache.keep(probe, lane);
      L.kap = kpre;
      if constexpr (THIN) L.kap64 = K64 ? kpre64 : (double)kpre;
      // out of the root grid, or into another frame
      const unsigned long long out = run & leave & root;
      at_out |= out;
      const unsigned long long cross = run & ~out & (leave | wave_mask(kpre < (R)0));
      run &= ~(out | cross);
      if (cross) {
        at_cross |= cross;
        if (in_mask(cross)) {
          again = kCross + x.axis();
          from = L.lin - x.pick(L.st[0], L.st[1], L.st[2]);
        }
      }
      if (--todo == 0) break;
    }
    steps += allowed - todo;
    active = in_mask(run);
    if (in_mask(at_split)) ended = 2;
    if (in_mask(at_end)) ended = 1;
    if (in_mask(at_out)) ended = 0;
    if (in_mask(at_halt)) ended = 3;
#pragma unroll
    for (int g = 0; g < NG; ++g)
      if (in_mask(run | at_split | at_end | at_out | at_halt | at_cross)) L.alive[g] = in_mask(carries[g]);
    if (run && steps >= a.max_steps) {
      if (lane == 0) atomicOr(&a.ctr->err, kErrInternal);
      break;
    }
    if constexpr (sizeof(R) == 4) {
      if (active) {
        // kResync steps: every ray in flight goes on in the same cell, its plane distances formed afresh
        again = kResyncFrame;
        from = L.lin;
        active = false;
      }
    }
  }
  cache.flush(a.acc, lane);
  tally.flush(a.stats, lane);
  if constexpr (HALT) halts.close(a, lane);
  splits.close(a, lane);
}

// ---------------------------------------------------------------------------
// Per-cell kernels
// ---------------------------------------------------------------------------
__device__ __forceinline__ int grid_of(const GridDev* grids, int n_grids, long long cell) {
  int lo = 0, hi = n_grids - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (grids[mid].cell_off <= cell) lo = mid; else hi = mid - 1;
  }
  return lo;
}

__global__ void reset_kernel(Counters* ctr, SgStats* stats, int n_sg) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < kLevels * kSegMax) {
    (&ctr->count[0][0])[i] = 0;
    (&ctr->head[0][0])[i].n = 0;
  }
  if (i == 0) ctr->err = 0;
  if (i < kLevels * kHaltSpread) (&ctr->halted[0][0])[i] = Counters::Halted{0.0, 0ull};
  if (i == 0) ctr->halt_count = 0;
  if (i < n_sg) stats[i] = SgStats{0.0, 0.0, 0ull, 0ull, 0ull, 0ull};
}

__global__ void reset_levels_kernel(Counters* ctr) {
  for (int i = threadIdx.x; i < kLevels * kSegMax; i += blockDim.x) {
    (&ctr->count[0][0])[i] = 0;
    (&ctr->head[0][0])[i].n = 0;
  }
}

// Before a launch of the serving engine: the input queue's claim counters and
// the output queue's write counters start at zero; earlier overflow flags are
// cleared (the host has read them).
__global__ void reset_generation_kernel(Counters* ctr, int cin, int cout) {
  for (int s = threadIdx.x; s < kSegMax; s += blockDim.x) {
    ctr->head[cin][s].n = 0;
    ctr->count[cout][s] = 0;
  }
  if (threadIdx.x == 0) ctr->err &= ~kErrOverflow;
}

__global__ void reset_stats_kernel(SgStats* stats, int first, int count) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < count) stats[first + i] = SgStats{0.0, 0.0, 0ull, 0ull, 0ull, 0ull};
}

// Absorber column per root-cell length, input checks, zeroed accumulators.
// `grids` holds the n_grids grids (grid-table indices grid_base...) whose
// cells fill [cell_begin, cell_end) of the batch-wide numbering.
template <typename R>
__global__ void prep_kernel(const GridDev* __restrict__ grids, int n_grids, int grid_base,
                            const ProblemDev* __restrict__ probs, long long cell_begin, long long cell_end,
                            R* __restrict__ kappa, double* __restrict__ acc, Counters* ctr, uint8_t* __restrict__ mark,
                            long long n_mark, double* __restrict__ kappa64) {
  const long long thread = blockIdx.x * (long long)blockDim.x + threadIdx.x, threads = (long long)gridDim.x * blockDim.x;
  // the marks, 16 bytes a store (a byte per tree of each cell took 170 of 188 us
  // at 128^3 and 64 trees)
  for (long long i = thread; i < n_mark / 16; i += threads) ((uint4*)mark)[i] = make_uint4(0u, 0u, 0u, 0u);
  for (long long i = n_mark / 16 * 16 + thread; i < n_mark; i += threads) mark[i] = 0;
  for (long long c = cell_begin + thread; c < cell_end; c += threads) {
    // the grid of the wave's first cell, which is nearly always every lane's
    const long long c0 = (long long)uniform64((unsigned long long)c);
    int g = grid_of(grids, n_grids, c0);
    if (g + 1 < n_grids && grids[g + 1].cell_off <= c) g = grid_of(grids, n_grids, c);
    const GridDev& G = grids[g];
    const ProblemDev& P = probs[G.problem];
    const long long local = c - G.cell_off;
    const float nh = G.n_h[local], xh = G.x_hi[local];
    if (!(nh >= 0.0f) || !(xh >= 0.0f) || !(xh <= 1.0f) || !isfinite(nh)) atomicOr(&ctr->err, kErrBadInput);
    const double dx_root = G.is_child ? 2.0 * G.dx_cm : G.dx_cm;
    double k64 = (double)nh * (double)xh * dx_root;
    // children follow their root in the grid table
    if (!G.is_child && g + 1 < n_grids && grids[g + 1].is_child && grids[g + 1].problem == G.problem) {
      // a root cell under a child grid carries -(child + 1)
      const int i = (int)(local % G.nx), j = (int)((local / G.nx) % G.ny), kk = (int)(local / ((long long)G.nx * G.ny));
      for (int q = g + 1; q < n_grids && grids[q].is_child && grids[q].problem == G.problem; ++q) {
        const GridDev& C = grids[q];
        if (i >= C.ox && i < C.ox + C.nx / 2 && j >= C.oy && j < C.oy + C.ny / 2 && kk >= C.oz && kk < C.oz + C.nz / 2)
          k64 = (double)(-(grid_base + q + 1));
      }
    }
    kappa[c] = in_range<R>(k64);
    if (kappa64) kappa64[c] = k64;
    const long long base = P.acc_off + P.acc_stride * (c - P.cell_off), gstride = P.acc_stride * P.n_cells;
    if (P.acc_stride == 1) {
      for (int gr = 0; gr < P.acc_planes; ++gr) acc[base + gr * gstride] = 0.0;
    } else {                                       // 2 or 4, in records aligned to their length
      for (int gr = 0; gr < P.acc_planes; ++gr)
        for (int k = 0; k < P.acc_stride; k += 2) *(double2*)(acc + base + gr * gstride + k) = make_double2(0.0, 0.0);
    }
  }
}

// k_ph = sum_g absorbed_g / (n_H x_HI V); heating = sum_g absorbed_g (E_g - E_ion) / (n_H x_HI V);
// with radiation pressure, accel = (absorbed momentum rate) / (m_H n_H V) per component;
// with the optically-thin approximation, the thin deposits in cells that hold a source join the
// absorbed sums of k_ph and heating (not the absorbed total), and every tree marked on the cell
// adds its rate thin_coef / r^2 (r from its source to the cell centre, root cells) to k_ph and
// that times (E_g - E_ion) to the heating (section 2.4, Eq. optthin), whatever n_H x_HI is;
// per-block sums of the absorbed rate (no atomics).
__global__ __launch_bounds__(kFinalBlock) void finalize_kernel(
    const GridDev* __restrict__ grids, const ProblemDev* __restrict__ probs, const FinalBlock* __restrict__ blocks,
    const double* __restrict__ acc, const double* __restrict__ eexc, double* __restrict__ partial,
    const Counters* __restrict__ ctr, const TreeDev* __restrict__ trees, const uint8_t* __restrict__ mark) {
  __shared__ double red[kFinalBlock / kWave];
  if (ctr->err & kErrBadInput) return;
  const FinalBlock B = blocks[blockIdx.x];
  const GridDev& G = grids[B.grid];
  const ProblemDev& P = probs[G.problem];
  const double vol = G.dx_cm * G.dx_cm * G.dx_cm;
  double sum = 0.0;
  for (int t = threadIdx.x; t < B.count; t += kFinalBlock) {
    const long long local = B.first + t;
    const long long c = G.cell_off + local;
    const long long base = P.acc_off + P.acc_stride * (c - P.cell_off), gstride = P.acc_stride * P.n_cells;
    double ab = 0.0, he = 0.0, tab = 0.0, the = 0.0;
    double mom[3] = {0.0, 0.0, 0.0};
    if (P.acc_mode == kAccMoments) {
      ab = acc[base];
      he = acc[base + 1];
    } else {
      for (int gr = 0; gr < P.n_groups; ++gr) {
        const double v = acc[base + gr * gstride];
        ab += v;
        he += v * eexc[P.eexc_off + gr];
        if (P.acc_mode == kAccThin) {
          const double w = acc[base + gr * gstride + 1];
          tab += w;
          the += w * eexc[P.eexc_off + gr];
        }
        if (P.acc_mode == kAccRadp)
          for (int d = 0; d < 3; ++d) mom[d] += acc[base + gr * gstride + 1 + d];
      }
    }
    double kt = 0.0, ht = 0.0;
    if (P.mark_trees > 0) {
      const int i = (int)(local % G.nx), j = (int)((local / G.nx) % G.ny);
      const int kk = (int)(local / ((long long)G.nx * G.ny));
      const double cx = G.is_child ? (double)G.ox + 0.5 * ((double)i + 0.5) : (double)i + 0.5;
      const double cy = G.is_child ? (double)G.oy + 0.5 * ((double)j + 0.5) : (double)j + 0.5;
      const double cz = G.is_child ? (double)G.oz + 0.5 * ((double)kk + 0.5) : (double)kk + 0.5;
      // Eight marks are read at a time, and the groups of a source share the
      // reciprocal of its distance: read one by one under a branch, with a division
      // each, 64 trees took 364 us at 128^3. The quotients are Markstein's (see ratio).
      const uint8_t* at = mark + P.mark_off + (c - P.cell_off);
      double d2 = 0.0, y = 0.0;
      int group = 0;
      bool known = false;                          // d2 and y are those of the current source
      for (int t0 = 0; t0 < P.mark_trees; t0 += 8) {
        uint8_t m[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) m[e] = t0 + e < P.mark_trees ? at[(t0 + e) * P.n_cells] : (uint8_t)0;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          if (t0 + e >= P.mark_trees) break;
          if (group == 0) known = false;
          if (wave_mask(m[e] != 0)) {
            const TreeDev& S = trees[P.tree_first + t0 + e];
            if (!known) {
              const double dx0 = cx - S.sx, dx1 = cy - S.sy, dx2 = cz - S.sz;
              d2 = dx0 * dx0 + dx1 * dx1 + dx2 * dx2;
              y = reciprocal(d2);
              known = true;
            }
            const double q = S.thin_coef * y, kv = m[e] ? fma(fma(-d2, q, S.thin_coef), y, q) : 0.0;
            kt += kv;
            ht += kv * eexc[P.eexc_off + group];
          }
          if (++group == P.n_groups) group = 0;
        }
      }
    }
    const double nabs = (double)G.n_h[local] * (double)G.x_hi[local];
    double k = kt, h = ht;
    if (nabs > 0.0) {
      k = (ab + tab) / (nabs * vol) + kt;
      h = (he + the) / (nabs * vol) + ht;
    }
    G.out_kph[local] = k;
    G.out_heat[local] = h;
    if (P.acc_mode == kAccRadp && G.out_acc) {
      const double rho = kHydrogenMassG * (double)G.n_h[local];
      for (int d = 0; d < 3; ++d) G.out_acc[d * P.n_cells + local] = rho > 0.0 ? mom[d] / (rho * vol) : 0.0;
    }
    sum += ab;
  }
  for (int off = kWave / 2; off > 0; off >>= 1) sum += __shfl_down(sum, off);
  if ((threadIdx.x & (kWave - 1)) == 0) red[threadIdx.x / kWave] = sum;
  __syncthreads();
  if (threadIdx.x == 0) {
    double s = 0.0;
    for (int w = 0; w < kFinalBlock / kWave; ++w) s += red[w];
    partial[blockIdx.x] = s;
  }
}

// ---------------------------------------------------------------------------
// Host-side launchers (called by the runtime on its stream).
// ---------------------------------------------------------------------------
hipError_t launch_reset(hipStream_t s, Counters* ctr, SgStats* stats, int n_sg) {
  const int n = n_sg > kLevels * kSegMax ? n_sg : kLevels * kSegMax;
  const int blocks = n / 256 + 1;
  hipLaunchKernelGGL(reset_kernel, dim3(blocks), dim3(256), 0, s, ctr, stats, n_sg);
  return hipGetLastError();
}

hipError_t launch_reset_generation(hipStream_t s, Counters* ctr, int cin, int cout) {
  hipLaunchKernelGGL(reset_generation_kernel, dim3(1), dim3(kSegMax), 0, s, ctr, cin, cout);
  return hipGetLastError();
}

hipError_t launch_reset_stats(hipStream_t s, SgStats* stats, int first, int count) {
  if (count < 1) return hipSuccess;
  hipLaunchKernelGGL(reset_stats_kernel, dim3((count + 255) / 256), dim3(256), 0, s, stats, first, count);
  return hipGetLastError();
}

hipError_t launch_reset_levels(hipStream_t s, Counters* ctr) {
  hipLaunchKernelGGL(reset_levels_kernel, dim3(1), dim3(256), 0, s, ctr);
  return hipGetLastError();
}

template <typename R>
hipError_t launch_prep(hipStream_t s, int num_cu, const GridDev* grids, int n_grids, int grid_base,
                       const ProblemDev* probs, long long cell_begin, long long cell_end, R* kappa, double* acc,
                       Counters* ctr, uint8_t* mark, long long n_mark, double* kappa64) {
  long long blocks = (cell_end - cell_begin + 255) / 256;
  if (blocks > 32LL * num_cu) blocks = 32LL * num_cu;
  if (blocks < 1) blocks = 1;
  hipLaunchKernelGGL(prep_kernel<R>, dim3((unsigned)blocks), dim3(256), 0, s, grids, n_grids, grid_base, probs,
                     cell_begin, cell_end, kappa, acc, ctr, mark, n_mark, kappa64);
  return hipGetLastError();
}

// Blocks per CU a kernel can keep resident.
template <typename K>
static int resident_blocks(K kernel) {
  int n = 0;
  return hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, kernel, kTraceBlock, 0) == hipSuccess && n > 0 ? n : 1;
}

// `blocks` is what the context asks for, at most what the plain kernel keeps
// resident. A variant may keep fewer: the float64 kernels for three or four groups
// run at two waves a SIMD (200 to 220 VGPRs), the plain one at three.
template <typename R, int PHYS, int NG, bool CACHE>
static void launch_as(hipStream_t s, int num_cu, int blocks, const TraceArgs<R>& args) {
  static const int per_cu = resident_blocks(trace_level_kernel<R, CACHE, PHYS, NG>);    // looked up once per kernel
  blocks = launch_blocks(blocks, per_cu, num_cu);
  hipLaunchKernelGGL((trace_level_kernel<R, CACHE, PHYS, NG>), dim3(blocks), dim3(kTraceBlock), 0, s, args);
}
template <typename R, int PHYS, int NG>
static void launch_one(hipStream_t s, int num_cu, int blocks, const TraceArgs<R>& args, bool cache) {
  if (cache) launch_as<R, PHYS, NG, true>(s, num_cu, blocks, args);
  else launch_as<R, PHYS, NG, false>(s, num_cu, blocks, args);
}

// `width`: the widest pack of the launch's trees; 3 takes the kernel for 4 (the
// fourth group is never alive, which skips it)
template <typename R, int PHYS>
static void launch_phys(hipStream_t s, int num_cu, int blocks, const TraceArgs<R>& args, bool cache, int width) {
  if (width <= 1) launch_one<R, PHYS, 1>(s, num_cu, blocks, args, cache);
  else if (width == 2) launch_one<R, PHYS, 2>(s, num_cu, blocks, args, cache);
  else launch_one<R, PHYS, 4>(s, num_cu, blocks, args, cache);
}

template <typename R>
hipError_t launch_trace_level(hipStream_t s, int num_cu, int blocks, const TraceArgs<R>& args, bool cache, int width,
                              bool cover, bool radp, bool thin) {
  if ((thin && radp) || ((thin || radp) && width > 1) || width > kPack) return hipErrorInvalidValue;
  if (thin && cover) launch_one<R, kPhysThin | kPhysCover, 1>(s, num_cu, blocks, args, cache);
  else if (thin) launch_one<R, kPhysThin, 1>(s, num_cu, blocks, args, cache);
  else if (cover && radp) launch_one<R, kPhysCover | kPhysRadp, 1>(s, num_cu, blocks, args, cache);
  else if (radp) launch_one<R, kPhysRadp, 1>(s, num_cu, blocks, args, cache);
  else if (cover) launch_phys<R, kPhysCover>(s, num_cu, blocks, args, cache, width);
  else launch_phys<R, 0>(s, num_cu, blocks, args, cache, width);
  return hipGetLastError();
}

template <typename R>
hipError_t launch_trace_level_halt(hipStream_t s, int num_cu, int blocks, const TraceArgs<R>& args, bool cache, int width) {
  if (width > kPack) return hipErrorInvalidValue;
  launch_phys<R, kPhysHalt>(s, num_cu, blocks, args, cache, width);
  return hipGetLastError();
}

// Serving: rays of removed problems leave the queue between two launches.
// Block b walks segment b % nseg (blocks share a segment by their quotient)
// over its written slots and empties every record whose tree index lies in
// one of the n ranges [lo[i], hi[i]).
struct DropRanges {
  int n;
  int lo[kDropRanges], hi[kDropRanges];
};

__global__ __launch_bounds__(256) void drop_trees_kernel(uint32_t* __restrict__ tree, const Counters* __restrict__ ctr,
                                                         int row, unsigned long long seg_cap, int nseg, DropRanges r) {
  const int seg = (int)(blockIdx.x % (unsigned)nseg);
  const unsigned long long part = blockIdx.x / (unsigned)nseg, parts = gridDim.x / (unsigned)nseg;
  const unsigned long long cnt = ctr->count[row][seg] < seg_cap ? ctr->count[row][seg] : seg_cap;
  uint32_t* q = tree + (unsigned long long)seg * seg_cap;
  for (unsigned long long i = part * 256ull + threadIdx.x; i < cnt; i += parts * 256ull) {
    const uint32_t t = q[i];
    bool drop = false;
    for (int k = 0; k < r.n; ++k) drop = drop || ((int)t >= r.lo[k] && (int)t < r.hi[k]);
    if (t != kNoTree && drop) q[i] = kNoTree;
  }
}

hipError_t launch_drop_trees(hipStream_t s, uint32_t* tree, const Counters* ctr, int row, unsigned long long seg_cap,
                             int nseg, const int* lo, const int* hi, int n) {
  if (n <= 0) return hipSuccess;
  if (n > kDropRanges || nseg < 1) return hipErrorInvalidValue;
  DropRanges r{};
  r.n = n;
  for (int k = 0; k < n; ++k) {
    r.lo[k] = lo[k];
    r.hi[k] = hi[k];
  }
  hipLaunchKernelGGL(drop_trees_kernel, dim3((unsigned)nseg * 16u), dim3(256), 0, s, tree, ctr, row, seg_cap, nseg, r);
  return hipGetLastError();
}

hipError_t launch_finalize(hipStream_t s, int n_blocks, const GridDev* grids, const ProblemDev* probs,
                           const FinalBlock* blocks, const double* acc, const double* eexc, double* partial,
                           const Counters* ctr, const TreeDev* trees, const uint8_t* mark) {
  if (n_blocks < 1) return hipSuccess;
  hipLaunchKernelGGL(finalize_kernel, dim3(n_blocks), dim3(kFinalBlock), 0, s, grids, probs, blocks, acc, eexc,
                     partial, ctr, trees, mark);
  return hipGetLastError();
}

template hipError_t launch_prep<float>(hipStream_t, int, const GridDev*, int, int, const ProblemDev*, long long,
                                       long long, float*, double*, Counters*, uint8_t*, long long, double*);
template hipError_t launch_prep<double>(hipStream_t, int, const GridDev*, int, int, const ProblemDev*, long long,
                                        long long, double*, double*, Counters*, uint8_t*, long long, double*);
template hipError_t launch_trace_level<float>(hipStream_t, int, int, const TraceArgs<float>&, bool, int, bool, bool, bool);
template hipError_t launch_trace_level<double>(hipStream_t, int, int, const TraceArgs<double>&, bool, int, bool, bool, bool);
template hipError_t launch_trace_level_halt<float>(hipStream_t, int, int, const TraceArgs<float>&, bool, int);
template hipError_t launch_trace_level_halt<double>(hipStream_t, int, int, const TraceArgs<double>&, bool, int);

hipError_t trace_occupancy(int precision, bool cache, int* blocks_per_cu) {
  auto ask = [&](auto kernel) {
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks_per_cu, kernel, kTraceBlock, 0);
  };
  if (precision == 0)
    return cache ? ask(trace_level_kernel<double, true, 0, 1>) : ask(trace_level_kernel<double, false, 0, 1>);
  return cache ? ask(trace_level_kernel<float, true, 0, 1>) : ask(trace_level_kernel<float, false, 0, 1>);
}

}  // namespace moray
