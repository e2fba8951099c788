// Box 12: transport (Sect. 3.4, 3.5.1).
//   12a  left/right momenta Pi- = rho m(v_{i-1/2}), Pi+ = rho m(v_{i+1/2})
//        with the factors m of Tab. "momenta" (Eqs. 16, 17).  They are formed
//        on the fly by the Y sweep, which reads the state directly.
//   12b/c directional finite-volume updates in the order Y, Z, X: van Leer
//        slopes (harmonic mean of the one-sided differences per unit length,
//        zero unless of equal sign), interface value at half step upwinded on
//        the face velocity (Eqs. 14, 15), mass flux w rho* S dt (Eq. flux),
//        consistent transport (Q/rho interpolated, flux q* F_rho).  The Y
//        sweep also covers the two nearest ghost rows of each Z side, which
//        the Z sweep reads next.  The X sweep of each ring uses the residual
//        velocity v_x - v0 (Eq. fargo1); it is followed by the circular shift
//        by N zones (Eq. 32) and the PPA fractional residual (Eqs. 33-36);
//        both act identically on every zone of a ring, so the shift is applied
//        when the ring is stored.
//   12d  velocities from the transported momenta (Eq. 18): v_x, and on 2D
//        meshes v_y, by the pass that transports along X, v_y and v_z of 3D
//        meshes by a final pass.
//
// The Y sweep and, in the pass that it shares with the X transport, the Z sweep
// are column sweeps: a thread walks a chunk of one column with a sliding window
// of three zones in registers, so that every value is loaded once and every face
// flux and slope is computed once.
//
// The field type F is double, or float for the FP32-bulk state; the arithmetic
// of a kernel is carried out in F (per-ring constants such as dt/dX and the
// PPA residual xi are formed in FP64 and rounded to F).  In FP32, v_x and the
// X momenta are deviations from a per-ring FP64 background (v_x - vb and
// rho R (v_x - vb)): the Y and Z sweeps add the background's increments
// between rings (column_sweep), the X transport, where it is constant, needs
// nothing, and 12d forms the deviation again.
#include <type_traits>

#include "fargo_internal.h"

namespace fargo {

namespace {

// Reciprocal and quotient for the ring kernel, which is bound by its vector
// instruction count: the hardware reciprocal estimate r refined by the series
// of 1 / (d r) = 1 + e + e^2 + ..., e = 1 - d r.  In FP64 (e some 2^-23) two
// terms, three fused operations; in FP32 one, two operations.  That leaves the
// result within about one unit in the last place (the correctly rounded
// division costs more than twice the instructions), rounded differently from
// zone to zone like a division.  d must be a normal number; a zero or denormal
// d, which the kernel only meets in discarded selects and halo lanes, gives an
// infinite or meaningless value and no trap.
__device__ inline double ring_rcp(double d) {
  const double r = __builtin_amdgcn_rcp(d), e = fma(-d, r, 1.0);
  return fma(r, fma(e, e, e), r);
}
__device__ inline double ring_div(double n, double d) {
  const double r = __builtin_amdgcn_rcp(d), e = fma(-d, r, 1.0), q = n * r;
  return fma(q, fma(e, e, e), q);
}
__device__ inline float ring_rcp(float d) {
  const float r = __builtin_amdgcn_rcpf(d);
  return fmaf(r, fmaf(-d, r, 1.0f), r);
}
__device__ inline float ring_div(float n, float d) { return n * ring_rcp(d); }
// The quotient of the Y sweep's van Leer slope: correctly rounded in FP64
// (the sweep is bound by memory there), the refined reciprocal in FP32, where
// it is bound by its vector instructions (as the ring kernel and k_zx are)
__device__ inline double sweep_div(double n, double d) { return n / d; }
__device__ inline float sweep_div(float n, float d) { return ring_div(n, d); }

// The product that is a flux: rounded by itself, so that the two zones of a face
// take the same number (contracted into one zone's difference it would not be
// rounded there, and the sum over the zones would drift: the FP32 density of 2048
// x 768 x 96 zones is off by up to 2.9e-7 after 100 steps, against 2.4e-7).  With
// it the FP32 errors after 100 steps are, in the mean square, those of three
// factors multiplied one after the other with a division for each quotient, or
// less (1.33e-9 and 1.34e-9 here); the largest error of one run, a single zone's,
// moves by a tenth with any change of rounding (2.26e-7 with those).
template <typename F>
__device__ inline F flux_of(F a, F b) {
#pragma clang fp contract(off)
  return a * b;
}
// Half the van Leer slope per unit length from the one-sided differences and
// the centre distances below (hm) and above (hp): dl dr/(dl + dr) with
// dl = dm/hm, dr = dp/hp, zero unless dl dr > 0.  b adds, for a quantity stored
// as a deviation from a background that changes from zone to zone, the
// background's increments across the lower and upper face (bm, bp), so that the
// differences are those of the full values.
// Contraction is off in the slopes and their one fused operation is written
// out: a sweep forms the first slope of a chunk of zones before its loop and
// the others inside it, and the same rounding in both places keeps the result
// independent of the chunk size.  DIV: the quotient.
template <class DIV, typename F>
__device__ inline F vl_half(F dm, F dp, F hm, F hp) {
#pragma clang fp contract(off)
  const F pr = dm * dp;
  return pr > F(0) ? DIV::of(pr, fma(dm, hp, dp * hm)) : F(0);
}
template <class DIV, typename F>
__device__ inline F vl_slope(F qm, F q0, F qp, F hm, F hp) {
#pragma clang fp contract(off)
  return vl_half<DIV>(q0 - qm, qp - q0, hm, hp);
}
template <class DIV, typename F>
__device__ inline F vl_slope_b(F qm, F q0, F qp, F hm, F hp, F bm, F bp) {
#pragma clang fp contract(off)
  return vl_half<DIV>((q0 - qm) + bm, (qp - q0) + bp, hm, hp);
}
struct SweepDiv {
  template <typename F>
  __device__ static inline F of(F n, F d) { return sweep_div(n, d); }
};
struct RingDiv {
  template <typename F>
  __device__ static inline F of(F n, F d) { return ring_div(n, d); }
};

// Upwinding at a face with velocity w (Eq. 15): the half-step interface value is
// q + s (L - w dt) from the zone below (width Ll), q - s (L + w dt) from the one
// above (width Lr), with s half the slope; the factors serve every quantity.
template <typename F>
struct Upface {
  bool pos;
  F cl, cr;
  __device__ inline Upface(F w, F dt, F Ll, F Lr) : pos(w >= F(0)), cl(Ll - w * dt), cr(Lr + w * dt) {}
  __device__ inline F star(F ql, F sl, F qr, F sr) const { return pos ? ql + sl * cl : qr - sr * cr; }
};

template <typename F, int NQ>
struct Zone {
  F rho, q[NQ]; // density, Q/rho
  F w;          // velocity on the zone's lower face in the sweep direction
  F e;          // the energy, as loaded
};

// Column sweep over zones [a0, a1) of one column.  `raw(a, RW&)` issues the
// loads of zone a, `derive(a, const RW&, Zone&)` forms its density, Q/rho and
// lower-face velocity, `Tof(a, const Zone&, q)` gives the conserved Q of zone
// a; `geo` gives L(a) (zone width), h(f) (centre distance at face f), S(f),
// Vi(a); `st(a, rho, T[])` stores the updated zone.  The loads of zone f + 3
// are issued while zone f is being computed (two zones of loads in flight,
// measured faster than one on 3D meshes and on the fused batch of 2D disks; the
// two load buffers take turns, so that no copy waits for a load).
// With DEV, quantities 0 and 1 (the X momenta) are deviations from a
// background ell that is constant on a ring (the FP32-bulk state): `dl(f)`
// gives ell(f) - ell(f - 1) at face f.  Slopes take the full differences,
// the interface value is taken relative to the background of the face's
// lower zone, and the update of a zone adds the background carried in
// through its lower face, so that in exact arithmetic the result is the
// full update minus ell times the updated density.
template <typename F, int NQ, bool DEV, class RW, class RAW, class DER, class TOF, class GEO, class ST, class DLF>
__device__ inline void column_sweep(int a0, int a1, F dt, const RAW &raw, const DER &derive, const TOF &Tof,
                                    const GEO &geo, const ST &st, const DLF &dl) {
  Zone<F, NQ> zm, z0, zp;
  RW rn, rn2;
  raw(a0 - 2, rn);
  derive(a0 - 2, rn, zp); // used only for the first slope
  raw(a0 - 1, rn);
  derive(a0 - 1, rn, zm);
  raw(a0, rn);
  derive(a0, rn, z0);
  raw(a0 + 1, rn);
  if (a0 + 2 <= a1 + 1) raw(a0 + 2, rn2);
  F sm[NQ + 1], s0[NQ + 1];
  F dlf = DEV ? dl(a0) : F(0); // background increment at face f
  {
    F hm = geo.h(a0 - 1), hp = geo.h(a0);
    sm[NQ] = vl_slope<SweepDiv>(zp.rho, zm.rho, z0.rho, hm, hp);
#pragma unroll
    for (int q = 0; q < NQ; q++)
      sm[q] = (DEV && q < 2) ? vl_slope_b<SweepDiv>(zp.q[q], zm.q[q], z0.q[q], hm, hp, dl(a0 - 1), dlf)
                             : vl_slope<SweepDiv>(zp.q[q], zm.q[q], z0.q[q], hm, hp);
  }
  F Fp = F(0), FQp[NQ];
#pragma unroll
  for (int q = 0; q < NQ; q++) FQp[q] = F(0);
  F Lm = geo.L(a0 - 1);
  // face f: zone f + 1 from buffer cur, whose loads are then refilled with
  // those of zone f + 3
  auto face = [&](int f, RW &cur) {
    derive(f + 1, cur, zp);
    if (f + 3 <= a1 + 1) raw(f + 3, cur);
    const F dlf1 = DEV ? dl(f + 1) : F(0);
    F hm = geo.h(f), hp = geo.h(f + 1);
    s0[NQ] = vl_slope<SweepDiv>(zm.rho, z0.rho, zp.rho, hm, hp);
#pragma unroll
    for (int q = 0; q < NQ; q++)
      s0[q] = (DEV && q < 2) ? vl_slope_b<SweepDiv>(zm.q[q], z0.q[q], zp.q[q], hm, hp, dlf, dlf1)
                             : vl_slope<SweepDiv>(zm.q[q], z0.q[q], zp.q[q], hm, hp);
    F L0 = geo.L(f);
    F w = z0.w;
    const Upface<F> U(w, dt, Lm, L0);
    F Fr = flux_of(w * U.star(zm.rho, sm[NQ], z0.rho, s0[NQ]) * geo.S(f), dt);
    F FQ[NQ];
#pragma unroll
    for (int q = 0; q < NQ; q++)
      FQ[q] = flux_of(U.star(zm.q[q], sm[q], (DEV && q < 2) ? z0.q[q] + dlf : z0.q[q], s0[q]), Fr);
    if (f > a0) {
      F vi = geo.Vi(f - 1);
      F Tn[NQ];
#pragma unroll
      for (int q = 0; q < NQ; q++) Tn[q] = Tof(f - 1, zm, q) - vi * (FQ[q] - FQp[q]);
      st(f - 1, zm.rho - vi * (Fr - Fp), Tn);
    }
    Fp = Fr;
#pragma unroll
    for (int q = 0; q < NQ; q++) {
      // the flux through face f relative to the background of its upper zone
      FQp[q] = (DEV && q < 2) ? FQ[q] - dlf * Fr : FQ[q];
      sm[q] = s0[q];
    }
    sm[NQ] = s0[NQ];
    zm = z0;
    z0 = zp;
    Lm = L0;
    dlf = dlf1;
  };
#pragma unroll 1
  for (int f = a0; f <= a1; f += 2) {
    face(f, rn);
    if (f + 1 <= a1) face(f + 1, rn2);
  }
}

// ------------------------------------------------------------------------
// Y sweep, forming the momenta from the post-source state (box 12a fused).
// Quantities: Pi-_x, Pi+_x, Pi-_y, Pi+_y [, Pi-_z, Pi+_z] [, e].
// ------------------------------------------------------------------------
template <typename F, int NQ, bool D3, bool ADI>
__device__ __forceinline__ void sweep_y_body(Mesh m, const F *__restrict__ rho, const F *__restrict__ vx,
                                                 const F *__restrict__ vy, const F *__restrict__ vz,
                                                 const F *__restrict__ e, TSetT<F> out,
                                                 const double *__restrict__ dtp, int nchunk, unsigned bid_, unsigned nbk_) {
  const int nrows = D3 ? m.nz + 4 : 1, kbase = D3 ? m.k0 - 2 : 0;
  unsigned Lb = xcd_remap(bid_, nbk_);
  int kr = (int)(Lb % (unsigned)nrows);
  unsigned rest = Lb / (unsigned)nrows;
  int ch = (int)(rest % (unsigned)nchunk), ib = (int)(rest / (unsigned)nchunk);
  int i = ib * (int)blockDim.x + (int)threadIdx.x;
  if (i >= m.nx) return;
  const int k = kbase + kr;
  const int a0 = m.j0 + ch * m.chunk, a1 = min(a0 + m.chunk, m.jn);
  const F dt = (F)*dtp;
  const int ip = i + 1 == m.nx ? 0 : i + 1;
  constexpr bool DEV = sizeof(F) == 4;
  const unsigned pitch = m.pitch, plane = (unsigned)m.plane();
  struct Raw {
    F rho, vx0, vx1, vy0, vy1, vz0, vz1, e;
  };
  auto raw = [&](int a, Raw &z) {
    const unsigned c = m.o32(i, a, k);
    z.rho = rho[c];
    z.vx0 = vx[c];
    z.vx1 = vx[c - i + ip];
    z.vy0 = vy[c];
    z.vy1 = vy[c + pitch];
    if (D3) {
      z.vz0 = vz[c];
      z.vz1 = vz[c + plane];
    }
    if (ADI) z.e = e[c];
  };
  auto derive = [&](int a, const Raw &w, Zone<F, NQ> &z) {
    const F r = w.rho;
    z.rho = r;
    z.w = w.vy0;
    if constexpr (DEV) { // FP32: v_x is a deviation, and so are the X momenta
      z.q[0] = m.mxd(a, k, w.vx0);
      z.q[1] = m.mxd(a, k, w.vx1);
    } else {
      z.q[0] = m.mx(a, k, w.vx0);
      z.q[1] = m.mx(a, k, w.vx1);
    }
    z.q[2] = w.vy0;
    z.q[3] = w.vy1;
    if (D3) {
      z.q[4] = m.mz(a, w.vz0);
      z.q[5] = m.mz(a, w.vz1);
    }
    if (ADI) {
      z.q[NQ - 1] = w.e / r;
      z.e = w.e;
    }
  };
  // the momenta are rho m(v) exactly as formed; e as loaded, carried in the
  // window (read again three rows later, it would come from memory again)
  auto Tof = [&](int, const Zone<F, NQ> &z, int q) {
    if (ADI && q == NQ - 1) return z.e;
    return z.rho * z.q[q];
  };
  struct Geo {
    const Mesh &m;
    int k;
    __device__ F L(int a) const { return (F)m.g.Ly(a); }
    __device__ F h(int f) const { return (F)m.g.hy(f); }
    __device__ F S(int f) const { return (F)m.Sy(f, k); }
    __device__ F Vi(int a) const { return (F)m.Vinv(a, k); }
  } geo{m, k};
  auto st = [&](int a, F r, const F (&T)[NQ]) {
    unsigned c = m.o32(i, a, k);
    out.a[T_RHO][c] = r;
#pragma unroll
    for (int q = 0; q < NQ; q++) out.q[q][c] = T[q];
  };
  auto dl = [&](int f) { return (F)m.bg(BG_DLY, f, k); };
  column_sweep<F, NQ, DEV, Raw>(a0, a1, dt, raw, derive, Tof, geo, st, dl);
}
template <typename F, int NQ, bool D3, bool ADI>
__global__ __launch_bounds__(256) void k_sweep_y(Mesh m, const F *__restrict__ rho, const F *__restrict__ vx,
                                                 const F *__restrict__ vy, const F *__restrict__ vz,
                                                 const F *__restrict__ e, TSetT<F> out,
                                                 const double *__restrict__ dtp, int nchunk) {
  sweep_y_body<F, NQ, D3, ADI>(m, rho, vx, vy, vz, e, out, dtp, nchunk, blockIdx.x, gridDim.x);
}

// ------------------------------------------------------------------------
// X: every wave owns a segment of one ring.  Lane l holds the M consecutive
// zones z0 + M l .. z0 + M l + M - 1 of a window of 64 M zones that starts
// HL zones before the segment and ends HR zones after it; zone neighbours
// come from the lane's own registers or, across lanes, by DPP lane moves.  The
// halo is recomputed instead of exchanged, so no wave waits for another and
// nothing goes through LDS.  The dependency cone of an output zone (van Leer
// residual sweep, PPA residual, 12d along X) spans zones z-6 .. z+5.
// Outputs are written out of place (shifted by N on store), so that the
// segments of a ring can run in any order.
// ------------------------------------------------------------------------
// Zones per lane.  The ring kernel takes two.  (Four in FP32 save lane moves and
// halo, but cost it half its waves: the batch of 256 disks 820 us against 768.)
// The fused Z/X pass, which also holds the window of the Z sweep, takes one in
// FP64 (160 registers, three waves per SIMD; two needed 310, one wave) and two
// in FP32.
constexpr int RING_M = 2;
template <typename F>
constexpr int zx_m() { return sizeof(F) == 8 ? 1 : 2; }
// halo lanes below and above: a zone's result depends on zones z - 6 .. z + 5
constexpr int halo_below(int M) { return (6 + M - 1) / M; } // halo lanes
constexpr int halo_above(int M) { return (5 + M - 1) / M; }

// The differences of neighbouring zones: d[x] between zones x - 1 and x of the
// lane, x = 0 .. M, and the value below the first zone.
template <typename F, int M>
struct Diffs {
  F below, d[M + 1];
  __device__ inline explicit Diffs(const F (&a)[M]) {
    below = from_prev_lane(a[M - 1]);
    d[0] = a[0] - below;
#pragma unroll
    for (int x = 1; x < M; x++) d[x] = a[x] - a[x - 1];
    d[M] = from_next_lane(a[0]) - a[M - 1];
  }
};

template <typename F, int M>
__device__ inline void next_of(const F (&a)[M], F (&out)[M]) { // value of zone z + 1
  const F n1 = from_next_lane(a[0]);
#pragma unroll
  for (int m = 0; m < M; m++) out[m] = m + 1 < M ? a[m + 1] : n1;
}
template <typename F, int M>
__device__ inline void prev_of(const F (&a)[M], F (&out)[M]) { // value of zone z - 1
  const F p1 = from_prev_lane(a[M - 1]);
#pragma unroll
  for (int m = 0; m < M; m++) out[m] = m > 0 ? a[m - 1] : p1;
}

// Interface values on the lane's zones; each zone's slope and each face's
// edge value is computed once and handed to the neighbouring zone (in a
// register, or by a DPP lane move).
//   vlx_faces: van Leer on a uniform zone width, slopes in units of the zone
//   (harmonic mean of the two one-sided differences, zero unless they have
//   the same sign), and the half-step value at each zone's lower face
//   upwinded on w, with cw = w dt / dX (Eq. 15).  The factors 2 of the
//   harmonic mean and 1/2 of the half step cancel (both exact): a holds half a
//   slope, and 1 - cw and 1 + cw, formed once for all quantities, multiply it.
template <typename F, int M>
struct Upwind {
  bool pos[M]; // w >= 0
  F cl[M], cr[M];
  __device__ inline void set(const F (&w)[M], F cdt) {
#pragma unroll
    for (int q = 0; q < M; q++) {
      const F cw = w[q] * cdt;
      pos[q] = w[q] >= F(0);
      cl[q] = F(1) - cw;
      cr[q] = F(1) + cw;
    }
  }
};
template <typename F, int M>
__device__ inline void vlx_faces(const F (&Q)[M], const Upwind<F, M> &U, F (&out)[M]) {
  const Diffs<F, M> D(Q);
  F a[M], ap[M];
#pragma unroll
  for (int q = 0; q < M; q++) {
    const F pr = D.d[q] * D.d[q + 1];
    a[q] = pr > F(0) ? ring_div(pr, D.d[q] + D.d[q + 1]) : F(0);
  }
  prev_of(a, ap);
#pragma unroll
  for (int q = 0; q < M; q++)
    out[q] = U.pos[q] ? (q > 0 ? Q[q > 0 ? q - 1 : 0] : D.below) + ap[q] * U.cl[q] : Q[q] - a[q] * U.cr[q];
}
//   ppa_values (Eqs. 34-36): the interface value that each zone supplies, the
//   mean of its limited parabola over the fraction x = |xi| next to its right
//   edge (RIGHT: xi >= 0) or left edge.  The parabola is held as its edges'
//   distances from the mean, a = q^R - q and b = q - q^L.  With the monotonised
//   slope limited by twice each one-sided difference an edge value lies between
//   its two zones, so away from an extremum a and b have the sign of the slope,
//   and the tests of Eq. 36 (D C > D^2 / 6, -D^2 / 6 > D C with D = a + b, C =
//   (b - a) / 2) read |b| > 2 |a|, |a| > 2 |b|; the steepened edges are b = 2 a
//   and a = 2 b.  The mean over the fraction is then q + (1 - x)(a + x (b - a))
//   on the right, q - (1 - x)(b + x (a - b)) on the left, and q at an extremum.
//   (d is half the slope; scalings by powers of two are exact.)  About two
//   thirds of the operations of the edge values written out.
template <typename F>
struct PpaX {
  F x, omx; // |xi| and 1 - |xi|
  bool right; // xi >= 0
};
template <bool RIGHT, typename F, int M>
__device__ inline void ppa_values(const F (&Q)[M], const PpaX<F> &X, F (&out)[M]) {
  const F third = F(1) / F(3);
  const Diffs<F, M> D(Q);
  F d[M], dp[M], a[M], b[M], low[M];
  bool flat[M];
#pragma unroll
  for (int q = 0; q < M; q++) {
    const F l = D.d[q], r = D.d[q + 1];
    flat[q] = l * r <= F(0);
    const F mag = fmin(fmin(fabs(l), fabs(r)), F(0.25) * fabs(l + r));
    d[q] = flat[q] ? F(0) : copysign(mag, r);
  }
  prev_of(d, dp);
#pragma unroll
  for (int q = 0; q < M; q++) { // the zone's lower face: q - q^L, and q^R - q of the zone below
    const F t = d[q] - dp[q], h = F(0.5) * D.d[q];
    b[q] = h + third * t;
    low[q] = h - third * t;
  }
  next_of(low, a);
#pragma unroll
  for (int q = 0; q < M; q++) {
    const F a2 = a[q] + a[q], b2 = b[q] + b[q];
    const F bl = fabs(b[q]) > fabs(a2) ? a2 : b[q], al = fabs(a[q]) > fabs(b2) ? b2 : a[q];
    const F v = RIGHT ? Q[q] + X.omx * (al + X.x * (bl - al)) : Q[q] - X.omx * (bl + X.x * (al - bl));
    out[q] = flat[q] ? Q[q] : v;
  }
}

// Element i of the row that starts at p, for 0 <= i < 2^31 / sizeof(T): a
// uniform (scalar) row pointer plus a 32-bit byte offset, the addressing mode
// of a global access with a scalar base, which saves the 64-bit address
// arithmetic of every access.
template <typename T>
__device__ inline T *at(T *p, unsigned i) {
  using B = typename std::conditional<std::is_const<T>::value, const char, char>::type;
  return reinterpret_cast<T *>(reinterpret_cast<B *>(p) + i * (unsigned)sizeof(T));
}

// The lane's place in a segment of a ring: its M zones start at window (=
// ring) coordinate zl, iz[] are the ring indices `off` zones before them
// (wrapped into [0, n)), and contig tells whether they are consecutive in
// memory.  Only the lanes outside the halo store, and only zones before the end
// of the segment.
template <typename F, int M_>
struct RingLane {
  static constexpr int M = M_, HLL = halo_below(M), HRL = halo_above(M);
  static constexpr int U = (WAVE - HLL - HRL) * M; // output zones per wave
  int n, lane, zl, aend, iz[M];
  bool contig;
  __device__ inline RingLane(int nx, int seg, int ln, int off = 0) : n(nx), lane(ln) {
    const int a0 = seg * U;      // first output zone of the segment
    zl = a0 - HLL * M + ln * M;  // first zone of the lane
    aend = min(a0 + U, n);
#pragma unroll
    for (int q = 0; q < M; q++) {
      int z = zl + q - off;
      if (n >= WAVE * M) { // the window is no longer than the ring: one wrap at most for it, one for the offset
        z = z < 0 ? z + n : z;
        z = z < 0 ? z + n : (z >= n ? z - n : z);
        iz[q] = z;
      } else {
        const int y = z % n;
        iz[q] = y < 0 ? y + n : y;
      }
    }
    contig = iz[0] + M <= n;
  }
  __device__ inline bool useful(int q) const { return lane >= HLL && lane < WAVE - HRL && zl + q < aend; }
  // the lane's zones of the row that starts at p, one load per zone and no
  // branch on contig (for loads inside a loop)
  __device__ inline void load_each(const F *p, F (&out)[M]) const {
#pragma unroll
    for (int q = 0; q < M; q++) out[q] = *at(p, (unsigned)iz[q]);
  }
  // the lane's zones of the row that starts at p (loads of two elements, at any
  // alignment, where they are consecutive)
  __device__ inline void load(const F *p, F (&out)[M]) const {
    static_assert(M % 2 == 0, "pairs of zones per lane");
    if (contig) {
      using V2 = F __attribute__((ext_vector_type(2), aligned(sizeof(F))));
      const V2 *v = reinterpret_cast<const V2 *>(at(p, (unsigned)iz[0]));
#pragma unroll
      for (int q = 0; q < M / 2; q++) {
        const V2 t = v[q];
        out[2 * q] = t.x;
        out[2 * q + 1] = t.y;
      }
    } else {
#pragma unroll
      for (int q = 0; q < M; q++) out[q] = *at(p, (unsigned)iz[q]);
    }
  }
};

// Where the lane's zones go when the ring is stored shifted by Nm zones: pairs
// (at any alignment) where both zones are wanted and consecutive.  Formed once
// for the quantities of a ring.
template <typename F, int M>
struct RingOut {
  static constexpr int P = M == 1 ? 1 : 2, H = M / P; // zones per store, stores
  unsigned o[H];
  bool one[H], two[H], wrap[H]; // the first zone alone, both at o, the second at the ring's start
  __device__ inline RingOut(const RingLane<F, M> &L, int Nm) {
#pragma unroll
    for (int h = 0; h < H; h++) {
      const int q = P * h;
      int z = L.iz[q] + Nm;
      z = z >= L.n ? z - L.n : z;
      o[h] = (unsigned)z;
      const bool second = P == 2 && L.useful(q + P - 1);
      two[h] = second && z + 1 < L.n;
      wrap[h] = second && !two[h];
      one[h] = L.useful(q) && !two[h];
    }
  }
  __device__ inline void operator()(F *p, const F (&v)[M]) const {
    using V2 = F __attribute__((ext_vector_type(2), aligned(sizeof(F))));
#pragma unroll
    for (int h = 0; h < H; h++) {
      if constexpr (P == 1) {
        if (one[h]) *at(p, o[h]) = v[h];
      } else if (two[h]) {
        *reinterpret_cast<V2 *>(at(p, o[h])) = V2{v[2 * h], v[2 * h + 1]};
      } else if (one[h]) {
        *at(p, o[h]) = v[2 * h];
        if (wrap[h]) *at(p, 0u) = v[2 * h + 1];
      }
    }
  }
};

// as the fused Z/X pass stores: the momenta into Tout
template <typename F, int M>
struct RingShift : RingOut<F, M> {
  const TSetT<F> &T;
  __device__ inline RingShift(const RingLane<F, M> &L, int Nm, const TSetT<F> &Tout) : RingOut<F, M>(L, Nm), T(Tout) {}
  __device__ inline void momentum(int qi, unsigned base, const F (&v)[M]) const { (*this)(T.q[qi] + base, v); }
  __device__ inline void density(F *p, const F (&v)[M]) const { (*this)(p, v); }
};
// The same where the lane's zones are already those that it stores.
template <typename F, int M>
struct RingPut {
  unsigned o;
  bool one[M / 2], two[M / 2];
  __device__ inline explicit RingPut(const RingLane<F, M> &L) : o((unsigned)L.zl) {
#pragma unroll
    for (int h = 0; h < M / 2; h++) {
      two[h] = L.useful(2 * h + 1);
      one[h] = L.useful(2 * h) && !two[h];
    }
  }
  __device__ inline void operator()(F *p, const F (&v)[M]) const {
    using V2 = F __attribute__((ext_vector_type(2), aligned(sizeof(F))));
#pragma unroll
    for (int h = 0; h < M / 2; h++) {
      if (two[h]) *reinterpret_cast<V2 *>(at(p, o + 2 * h)) = V2{v[2 * h], v[2 * h + 1]};
      else if (one[h]) *at(p, o + 2 * h) = v[2 * h];
    }
  }
};

// Constants of ring (j, k): time step, face area, inverse volume, the
// shift velocity v0, the integer shift (as a store offset in [0, n)) and the
// PPA residual xi (Eqs. 32, 33), dt/dX, the PPA flux factor xi dX S, and the
// factors of 12d along X (Tab. "momenta": v = Pi/R - R Omega; R = 1 and
// Omega = 0 on a Cartesian mesh).
template <typename F>
struct RingConst {
  F Sdt, vinv, vb, cdt, pfac, R, iR, Rw; // Sdt: face area times dt
  PpaX<F> X;
  bool fg;
  int Nm;
};
// The split of Eq. 29 for one ring: D = v0 dt / dX in this operation order
// with contraction off, N the nearest integer (ties away from zero) and
// xi = D - N, exact; the same arithmetic as the stand-alone split and the
// oracle, so N is reproduced bit for bit.
__device__ inline void ring_split_at(double v0, double dt, double dX, int &N, double &xi) {
#pragma clang fp contract(off)
  const double D = (v0 * dt) / dX;
  const double rn = round(D);
  N = (int)rn;
  xi = D - rn;
}

template <typename F>
__device__ inline RingConst<F> ring_const(const Mesh &m, int j, int k, int r, double dtd,
                                          const double *__restrict__ v0) {
  RingConst<F> C;
  const int n = m.nx;
  const double dXd = m.DX(j, k), Sd = m.Sx(j, k);
  C.Sdt = (F)(Sd * dtd);
  C.vinv = (F)m.Vinv(j, k);
  C.fg = m.fargo != 0;
  const double v0d = C.fg ? v0[r] : 0.0;
  // an FP32 v_x is a deviation from the ring's background vb: the residual
  // velocity is v_x - (v0 - vb)
  if constexpr (sizeof(F) == 4) C.vb = (F)(v0d - m.bg(BG_V, j, k));
  else C.vb = (F)v0d;
  int N = 0;
  double xid = 0.0;
  if (C.fg) ring_split_at(v0d, dtd, dXd, N, xid);
  // shift on store: zone i goes to (i + Nm) mod n
  N = __builtin_amdgcn_readfirstlane(N);
  if (N < -n || N >= n) N %= n;
  C.Nm = N < 0 ? N + n : N;
  const F xi = (F)xid;
  C.X = PpaX<F>{fabs(xi), F(1) - fabs(xi), xi >= F(0)};
  const double idX = m.g.inv_dxlen((size_t)k * m.nyg + j);
  C.cdt = (F)div_by(dtd, dXd, idX);
  C.pfac = (F)(xid * dXd * Sd);
  if (m.geo == FARGO_CARTESIAN) {
    C.R = C.iR = F(1);
    C.Rw = F(0);
  } else {
    const double R = m.Rcyl(j, k);
    C.R = (F)R;
    // (rounded once: dx idX itself, three roundings off, shows in v_x, whose error
    // after one spherical step it raised by 6 % in the mean square)
    C.iR = (F)(m.geo == FARGO_SPHERICAL ? div_by(1.0, R, m.dx * idX) : m.g.inv_ymed(j));
    // FP32: the X momenta are deviations R (v_x - vb) from the ring's
    // background, and so is the v_x formed from them (no frame term)
    C.Rw = sizeof(F) == 4 ? F(0) : C.R * (F)m.omega;
  }
  return C;
}

// Load order of the quantities of a ring: Pi-_y, Pi+_y [, Pi-_z, Pi+_z] [, e],
// then Pi-_x and Pi+_x, which 12d needs last (T.q holds Pi-_x, Pi+_x first).
template <int NQ>
__device__ constexpr int ring_qorder(int t) { return t + 2 < NQ ? t + 2 : t + 2 - NQ; }

// X transport of one ring segment held in registers (Ra: density, w: v_x on
// the lower faces, Qall[t]: quantity ring_qorder(t)), and its stores:
// van Leer residual sweep with w - v0, PPA residual, 12d along X; every
// output is stored shifted by N zones, out of place, by `put` (e, the density
// and v_x into the state; what becomes of Pi+-_y and Pi+-_z is put's matter).
// RIGHT: xi >= 0.
// Bound by its vector instructions, which went from some 1250 to 950 a wave (one
// sign of xi per compiled form, the parabola's edges as distances, the
// reciprocal's series, one wrap instead of a modulo, stores in pairs): in the ring
// pass of 3072 x 1024 zones 75 to 66 us, of 48 FP64 disks 355 to 290 and of 256 FP32
// disks 962 to 834, in the FP32 Z/X pass of 2048 x 768 x 96 3.26 to 2.88 ms.
template <bool RIGHT, typename F, int NQ, int M, class PUT>
__device__ inline void ring_update_dir(const RingConst<F> &C, unsigned base, const F (&Ra)[M], F (&w)[M],
                                       const F (&Qall)[NQ][M], bool has_e, const StateT<F> &s, const PUT &put) {
  const F vinv = C.vinv;
  F ri0[M], Fl[M], ri1[M], El[M], Eh[M], rf[M];
  // ---- density: van Leer residual sweep, then the PPA residual
  Upwind<F, M> Uw;
  {
#pragma unroll
    for (int q = 0; q < M; q++) {
      w[q] -= C.vb;
      ri0[q] = ring_rcp(Ra[q]);
    }
    F st[M];
    Uw.set(w, C.cdt);
    vlx_faces(Ra, Uw, st);
#pragma unroll
    for (int q = 0; q < M; q++) Fl[q] = flux_of(w[q] * st[q], C.Sdt);
    F Fh[M], R1[M];
    next_of(Fl, Fh);
#pragma unroll
    for (int q = 0; q < M; q++) {
      R1[q] = Ra[q] - vinv * (Fh[q] - Fl[q]);
      ri1[q] = ring_rcp(R1[q]);
      rf[q] = R1[q];
    }
    if (C.fg) {
      // El, Eh: PPA mass flux through the zone's lower and upper face, each
      // supplied by the zone upstream of it
      F val[M];
      ppa_values<RIGHT>(R1, C.X, val);
#pragma unroll
      for (int q = 0; q < M; q++) (RIGHT ? Eh[q] : El[q]) = flux_of(C.pfac, val[q]);
      if (RIGHT) prev_of(Eh, El);
      else next_of(El, Eh);
#pragma unroll
      for (int q = 0; q < M; q++) rf[q] = R1[q] - vinv * (Eh[q] - El[q]);
    }
  }
  // ---- the other quantities
  F pxm[M], pxp[M];
#pragma unroll
  for (int t = 0; t < NQ; t++) {
    const int qi = ring_qorder<NQ>(t);
    F Qv[M], Qs[M], G[M], Gh[M];
#pragma unroll
    for (int q = 0; q < M; q++) Qs[q] = Qall[t][q] * ri0[q];
    vlx_faces(Qs, Uw, G);
#pragma unroll
    for (int q = 0; q < M; q++) G[q] = flux_of(G[q], Fl[q]);
    next_of(G, Gh);
#pragma unroll
    for (int q = 0; q < M; q++) Qv[q] = Qall[t][q] - vinv * (Gh[q] - G[q]);
    if (C.fg) {
#pragma unroll
      for (int q = 0; q < M; q++) Qs[q] = Qv[q] * ri1[q];
      F st[M], Hl[M], Hh[M];
      ppa_values<RIGHT>(Qs, C.X, st);
#pragma unroll
      for (int q = 0; q < M; q++) (RIGHT ? Hh[q] : Hl[q]) = flux_of(st[q], RIGHT ? Eh[q] : El[q]);
      if (RIGHT) prev_of(Hh, Hl);
      else next_of(Hl, Hh);
#pragma unroll
      for (int q = 0; q < M; q++) Qv[q] = Qv[q] - vinv * (Hh[q] - Hl[q]);
    }
    if (qi == 0) {
#pragma unroll
      for (int q = 0; q < M; q++) pxm[q] = Qv[q];
    } else if (qi == 1) {
#pragma unroll
      for (int q = 0; q < M; q++) pxp[q] = Qv[q];
    } else {
      if (has_e && qi == NQ - 1) put(s.e + base, Qv);
      else put.momentum(qi, base, Qv);
    }
  }
  // ---- box 12d along X (Eq. 18) on the shifted ring: face i + N takes zones i - 1, i
  F pp[M], rp[M], vx[M];
  prev_of(pxp, pp);
  prev_of(rf, rp);
#pragma unroll
  for (int q = 0; q < M; q++) {
    const F mom = ring_div(pp[q] + pxm[q], rp[q] + rf[q]);
    // FP64: the product with the ring's 1/R; FP32 divides, since there a
    // rounded 1/R would bias v_x the same way at every step
    if constexpr (sizeof(F) == 8) vx[q] = mom * C.iR - C.Rw;
    else vx[q] = mom / C.R - C.Rw;
  }
  put(s.vx + base, vx);
  put.density(s.rho + base, rf);
}
// xi has one sign on a ring: a wave takes one of the two forms.
template <typename F, int NQ, int M, class PUT>
__device__ inline void ring_update(const RingConst<F> &C, unsigned base, const F (&Ra)[M], F (&w)[M],
                                   const F (&Qall)[NQ][M], bool has_e, const StateT<F> &s, const PUT &put) {
  if (C.X.right) ring_update_dir<true, F, NQ, M>(C, base, Ra, w, Qall, has_e, s, put);
  else ring_update_dir<false, F, NQ, M>(C, base, Ra, w, Qall, has_e, s, put);
}

// X transport of every active ring and 12d, both velocities (2D meshes, where
// there is no Z sweep).  v_y on a face takes the density and momentum of its two
// rings after their shifts, so a wave's window is placed on the zones that it
// stores: it reads each ring as far back as the ring shifts.  A workgroup of
// RX_W waves takes RX_W rl consecutive rings of a segment, rl to a wave in
// order; a ring hands its density and Pi+_y to the next one in registers, the
// last one of a wave through LDS.  The first ring of a workgroup is only read
// for the face above it (again the last one of the workgroup below).  A pass of
// its own for v_y read and wrote 4 words a zone more and wrote and read the
// momenta: 3072 x 1024 zones 66 + 19 to 68 us; the batches of 256 FP32 disks 765
// + 279 to 768 us and of 48 FP64 disks 299 + 92 to 313; 384 x 128 6.6 + 2.7 to 6.4.
// Eight waves: 68, 810, 326 and 7.7 us; eight rings a wave in place of at most
// four: 72, 772, 321; one ring (then eight waves): 71, 992, 376 us.
constexpr int RX_W = 4;
template <typename F, int M>
struct RingKeep : RingPut<F, M> {
  F *pm, *pp, *rh; // where Pi-_y, Pi+_y and the density are left
  bool keep_only;  // store nothing
  __device__ inline RingKeep(const RingLane<F, M> &L, F *a, F *b, F *c, bool only)
      : RingPut<F, M>(L), pm(a), pp(b), rh(c), keep_only(only) {
    if (only) {
#pragma unroll
      for (int h = 0; h < M / 2; h++) this->one[h] = this->two[h] = false;
    }
  }
  __device__ inline void momentum(int qi, unsigned, const F (&v)[M]) const {
#pragma unroll
    for (int q = 0; q < M; q++) (qi == 2 ? pm : pp)[q] = v[q];
  }
  __device__ inline void density(F *p, const F (&v)[M]) const {
    (*this)(p, v);
#pragma unroll
    for (int q = 0; q < M; q++) rh[q] = v[q];
  }
};
template <typename F, int NQ>
__device__ __forceinline__ void ring_x_body(Mesh m, const F *__restrict__ vx2, TSetT<F> T, StateT<F> s,
                                                const double *__restrict__ v0, const double *__restrict__ dtp,
                                                int nseg, int rl, unsigned bid_, unsigned nbk_) {
  constexpr int M = RING_M;
  __shared__ F edge[RX_W][2][M][WAVE];
  const unsigned blk = xcd_remap(bid_, nbk_);
  const int lane = threadIdx.x & (WAVE - 1);
  // wave-uniform (readfirstlane), so that the ring's constants come through
  // scalar loads
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
  const int seg = (int)(blk % (unsigned)nseg), first = m.j0 + (int)(blk / (unsigned)nseg) * (RX_W * rl - 1);
  const double dtd = *dtp;
  const bool has_e = T.a[T_E] != nullptr;
  F rho_b[M], pp_b[M]; // of the ring below
  F rho_1[M], pm_1[M]; // of the wave's first ring
  int j1 = m.jn;       // the wave's first ring, if it owns the face below
  auto store_vy = [&](int j, const RingPut<F, M> &put, const F (&pp)[M], const F (&rb)[M], const F (&pm)[M],
                      const F (&r)[M]) {
    F v[M];
#pragma unroll
    for (int q = 0; q < M; q++) v[q] = (pp[q] + pm[q]) / (rb[q] + r[q]);
    put(s.vy + m.o32(0, j, 0), v);
  };
  const RingLane<F, M> L0(m.nx, seg, lane);
  const RingPut<F, M> put(L0);
#pragma unroll 1
  for (int t = 0; t < rl; t++) {
    const int u = wv * rl + t, jr = first - 1 + u; // the workgroup's ring u
    if (jr >= m.jn || (u == 0 && first == m.j0 && !m.yper())) continue;
    const int j = u == 0 ? m.jbelow(first) : jr;
    const RingConst<F> C = ring_const<F>(m, j, 0, j - m.j0, dtd, v0);
    const RingLane<F, M> L(m.nx, seg, lane, C.Nm);
    const unsigned base = m.o32(0, j, 0);
    // every load of the window is issued before the first use
    F w[M], Ra[M], Qall[NQ][M];
    L.load(T.a[T_RHO] + base, Ra);
    L.load(vx2 + base, w);
#pragma unroll
    for (int q = 0; q < NQ; q++) L.load(T.q[ring_qorder<NQ>(q)] + base, Qall[q]);
    F pm[M], pp[M], rh[M];
    const RingKeep<F, M> keep(L, pm, pp, rh, u == 0);
    ring_update<F, NQ, M>(C, base, Ra, w, Qall, has_e, s, keep);
    if (u > 0 && j >= m.ylo()) {
      if (t > 0) {
        store_vy(j, put, pp_b, rho_b, pm, rh);
      } else {
        j1 = j;
#pragma unroll
        for (int q = 0; q < M; q++) {
          rho_1[q] = rh[q];
          pm_1[q] = pm[q];
        }
      }
    }
#pragma unroll
    for (int q = 0; q < M; q++) {
      rho_b[q] = rh[q];
      pp_b[q] = pp[q];
    }
  }
#pragma unroll
  for (int q = 0; q < M; q++) {
    edge[wv][0][q][lane] = rho_b[q];
    edge[wv][1][q][lane] = pp_b[q];
  }
  __syncthreads();
  if (j1 < m.jn) {
#pragma unroll
    for (int q = 0; q < M; q++) {
      rho_b[q] = edge[wv - 1][0][q][lane];
      pp_b[q] = edge[wv - 1][1][q][lane];
    }
    store_vy(j1, put, pp_b, rho_b, pm_1, rho_1);
  }
}
template <typename F, int NQ>
__global__ __launch_bounds__(RX_W * WAVE, 4) void k_ring_x(Mesh m, const F *__restrict__ vx2, TSetT<F> T, StateT<F> s,
                                                           const double *__restrict__ v0,
                                                           const double *__restrict__ dtp, int nseg, int rl) {
  ring_x_body<F, NQ>(m, vx2, T, s, v0, dtp, nseg, rl, blockIdx.x, gridDim.x);
}

// Z sweep and X transport fused (3D meshes).  A wave owns one segment of the
// rings of row j and walks up a chunk of planes.  For each of its M zones a
// lane carries the Z column window of the sweep (three zones, the slopes and
// the flux through the lower face), as a column sweep does; once the fluxes
// through face k are known the Z update of plane k - 1 is complete, and it is
// handed, in registers, to the X transport of ring (j, k - 1).  The Z-swept
// quantities never go through memory.  The halo zones of the segment are
// swept along Z as well, so segments stay independent.
// The quotients of its slopes, as those of the X part, are those of ring_div; in
// FP64 a zone's 1 / rho is correctly rounded.  The error of an FP64 step against
// extended precision is that of the separate passes with divided slopes or less
// (80 x 72 x 60 zones, 40 states, mean square: density 7.82e-17 both, with an energy
// 7.88e-17 both and the energy 1.236e-16 both).
// Bound by its vector instructions (some 850 a wave and plane in FP64, 4 cycles
// each), and yet faster than a Z sweep and a ring kernel apart, whose 29 words a
// zone between them become 16: 2048 x 768 x 96 in FP64 3.78 + 3.19 ms apart, 5.42
// fused, 5.25 with the stores' places formed once per ring, the half step's
// factors once per face and the halo a lane shorter; 1536 x 512 x 128 adiabatic
// 2.85 + 2.45, 4.61, 4.36 (at two waves per SIMD, where the three that the
// launch bound would allow spill: 4.74); 160 x 144 x 120: 96 + 83, 143, 134 us.
// In FP32 2.8 ms.  Selects in place of the branches around quotients
// cost registers and gained nothing, nor did two or three planes per turn of the
// loop, which save the window's moves but spill.
template <typename F, int NQ>
__global__ __launch_bounds__(256, (sizeof(F) == 8 && NQ == 7 ? 2 : 3)) void k_zx(Mesh m, const F *__restrict__ vx2, const F *__restrict__ vz,
                                            TSetT<F> T, TSetT<F> Tout, StateT<F> s, const double *__restrict__ v0,
                                            const double *__restrict__ dtp, int nseg, int nkc) {
  constexpr int M = zx_m<F>();
  const unsigned blk = xcd_remap(blockIdx.x, gridDim.x);
  const int lane = threadIdx.x & (WAVE - 1), wv = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
  const long gw = (long)blk * (blockDim.x / WAVE) + wv;
  if (gw >= (long)nseg * m.ny * nkc) return;
  const int seg = (int)(gw % nseg);
  const long rest = gw / nseg;
  const int j = m.j0 + (int)(rest % m.ny), kc = (int)(rest / m.ny);
  const int a0 = m.k0 + kc * m.chunk, a1 = min(a0 + m.chunk, m.kn);
  const RingLane<F, M> L(m.nx, seg, lane);
  const double dtd = *dtp;
  const F dt = (F)dtd;
  const bool has_e = T.a[T_E] != nullptr;
  // a zone of the window (M columns): density, Q/rho (CT: the reciprocal of the
  // density and the conserved Q), v_z on the lower face, v_x on the lower X face
  // (for the X transport).  FP64 hands the conserved Q on as loaded: formed again
  // as rho (Q/rho), the velocities of a step on 80 x 72 x 60 zones were 4 to 5 %
  // further off in the mean square.  With an energy, at two waves per SIMD either
  // way, Q comes from the window (CT).  Without one that would take 176 registers
  // and the third wave (5.18 to 5.70 ms on 2048 x 768 x 96); each lane leaves Q in
  // LDS for the two planes in between instead (KQ: 5.14 to 5.17 ms, 37 KB a
  // workgroup, three of them a compute unit).  FP32 forms it again.
  constexpr bool CT = sizeof(F) == 8 && NQ == 7, KQ = sizeof(F) == 8 && NQ == 6;
  __shared__ F kept[KQ ? 4 : 1][KQ ? 3 : 1][KQ ? NQ : 1][KQ ? WAVE : 1];
  auto keep = [&](const F (&T)[NQ][M], int slot) {
    if constexpr (KQ) {
#pragma unroll
      for (int q = 0; q < NQ; q++) kept[wv][slot][q][lane] = T[q][0];
    }
  };
  struct Zw {
    F rho[M], ri[CT ? M : 1], v[NQ][M], w[M], vx[M];
    __device__ inline F q(int t, int c) const { return CT ? v[t][c] * ri[CT ? c : 0] : v[t][c]; }
    __device__ inline F Q(int t, int c) const { return CT ? v[t][c] : rho[c] * v[t][c]; }
  };
  struct Zr {
    F rho[M], T[NQ][M], w[M], vx[M];
  };
  auto raw = [&](int a, Zr &z) {
    const unsigned b = m.o32(0, j, a);
    L.load_each(T.a[T_RHO] + b, z.rho);
#pragma unroll
    for (int q = 0; q < NQ; q++) L.load_each(T.q[q] + b, z.T[q]);
    L.load_each(vz + b, z.w);
    L.load_each(vx2 + b, z.vx);
  };
  auto derive = [&](const Zr &r, Zw &z) {
#pragma unroll
    for (int c = 0; c < M; c++) {
      z.rho[c] = r.rho[c];
      const F ri = sizeof(F) == 8 ? F(1) / r.rho[c] : ring_rcp(r.rho[c]);
      if (CT) z.ri[CT ? c : 0] = ri;
      z.w[c] = r.w[c];
      z.vx[c] = r.vx[c];
#pragma unroll
      for (int q = 0; q < NQ; q++) z.v[q][c] = CT ? r.T[q][c] : r.T[q][c] * ri;
    }
  };
  auto Lz = [&](int a) { return (F)m.Lz(j, a); };
  // FP32: the X momenta (quantities 0 and 1) are deviations from a background
  // constant on each ring, as in column_sweep; dl(f) is its increment across
  // Z face f
  constexpr bool DEV = sizeof(F) == 4;
  auto dl = [&](int f) { return DEV ? (F)m.bg(BG_DLZ, j, f) : F(0); };
  auto hz = [&](int f) { return (F)m.hz(j, f); };
  Zw zm, z0, zp;
  Zr rn;
  raw(a0 - 2, rn);
  derive(rn, zp); // used only for the first slope
  raw(a0 - 1, rn);
  derive(rn, zm);
  raw(a0, rn);
  derive(rn, z0);
  keep(rn.T, 0);
  int ks = 1; // the slot of zone f + 1; zone f - 1 has the one after it
  raw(a0 + 1, rn);
  F sm[NQ + 1][M], s0[NQ + 1][M];
  F dlf = dl(a0); // background increment at face f
  {
    const F hm = hz(a0 - 1), hp = hz(a0), dlm = dl(a0 - 1);
#pragma unroll
    for (int c = 0; c < M; c++) {
      sm[NQ][c] = vl_slope<RingDiv>(zp.rho[c], zm.rho[c], z0.rho[c], hm, hp);
#pragma unroll
      for (int q = 0; q < NQ; q++)
        sm[q][c] = (DEV && q < 2) ? vl_slope_b<RingDiv>(zp.q(q, c), zm.q(q, c), z0.q(q, c), hm, hp, dlm, dlf)
                                  : vl_slope<RingDiv>(zp.q(q, c), zm.q(q, c), z0.q(q, c), hm, hp);
    }
  }
  F Fp[M], FQp[NQ][M];
#pragma unroll
  for (int c = 0; c < M; c++) {
    Fp[c] = F(0);
#pragma unroll
    for (int q = 0; q < NQ; q++) FQp[q][c] = F(0);
  }
  F Lm = Lz(a0 - 1);
#pragma unroll 1
  for (int f = a0; f <= a1; f++) {
    derive(rn, zp); // zone f + 1
    keep(rn.T, ks);
    const int kr = ks = ks == 2 ? 0 : ks + 1;
    if (f + 2 <= a1 + 1) raw(f + 2, rn);
    const F hm = hz(f), hp = hz(f + 1), L0 = Lz(f), Sf = (F)m.Sz(j, f), dlf1 = dl(f + 1);
    F Fr[M], FQ[NQ][M];
#pragma unroll
    for (int c = 0; c < M; c++) {
      s0[NQ][c] = vl_slope<RingDiv>(zm.rho[c], z0.rho[c], zp.rho[c], hm, hp);
#pragma unroll
      for (int q = 0; q < NQ; q++)
        s0[q][c] = (DEV && q < 2) ? vl_slope_b<RingDiv>(zm.q(q, c), z0.q(q, c), zp.q(q, c), hm, hp, dlf, dlf1)
                                  : vl_slope<RingDiv>(zm.q(q, c), z0.q(q, c), zp.q(q, c), hm, hp);
      const F w = z0.w[c];
      const Upface<F> U(w, dt, Lm, L0);
      Fr[c] = flux_of(w * U.star(zm.rho[c], sm[NQ][c], z0.rho[c], s0[NQ][c]) * Sf, dt);
#pragma unroll
      for (int q = 0; q < NQ; q++) {
        // relative to the background of the face's lower zone
        const F qr = (DEV && q < 2) ? z0.q(q, c) + dlf : z0.q(q, c);
        FQ[q][c] = flux_of(U.star(zm.q(q, c), sm[q][c], qr, s0[q][c]), Fr[c]);
      }
    }
    if (f > a0) {
      // Z update of plane k = f - 1, then its ring
      const int k = f - 1;
      const F vi = (F)m.Vinv(j, k);
      F Ra[M], Qall[NQ][M], w[M];
#pragma unroll
      for (int c = 0; c < M; c++) {
        Ra[c] = zm.rho[c] - vi * (Fr[c] - Fp[c]);
        w[c] = zm.vx[c];
#pragma unroll
        for (int t = 0; t < NQ; t++) {
          const int q = ring_qorder<NQ>(t);
          F Qz;
          if constexpr (KQ) Qz = kept[wv][kr][q][lane];
          else Qz = zm.Q(q, c);
          Qall[t][c] = Qz - vi * (FQ[q][c] - FQp[q][c]);
        }
      }
      const int r = (k - m.k0) * m.ny + (j - m.j0);
      const RingConst<F> C = ring_const<F>(m, j, k, r, dtd, v0);
      ring_update<F, NQ, M>(C, m.o32(0, j, k), Ra, w, Qall, has_e, s, RingShift<F, M>(L, C.Nm, Tout));
    }
#pragma unroll
    for (int c = 0; c < M; c++) {
      Fp[c] = Fr[c];
#pragma unroll
      for (int q = 0; q <= NQ; q++) sm[q][c] = s0[q][c];
#pragma unroll
      for (int q = 0; q < NQ; q++) // relative to the background of the face's upper zone
        FQp[q][c] = (DEV && q < 2) ? FQ[q][c] - dlf * Fr[c] : FQ[q][c];
    }
    zm = z0;
    z0 = zp;
    Lm = L0;
    dlf = dlf1;
  }
}

// ------------------------------------------------------------------------
// 12d along Y and Z on the owned faces (Eq. 18 with Tab. "momenta").
// ------------------------------------------------------------------------
template <typename F>
__device__ __forceinline__ void vel_body(Mesh m, StateT<F> s, TSetT<F> T, unsigned bid_, unsigned nbk_) {
  unsigned Lb = xcd_remap(bid_, nbk_);
  int kk = (int)(Lb % (unsigned)m.nz);
  unsigned rest = Lb / (unsigned)m.nz;
  int jj = (int)(rest % (unsigned)m.ny), ib = (int)(rest / (unsigned)m.ny);
  int i = ib * (int)blockDim.x + (int)threadIdx.x;
  if (i >= m.nx) return;
  int j = m.j0 + jj, k = m.k0 + kk;
  unsigned c = m.o32(i, j, k);
  const bool dy = j >= m.ylo(), dz = k >= m.zlo();
  // all loads first: the stores below may alias them as far as the compiler
  // knows, and would otherwise hold the Z loads back behind the Y store
  F rc = s.rho[c], ry = F(0), py = F(0), my = F(0), rz = F(0), pz = F(0), mz = F(0);
  if (dy) {
    const unsigned cm = m.o32(i, m.jbelow(j), k);
    ry = s.rho[cm];
    py = T.a[T_PYP][cm];
    my = T.a[T_PYM][c];
  }
  if (dz) {
    const unsigned cm = m.o32(i, j, m.kbelow(k));
    rz = s.rho[cm];
    pz = T.a[T_PZP][cm];
    mz = T.a[T_PZM][c];
  }
  if (dy) s.vy[c] = (py + my) / (ry + rc);
  if (dz) {
    F v = (pz + mz) / (rz + rc);
    s.vz[c] = m.geo == FARGO_SPHERICAL ? v / (F)m.g.ymed(j) : v;
  }
}
template <typename F>
__global__ __launch_bounds__(256) void k_vel(Mesh m, StateT<F> s, TSetT<F> T) {
  vel_body<F>(m, s, T, blockIdx.x, gridDim.x);
}

// n zones split into nchunk chunks of equal length (the last one shorter by
// less than the count), so that the threads of a sweep end together: the mesh
// with that chunk length, and the number of chunks it takes.
inline Mesh chunked(const Mesh &m, int n, int &nchunk) {
  Mesh mm = m;
  mm.chunk = (n + nchunk - 1) / nchunk;
  nchunk = (n + mm.chunk - 1) / mm.chunk;
  return mm;
}
// The fewest chunks of at most m.chunk zones, or more where those would leave
// the chip idle (fill_chunks; `each` workers per chunk, of which `slots` run at
// once).  A 2D disk of 384 x 128 zones in two 64-zone chunks is swept along Y
// by 4 workgroups (58 us); 128 chunks of one zone take 6.2 us.  3072 x 1024:
// 77 to 47 us (5 TB/s of its 9 words a zone); the box of 160 x 144 x 120
// zones 93 to 78 us; the FP32 Z/X pass of 501 x 167 x 43 zones 258 to 153 us.
// Meshes that fill the chip with chunks of m.chunk zones (2048 x 768 x 96) keep
// them.
constexpr int SWEEP_OVER = 2; // zones a chunk costs beside its own (1, 2 and 4 measured alike)
inline Mesh filled(const Mesh &m, int n, long each, long slots, int &nchunk) {
  nchunk = fill_chunks(n, m.chunk, 1, each, slots, SWEEP_OVER);
  return chunked(m, n, nchunk);
}

template <typename F, int NQ, bool D3, bool ADI>
void sweep_y_launch(Launch &L, const Mesh &m0, const StateT<F> &s, const TSetT<F> &out, const double *dt) {
  constexpr auto kern = k_sweep_y<F, NQ, D3, ADI>;
  static const long slots[4] = {block_slots(kern, 64), block_slots(kern, 128), block_slots(kern, 192),
                                block_slots(kern, 256)};
  int nib, bs, nchunk;
  row_blocks(m0.nx, nib, bs);
  const int nrows = D3 ? m0.nz + 4 : 1;
  const Mesh m = filled(m0, m0.ny, (long)nib * nrows, slots[bs / WAVE - 1], nchunk);
  unsigned nb = (unsigned)nib * (unsigned)nchunk * (unsigned)nrows;
  k_sweep_y<F, NQ, D3, ADI><<<nb, bs, 0, L.s>>>(m, s.rho, s.vx, s.vy, s.vz, s.e, out, dt, nchunk);
}

} // namespace

// s: rho of the state, post-source velocities and energy (box 9 filled)
template <typename F>
void launch_sweep_y(Launch &L, const Mesh &m, const StateT<F> &s, const TSetT<F> &out, const double *dt) {
  prof_begin(L, K_SWEEP_Y);
  bool adi = m.eos == FARGO_ADIABATIC;
  if (m.d3) {
    if (adi) sweep_y_launch<F, 7, true, true>(L, m, s, out, dt);
    else sweep_y_launch<F, 6, true, false>(L, m, s, out, dt);
  } else {
    if (adi) sweep_y_launch<F, 5, false, true>(L, m, s, out, dt);
    else sweep_y_launch<F, 4, false, false>(L, m, s, out, dt);
  }
  prof_end(L, K_SWEEP_Y);
}

// The most rings per wave: twice as many while that leaves two workgroups for
// each compute unit; and the workgroups per segment.
constexpr int RX_RINGS = 4;
inline int ring_blocks(int ny, int rl) { return (ny + RX_W * rl - 2) / (RX_W * rl - 1); }

inline int ring_rows(long nring, int nseg, int most) {
  int rl = 1;
  while (rl < most && nseg * ((nring + 2 * RX_W * rl - 2) / (2 * RX_W * rl - 1)) >= 2 * CHIP_CUS) rl *= 2;
  return rl;
}

template <typename F>
void launch_ring_x(Launch &L, const Mesh &m, const F *vx2, const TSetT<F> &T, const StateT<F> &s, const double *v0,
                   const double *dt) {
  constexpr int U = RingLane<F, RING_M>::U;
  const int nseg = (m.nx + U - 1) / U;
  const int rl = ring_rows(m.ny, nseg, RX_RINGS);
  const unsigned nb = (unsigned)(nseg * ring_blocks(m.ny, rl));
  prof_begin(L, K_RING_X);
  if (T.nq == 5) k_ring_x<F, 5><<<nb, RX_W * WAVE, 0, L.s>>>(m, vx2, T, s, v0, dt, nseg, rl); // Pi-+_x, Pi-+_y, e
  else k_ring_x<F, 4><<<nb, RX_W * WAVE, 0, L.s>>>(m, vx2, T, s, v0, dt, nseg, rl);
  prof_end(L, K_RING_X);
}

// Fused Z sweep and X transport: one wave per (segment, row, chunk of planes).
template <typename F>
void launch_zx(Launch &L, const Mesh &m0, const F *vx2, const F *vz, const TSetT<F> &T, const TSetT<F> &Tout,
               const StateT<F> &s, const double *v0, const double *dt) {
  constexpr int U = RingLane<F, zx_m<F>()>::U;
  static const long slots[2] = {4 * block_slots(k_zx<F, 6>, 256), 4 * block_slots(k_zx<F, 7>, 256)};
  int nkc;
  const int nseg = (m0.nx + U - 1) / U;
  const Mesh m = filled(m0, m0.nz, (long)nseg * m0.ny, slots[T.nq == 7], nkc);
  const long waves = (long)nseg * m.ny * nkc;
  const unsigned nb = (unsigned)((waves + 3) / 4);
  prof_begin(L, K_ZX);
  if (T.nq == 7) k_zx<F, 7><<<nb, 256, 0, L.s>>>(m, vx2, vz, T, Tout, s, v0, dt, nseg, nkc);
  else k_zx<F, 6><<<nb, 256, 0, L.s>>>(m, vx2, vz, T, Tout, s, v0, dt, nseg, nkc);
  prof_end(L, K_ZX);
}

// The same with two consecutive zones per thread (16-byte loads and stores
// in FP64); rows of an even number of zones.
template <typename F>
__device__ __forceinline__ void vel2_body(Mesh m, StateT<F> s, TSetT<F> T, unsigned bid_, unsigned nbk_) {
  using V2 = typename std::conditional<sizeof(F) == 8, double2, float2>::type;
  unsigned Lb = xcd_remap(bid_, nbk_);
  int kk = (int)(Lb % (unsigned)m.nz);
  unsigned rest = Lb / (unsigned)m.nz;
  int jj = (int)(rest % (unsigned)m.ny), ib = (int)(rest / (unsigned)m.ny);
  int i = 2 * (ib * (int)blockDim.x + (int)threadIdx.x);
  if (i >= m.nx) return;
  int j = m.j0 + jj, k = m.k0 + kk;
  unsigned c = m.o32(i, j, k);
  const bool dy = j >= m.ylo(), dz = k >= m.zlo();
  auto ld = [&](const F *p, unsigned o) { return *reinterpret_cast<const V2 *>(p + o); };
  const V2 zero{F(0), F(0)};
  V2 rc = ld(s.rho, c), ry = zero, py = zero, my = zero, rz = zero, pz = zero, mz = zero;
  if (dy) {
    const unsigned cm = m.o32(i, m.jbelow(j), k);
    ry = ld(s.rho, cm);
    py = ld(T.a[T_PYP], cm);
    my = ld(T.a[T_PYM], c);
  }
  if (dz) {
    const unsigned cm = m.o32(i, j, m.kbelow(k));
    rz = ld(s.rho, cm);
    pz = ld(T.a[T_PZP], cm);
    mz = ld(T.a[T_PZM], c);
  }
  if (dy) *reinterpret_cast<V2 *>(s.vy + c) = V2{(py.x + my.x) / (ry.x + rc.x), (py.y + my.y) / (ry.y + rc.y)};
  if (dz) {
    V2 v{(pz.x + mz.x) / (rz.x + rc.x), (pz.y + mz.y) / (rz.y + rc.y)};
    if (m.geo == FARGO_SPHERICAL) {
      const F r = (F)m.g.ymed(j);
      v.x = v.x / r;
      v.y = v.y / r;
    }
    *reinterpret_cast<V2 *>(s.vz + c) = v;
  }
}
template <typename F>
__global__ __launch_bounds__(256) void k_vel2(Mesh m, StateT<F> s, TSetT<F> T) {
  vel2_body<F>(m, s, T, blockIdx.x, gridDim.x);
}

// multi-mesh forms (ManyGrid): the sweep and 12d in blocks of one wave
template <typename F>
struct SweepYArgs {
  Mesh m; // with the balanced chunk length
  const F *rho, *vx, *vy, *vz, *e;
  TSetT<F> out;
  const double *dt;
  int nchunk;
  unsigned nb;
};
template <typename F, int NQ, bool D3, bool ADI>
__global__ __launch_bounds__(256) void k_sweep_y_many(const void *args, const uint2 *tab) {
  const uint2 t = many_block(tab);
  if (t.x == MANY_NONE) return;
  const SweepYArgs<F> a = many_args<SweepYArgs<F>>(args, t.x);
  sweep_y_body<F, NQ, D3, ADI>(a.m, a.rho, a.vx, a.vy, a.vz, a.e, a.out, a.dt, a.nchunk, t.y, a.nb);
}
template <typename F>
struct RingArgs {
  Mesh m;
  const F *vx2;
  TSetT<F> T;
  StateT<F> s;
  const double *v0, *dt;
  int nseg, rl;
  unsigned nb, pad_;
};
template <typename F, int NQ>
__global__ __launch_bounds__(RX_W * WAVE, 4) void k_ring_x_many(const void *args, const uint2 *tab) {
  const uint2 t = many_block(tab);
  if (t.x == MANY_NONE) return;
  const RingArgs<F> a = many_args<RingArgs<F>>(args, t.x);
  ring_x_body<F, NQ>(a.m, a.vx2, a.T, a.s, a.v0, a.dt, a.nseg, a.rl, t.y, a.nb);
}

template <typename F>
void launch_vel(Launch &L, const Mesh &m, const StateT<F> &s, const TSetT<F> &T) {
  int nib, bs;
  prof_begin(L, K_VEL);
  if (m.nx % 2 == 0) {
    row_blocks(m.nx / 2, nib, bs);
    unsigned nb = (unsigned)nib * (unsigned)m.ny * (unsigned)m.nz;
    k_vel2<F><<<nb, bs, 0, L.s>>>(m, s, T);
  } else {
    row_blocks(m.nx, nib, bs);
    unsigned nb = (unsigned)nib * (unsigned)m.ny * (unsigned)m.nz;
    k_vel<F><<<nb, bs, 0, L.s>>>(m, s, T);
  }
  prof_end(L, K_VEL);
}

// multi-mesh launches (ManyGrid) on 2D meshes: blocks of one wave for the
// column sweep, so that narrow meshes leave few threads idle
constexpr int MANY_BS = 64;

template <typename F>
size_t sweep_y_args_bytes() { return sizeof(SweepYArgs<F>); }

template <typename F>
int sweep_y_rows(const std::vector<Mesh> &ms, int most) {
  const bool adi = ms[0].eos == FARGO_ADIABATIC;
  static const long slots[2] = {block_slots(k_sweep_y_many<F, 4, false, false>, MANY_BS),
                                block_slots(k_sweep_y_many<F, 5, false, true>, MANY_BS)};
  return fill_chunk_length(ms, most, slots[adi], SWEEP_OVER,
                           [](const Mesh &m) { return (m.nx + MANY_BS - 1) / MANY_BS; });
}

template <typename F>
unsigned sweep_y_args(const Mesh &m0, const StateT<F> &s, const TSetT<F> &out, const double *dt, void *dst) {
  int nchunk = (m0.ny + m0.chunk - 1) / m0.chunk;
  const Mesh m = chunked(m0, m0.ny, nchunk);
  const unsigned nb = (unsigned)((m.nx + MANY_BS - 1) / MANY_BS) * (unsigned)nchunk;
  *(SweepYArgs<F> *)dst = SweepYArgs<F>{m, s.rho, s.vx, s.vy, s.vz, s.e, out, dt, nchunk, nb};
  return nb;
}

template <typename F>
void launch_sweep_y_many(Launch &L, const Mesh &m0, const ManyGrid &g) {
  prof_begin(L, K_SWEEP_Y);
  if (m0.eos == FARGO_ADIABATIC) k_sweep_y_many<F, 5, false, true><<<g.nblk, MANY_BS, 0, L.s>>>(g.args, g.tab);
  else k_sweep_y_many<F, 4, false, false><<<g.nblk, MANY_BS, 0, L.s>>>(g.args, g.tab);
  prof_end(L, K_SWEEP_Y);
}

template <typename F>
size_t ring_x_args_bytes() { return sizeof(RingArgs<F>); }

template <typename F>
int ring_x_rows(const std::vector<Mesh> &ms) {
  constexpr int U = RingLane<F, RING_M>::U;
  long n = 0;
  for (const Mesh &m : ms) n += (long)((m.nx + U - 1) / U) * m.ny;
  return ring_rows(n, 1, RX_RINGS);
}

template <typename F>
unsigned ring_x_args(const Mesh &m, const F *vx2, const TSetT<F> &T, const StateT<F> &s, const double *v0,
                     const double *dt, int rl, void *dst) {
  constexpr int U = RingLane<F, RING_M>::U;
  const int nseg = (m.nx + U - 1) / U;
  const unsigned nb = (unsigned)(nseg * ring_blocks(m.ny, rl));
  *(RingArgs<F> *)dst = RingArgs<F>{m, vx2, T, s, v0, dt, nseg, rl, nb, 0};
  return nb;
}

template <typename F>
void launch_ring_x_many(Launch &L, int nq, const ManyGrid &g) {
  prof_begin(L, K_RING_X);
  if (nq == 5) k_ring_x_many<F, 5><<<g.nblk, RX_W * WAVE, 0, L.s>>>(g.args, g.tab);
  else k_ring_x_many<F, 4><<<g.nblk, RX_W * WAVE, 0, L.s>>>(g.args, g.tab);
  prof_end(L, K_RING_X);
}

#define FARGO_TRANSPORT_MANY(F)                                                                                     \
  template size_t sweep_y_args_bytes<F>();                                                                         \
  template int sweep_y_rows<F>(const std::vector<Mesh> &, int);                                                    \
  template unsigned sweep_y_args<F>(const Mesh &, const StateT<F> &, const TSetT<F> &, const double *, void *);    \
  template void launch_sweep_y_many<F>(Launch &, const Mesh &, const ManyGrid &);                                  \
  template size_t ring_x_args_bytes<F>();                                                                          \
  template int ring_x_rows<F>(const std::vector<Mesh> &);                                                          \
  template unsigned ring_x_args<F>(const Mesh &, const F *, const TSetT<F> &, const StateT<F> &, const double *,   \
                                   const double *, int, void *);                                                   \
  template void launch_ring_x_many<F>(Launch &, int, const ManyGrid &);
FARGO_TRANSPORT_MANY(double)
FARGO_TRANSPORT_MANY(float)
#undef FARGO_TRANSPORT_MANY

#define FARGO_TRANSPORT_INST(F)                                                                                    \
  template void launch_sweep_y<F>(Launch &, const Mesh &, const StateT<F> &, const TSetT<F> &, const double *);   \
  template void launch_ring_x<F>(Launch &, const Mesh &, const F *, const TSetT<F> &, const StateT<F> &,         \
                                 const double *, const double *);                                                \
  template void launch_zx<F>(Launch &, const Mesh &, const F *, const F *, const TSetT<F> &, const TSetT<F> &,    \
                             const StateT<F> &, const double *, const double *);                                  \
  template void launch_vel<F>(Launch &, const Mesh &, const StateT<F> &, const TSetT<F> &);
FARGO_TRANSPORT_INST(double)
FARGO_TRANSPORT_INST(float)
#undef FARGO_TRANSPORT_INST

} // namespace fargo
