// Box 3 (bulk azimuthal velocity per ring, Eq. 37), box 6 (time step,
// Eq. cfl2 items 1-3, Eq. 38) and the orbital-advection split of Eq. 29.
//
// A wave (or, where rings are few or long, a workgroup of four) takes a ring
// at a time: the ring's v0 and, for each of its zones, the cell time step and
// the shear rate; the ring's extremes go to its slot.  A workgroup then reduces
// the slots (exact and order independent: min/max) and forms dt; where they are
// few the source step does so itself.  The split of every ring's displacement into (N, xi) is taken by the ring kernel
// of the X transport (and by k_split for the stand-alone entry point).  The
// time step and the split use floating-point contraction off and the operation
// order of the written definition, so that the integer shift N is reproducible
// bit for bit.
#include <type_traits>

#include "fargo_internal.h"

namespace fargo {

namespace {

template <typename Op>
__device__ inline double block_reduce(double v, Op op, double id, double *lds) {
  for (int o = 32; o > 0; o >>= 1) v = op(v, __shfl_xor(v, o, 64));
  int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) lds[wid] = v;
  __syncthreads();
  int nw = (blockDim.x + 63) >> 6;
  v = lane < nw ? lds[lane] : id;
  for (int o = 32; o > 0; o >>= 1) v = op(v, __shfl_xor(v, o, 64));
  return v; // valid in every lane
}

struct Add { __device__ double operator()(double a, double b) const { return a + b; } };

__global__ void k_set_dt(DevWords w, double dt) { *w.dt = dt; }

// Constants of Eq. cfl2 for ring (j, k): lengths and their reciprocals.
struct CflRing {
  double Lx, iLx, iLy, iLz, iL2, k3, dXp, idXp;
};
__device__ inline CflRing cfl_ring(const Mesh &m, int j, int k, bool shear_on) {
#pragma clang fp contract(off)
  CflRing C;
  const double Lyy = m.g.Ly(j), Lzz = m.d3 ? m.Lz(j, k) : 0.0;
  C.Lx = m.DX(j, k);
  C.iLx = 1.0 / C.Lx;
  C.iLy = 1.0 / Lyy;
  C.iLz = m.d3 ? 1.0 / Lzz : 0.0;
  double Lmin = fmin(C.Lx, Lyy);
  if (m.d3) Lmin = fmin(Lmin, Lzz);
  C.iL2 = 1.0 / (Lmin * Lmin);
  C.k3 = 4.0 * m.cvnr * m.cvnr;
  C.dXp = shear_on ? m.DX(j + 1, k) : 1.0;
  C.idXp = 1.0 / C.dXp;
  return C;
}

// Eq. cfl2 for one zone through the inverse steps (rates u / Delta): the
// minimum step of a cell over directions is its maximum rate; returns the sum
// of the squared rates of items 1-3 (and 4 with viscosity), and flags a
// non-finite or non-positive state in `bad`.  q: sound speed (isothermal)
// or internal energy; vxc, vxp: full v_x on the zone's two X faces; vb: the
// ring's bulk velocity (0 without orbital advection).
template <bool D3, bool ADI>
__device__ inline double zone_rate2(const CflRing &C, double vb, double vxc, double vxp, double rho, double q,
                                    double vyc, double vyp, double vzc, double vzp, double nu, double gamma, int &bad) {
#pragma clang fp contract(off)
  double cw2; // squared wave speed
  if (!ADI) cw2 = q * q;
  else cw2 = gamma * ((gamma - 1.0) * q) / rho;
  bad |= !(rho > 0.0) || !isfinite(rho) || !isfinite(cw2) || !isfinite(vxc) || !isfinite(vyc);
  // item 1: sound waves (squared rate); item 2: fluid motion; item 3:
  // artificial viscosity on compressed directions
  const double r1s = cw2 * C.iL2;
  const double ux = fmax(fabs(vxc - vb), fabs(vxp - vb));
  const double uy = fmax(fabs(vyc), fabs(vyp));
  double r2 = fmax(ux * C.iLx, uy * C.iLy);
  const double dvx = vxp - vxc, dvy = vyp - vyc;
  // (an expansion gives a negative number, which the zero bounds)
  double r3 = fmax(fmax(0.0, C.k3 * -dvx * C.iLx), C.k3 * -dvy * C.iLy);
  if (D3) {
    bad |= !isfinite(vzc);
    const double uz = fmax(fabs(vzc), fabs(vzp));
    r2 = fmax(r2, uz * C.iLz);
    const double dvz = vzp - vzc;
    r3 = fmax(r3, C.k3 * -dvz * C.iLz);
  }
  double rate2 = r1s + r2 * r2 + r3 * r3;
  if (!D3 && !ADI) { // item 4: viscosity, 4 nu / Delta^2 (nu = 0 without)
    const double r4 = 4.0 * nu * C.iL2;
    rate2 += r4 * r4;
  }
  if (!(rate2 >= 0.0)) bad = 1;
  return rate2;
}

// Eq. 38 between a zone and its radial neighbour.  An infinite quotient, of an
// infinite velocity or of one too large for the zone's length, which div_by would
// turn into a NaN, sets *inf (its shear rate is infinite).
__device__ inline double shear_rate(const CflRing &C, double vxc, double vxn, int &inf) {
#pragma clang fp contract(off)
  inf |= __builtin_isinf(vxc * C.iLx) | __builtin_isinf(vxn * C.idXp);
  return fabs(div_by(vxc, C.Lx, C.iLx) - div_by(vxn, C.dXp, C.idXp));
}

// Two consecutive zones of a row, at any zone.
template <typename R>
using Pair = R __attribute__((ext_vector_type(2), aligned(sizeof(R))));

// LDS elements a ring of n zones takes: its v_x, the first zone's again after
// the last, and what the last pair of lanes reads beyond it.
__host__ __device__ inline int cfl_vlen(int n) { return (n + 7) & ~1; }

// The time-step pass.  A ring belongs to one wave (W = 1: no barrier, and the
// waves of a compute unit hide each other's loads), or to a workgroup of four
// (W = 4: rings too few to fill the chip, or too long for one wave's LDS).  A
// lane takes two consecutive zones of every 128-zone chunk.  First the ring's
// v_x goes to LDS, which gives v0 and later each zone's two X faces; then the
// other fields are streamed past it, the next chunk's loads in flight while
// one is computed.  Bound by memory: it reads 5 fields on 3D meshes, 5.8 TB/s
// on the 2048 x 768 x 96 disk in FP64.  Against a workgroup per ring that held
// it in registers (two divisions a zone): 1.50 to 1.05 ms there, FP32 1.31 to
// 0.59; 1536 x 512 x 128 1.02 to 0.73; 3072 x 1024 46 to 22 us; box of 160 x 144
// x 120 58 to 33; the FP32 batch of 256 disks 658 us in six launches to 297 in
// one.  On a few hundred rings latency is all there is (384 x 128: 5.0 to 5.7
// us).
// Rings come in XCD-contiguous logical order, by tiles of 16 planes with k
// fastest within a tile: the rings holding a ring's k + 1 and j + 1 neighbours
// (v_z and v_y on its upper faces) were read one and 16 rings earlier, still
// in L2 except across a tile boundary.  (Four rings in a row per wave, for a
// quarter of the slots, measured 666 against 594 us in FP32.)
// The state may be stored in FP32 (R = float); the time step is always formed
// in FP64 from the stored values.
template <int W, bool CFL, bool D3, bool ADI, typename R>
__device__ __forceinline__ void cfl_body(Mesh m, StateT<R> s, double *__restrict__ v0,
                                         double *__restrict__ ringrate, double *__restrict__ ringshear,
                                         int *__restrict__ err, unsigned bid_, unsigned nbk_) {
#pragma clang fp contract(off)
  extern __shared__ double cfl_lds[];
  __shared__ double red[W == 1 ? 1 : 3 * MAXW];
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = m.nx, nc = (n + 127) >> 7;
  // (V[-1] takes the unused half of a one-zone ring's pair)
  R *V = reinterpret_cast<R *>(cfl_lds) + (W == 1 ? wv * cfl_vlen(n) : 0) + 2;
  const unsigned blk = xcd_remap(bid_, nbk_);
  const int L = (int)(W == 1 ? blk * (blockDim.x >> 6) + (unsigned)wv : blk);
  if (L >= m.nring) return;
  const unsigned py = (unsigned)m.pitch, pz = (unsigned)m.plane();
  const R *qf = ADI ? s.e : s.cs, *nuf = !D3 && !ADI && m.visc ? s.nu : qf;
  constexpr int KT = 16;
  // A row's pair of zones for chunk c: past the ring's end, and on the last
  // zone of an odd ring, the ring's last two zones.  (No branch: every load of
  // a chunk is issued before the first one is waited for.  A ring of one zone
  // has it second in the pair, and no use for the first.)
  auto zone = [&](int c) { return 128 * c + 2 * lane; };
  auto at = [&](int c) { return min(zone(c), n - 2); };
  auto ld = [&](const R *row, int c) { return *reinterpret_cast<const Pair<R> *>(row + at(c)); };
  struct Chunk {
    Pair<R> r, q, y0, y1, z0, z1, nu, s;
  };
  const bool visc = !D3 && !ADI && m.visc;
  double rmax = 0.0, smax = 0.0;
  int bad = 0, inf = 0;
  const unsigned tile = (unsigned)L / ((unsigned)m.ny * KT), q = (unsigned)L % ((unsigned)m.ny * KT);
  const int kb = (int)tile * KT, kt = min(KT, m.nz - kb);
  const int kk = kb + (int)(q % (unsigned)kt), jj = (int)(q / (unsigned)kt);
  const int j = m.j0 + jj, k = m.k0 + kk;
  const int r = kk * m.ny + jj; // ring index (k - k0) * ny + (j - j0)
  const unsigned base = m.o32(0, j, k);
  const bool shear_on = CFL && m.fargo && m.shear_c0 > 0.0 && j + 1 < m.jn;
  const unsigned ps = shear_on ? py : 0u; // the next ring, or this one again
  auto load = [&](int c, Chunk &z) {
    z.r = ld(s.rho + base, c);
    z.q = ld(qf + base, c);
    z.y0 = ld(s.vy + base, c);
    z.y1 = ld(s.vy + base + py, c);
    if (D3) {
      z.z0 = ld(s.vz + base, c);
      z.z1 = ld(s.vz + base + pz, c);
    }
    if (!D3 && !ADI) z.nu = ld(nuf + base, c);
    z.s = ld(s.vx + base + ps, c);
  };
  // v_x into LDS, with its extremes, four chunks at a time (chunks past the
  // ring's end read its last zones again, which changes neither); the first
  // chunk's other fields are on their way before a v_x is used
  double vmax = -HUGE_VAL, vmin = HUGE_VAL;
  Chunk z[2];
  const int c0 = W == 1 ? 0 : wv;
  auto vx_load = [&](int c, Pair<R> (&x)[4]) {
#pragma unroll
    for (int u = 0; u < 4; u++) x[u] = ld(s.vx + base, c + u * W);
  };
  auto vx_take = [&](int c, Pair<R> (&x)[4]) {
#pragma unroll
    for (int u = 0; u < 4; u++) {
      if (n == 1) x[u].x = x[u].y;
      vmax = fmax(vmax, fmax((double)x[u].x, (double)x[u].y));
      vmin = fmin(vmin, fmin((double)x[u].x, (double)x[u].y));
      *reinterpret_cast<Pair<R> *>(V + at(c + u * W)) = x[u];
    }
  };
  {
    Pair<R> x[4];
    vx_load(c0, x);
    if (CFL) load(c0, z[0]);
    vx_take(c0, x);
    if (c0 == 0 && lane == 0) V[n] = x[0].x;
#pragma unroll 1
    for (int c = c0 + 4 * W; c < nc; c += 4 * W) {
      vx_load(c, x);
      vx_take(c, x);
    }
  }
  // an FP32 v_x is a deviation from the ring's FP64 background: the full
  // velocity is formed in FP64 (adding it is monotone, so the extremes of
  // the sums are the sums of the extremes)
  const double vbg = sizeof(R) == 4 ? m.bg(BG_V, j, k) : 0.0;
  const double vbg_p = sizeof(R) == 4 && shear_on ? m.bg(BG_V, j + 1, k) : 0.0;
  if (W == 1) {
    vmax = lane63(wave_reduce_dpp(vmax, Max(), -HUGE_VAL));
    vmin = lane63(wave_reduce_dpp(vmin, Min(), HUGE_VAL));
    // the wave's own LDS writes are seen by all of its lanes
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  } else {
    block_reduce2(vmax, Max(), -HUGE_VAL, vmin, Min(), HUGE_VAL, red);
  }
  double vb_ring = 0.5 * ((vmax + vbg) + (vmin + vbg));
  if (m.v0_mean) { // summed by every wave in one order, whatever W
    double a = 0.0;
    for (int i = lane; i < n; i += 64) a += (double)V[i] + vbg;
    for (int o = 32; o > 0; o >>= 1) a += __shfl_xor(a, o, 64);
    vb_ring = a / n;
  }
  if (tid == (W == 1 ? 64 * wv : 0)) v0[r] = vb_ring;
  if (CFL) {
    const double vb = m.fargo ? vb_ring : 0.0;
    // the smallest step is 1 / sqrt of the largest sum of squared rates
    // (taken in dt_of_extremes)
    const CflRing C = cfl_ring(m, j, k, shear_on);
    double sring = 0.0;
    auto one = [&](double x0, double x1, R rho, R q, R y0, R y1, R z0, R z1, R nu, R xs) {
      const double vxc = x0 + vbg, vxp = x1 + vbg;
      const double rate2 = zone_rate2<D3, ADI>(C, vb, vxc, vxp, (double)rho, (double)q, (double)y0, (double)y1,
                                               (double)z0, (double)z1, visc ? (double)nu : 0.0, m.gamma, bad);
      if (rate2 >= 0.0) rmax = rate2 > rmax ? rate2 : rmax;
      const double sh = shear_rate(C, vxc, (double)xs + vbg_p, inf);
      sring = sh > sring ? sh : sring;
    };
    // (every lane takes its pair, so that no load of a chunk outlives it; a
    // lane past the ring's end takes the last zones once more)
    auto zones = [&](int c, const Chunk &z) {
      const int i = at(c);
      const Pair<R> x = *reinterpret_cast<const Pair<R> *>(V + i);
      const double x0 = (double)x.x, x1 = (double)x.y, x2 = (double)V[i + 2];
      one(x1, x2, z.r.y, z.q.y, z.y0.y, z.y1.y, D3 ? z.z0.y : R(0), D3 ? z.z1.y : R(0), z.nu.y, z.s.y);
      if (n > 1) one(x0, x1, z.r.x, z.q.x, z.y0.x, z.y1.x, D3 ? z.z0.x : R(0), D3 ? z.z1.x : R(0), z.nu.x, z.s.x);
    };
#pragma unroll 1
    for (int c = c0; c < nc; c += 2 * W) {
      load(c + W, z[1]);
      zones(c, z[0]);
      if (c + W >= nc) break;
      load(c + 2 * W, z[0]);
      zones(c + W, z[1]);
    }
    if (shear_on) smax = inf ? HUGE_VAL : (sring > smax ? sring : smax);
  }
  if (!CFL) return;
  if (W == 1) {
    rmax = wave_reduce_dpp(rmax, Max(), 0.0);
    smax = wave_reduce_dpp(smax, Max(), 0.0);
    const bool anybad = __builtin_amdgcn_ballot_w64(bad != 0) != 0;
    if (lane == 63) {
      ringrate[L] = rmax; // the ring's largest squared rate
      ringshear[L] = smax;
      if (anybad) atomicOr(err, 1);
    }
  } else {
    int anybad = bad;
    block_reduce2(rmax, Max(), 0.0, smax, Max(), 0.0, red, &anybad);
    if (tid == 0) {
      ringrate[L] = rmax;
      ringshear[L] = smax;
      if (anybad) atomicOr(err, 1);
    }
  }
}
constexpr int CFL_BS1 = 128; // threads of a workgroup with W = 1: two waves
// CFL: the rates as well as v0
template <int W, bool CFL, bool D3, bool ADI, typename R>
__global__ __launch_bounds__(W == 1 ? CFL_BS1 : 256) void k_cfl_ring(Mesh m, StateT<R> s, double *__restrict__ v0,
                                                                     double *__restrict__ ringrate,
                                                                     double *__restrict__ ringshear,
                                                                     int *__restrict__ err) {
  cfl_body<W, CFL, D3, ADI, R>(m, s, v0, ringrate, ringshear, err, blockIdx.x, gridDim.x);
}

// One wave per ring (else four) where there are at least two rings per SIMD of
// the chip (a few hundred rings, 633 or 768 zones each: 6.6 and 7.2 us with
// four waves, 7.4 and 7.7 with one; 17280 rings of 160 zones 89 and 36 us, 7181
// of 501 in FP32 48 and 22) and a ring takes at most 10 KB, so that the LDS of a
// compute unit holds the sixteen waves its registers do (65536 rings of 1536
// doubles: 726 us with four waves, 744 with one; 73728 of 2048: 1049 and 1090,
// in FP32, 8 KB a ring, 702 and 594).
inline bool cfl_wave(const Mesh &m, size_t elem) { return m.nring >= 2048 && (size_t)m.nx * elem <= 10240; }

// Rings longer than one workgroup holds, in segments of CFL_SEG zones (256
// threads, four zones each).  First each segment's largest and smallest
// full v_x (or its sum, for the mean), then each segment combines its ring's
// entries into v0 (min/max exactly; the mean as the sum of the
// segment sums in segment order, over nx) and takes Eq. cfl2 on its zones,
// with the v_x of the zone after its last read from memory.
template <typename R>
__device__ inline double full_vx(const Mesh &m, const StateT<R> &s, unsigned c, double vbg) {
  return (double)s.vx[c] + vbg;
}

template <typename R>
__global__ __launch_bounds__(256) void k_bulk_seg(Mesh m, StateT<R> s) {
  constexpr int M = CFL_SEG / 256;
  __shared__ double red[2 * MAXW];
  const int r = (int)(blockIdx.x / (unsigned)m.cseg), g = (int)(blockIdx.x % (unsigned)m.cseg);
  const int j = m.j0 + r % m.ny, k = m.k0 + r / m.ny;
  const unsigned base = m.o32(0, j, k);
  const double vbg = sizeof(R) == 4 ? m.bg(BG_V, j, k) : 0.0;
  const int i0 = g * CFL_SEG, i1 = min(i0 + CFL_SEG, m.nx);
  double a = m.v0_mean ? 0.0 : -HUGE_VAL, b = HUGE_VAL;
#pragma unroll
  for (int mm = 0; mm < M; mm++) {
    const int i = i0 + (int)threadIdx.x + 256 * mm;
    if (i >= i1) continue;
    const double v = full_vx(m, s, base + (unsigned)i, vbg);
    if (m.v0_mean) a += v;
    else {
      a = v > a ? v : a;
      b = v < b ? v : b;
    }
  }
  if (m.v0_mean) {
    a = block_reduce(a, Add(), 0.0, red);
    b = 0.0;
  } else {
    block_reduce2(a, Max(), -HUGE_VAL, b, Min(), HUGE_VAL, red);
  }
  if (threadIdx.x == 0) {
    m.segmm[2 * (size_t)blockIdx.x] = a;
    m.segmm[2 * (size_t)blockIdx.x + 1] = b;
  }
}

template <bool D3, bool ADI, typename R>
__global__ __launch_bounds__(256) void k_cfl_seg(Mesh m, StateT<R> s, int with_cfl, double *__restrict__ v0,
                                                 double *__restrict__ ringrate, double *__restrict__ ringshear,
                                                 int *__restrict__ err) {
#pragma clang fp contract(off)
  constexpr int M = CFL_SEG / 256;
  __shared__ double red[3 * MAXW];
  __shared__ double V[CFL_SEG + 1]; // the segment's full v_x and the next zone's
  const int r = (int)(blockIdx.x / (unsigned)m.cseg), g = (int)(blockIdx.x % (unsigned)m.cseg);
  const int j = m.j0 + r % m.ny, k = m.k0 + r / m.ny;
  const int tid = threadIdx.x, n = m.nx;
  const unsigned base = m.o32(0, j, k);
  const bool shear_on = with_cfl && m.fargo && m.shear_c0 > 0.0 && j + 1 < m.jn;
  double vbg = 0.0, vbg_p = 0.0;
  if constexpr (sizeof(R) == 4) {
    vbg = m.bg(BG_V, j, k);
    if (shear_on) vbg_p = m.bg(BG_V, j + 1, k);
  }
  // the ring's bulk velocity from its segments' entries
  double a = m.v0_mean ? 0.0 : -HUGE_VAL, b = HUGE_VAL;
  const double *e = m.segmm + 2 * (size_t)r * m.cseg;
  if (m.v0_mean) {
    if (tid == 0)
      for (int q = 0; q < m.cseg; q++) a += e[2 * q];
    a = block_reduce(tid == 0 ? a : 0.0, Add(), 0.0, red);
  } else {
    for (int q = tid; q < m.cseg; q += 256) {
      a = e[2 * q] > a ? e[2 * q] : a;
      b = e[2 * q + 1] < b ? e[2 * q + 1] : b;
    }
    block_reduce2(a, Max(), -HUGE_VAL, b, Min(), HUGE_VAL, red);
  }
  const double vb_ring = m.v0_mean ? a / n : 0.5 * (a + b);
  if (g == 0 && tid == 0) v0[r] = vb_ring;
  if (!with_cfl) return;
  const int i0 = g * CFL_SEG, i1 = min(i0 + CFL_SEG, n);
  for (int i = i0 + tid; i <= i1; i += 256) V[i - i0] = full_vx(m, s, base + (unsigned)(i == n ? 0 : i), vbg);
  __syncthreads();
  const double vb = m.fargo ? vb_ring : 0.0;
  const CflRing C = cfl_ring(m, j, k, shear_on);
  const unsigned py = (unsigned)m.pitch, pz = (unsigned)m.plane();
  const R *qf = ADI ? s.e : s.cs;
  double rmax = 0.0, smax = 0.0;
  int bad = 0, inf = 0;
#pragma unroll
  for (int mm = 0; mm < M; mm++) {
    const int i = i0 + tid + 256 * mm;
    if (i >= i1) continue;
    const unsigned c = base + (unsigned)i;
    const double vxc = V[i - i0], vxp = V[i - i0 + 1];
    const double rate2 = zone_rate2<D3, ADI>(C, vb, vxc, vxp, (double)s.rho[c], (double)qf[c], (double)s.vy[c],
                                             (double)s.vy[c + py], D3 ? (double)s.vz[c] : 0.0,
                                             D3 ? (double)s.vz[c + pz] : 0.0,
                                             !D3 && !ADI && m.visc ? (double)s.nu[c] : 0.0, m.gamma, bad);
    if (rate2 >= 0.0) rmax = rate2 > rmax ? rate2 : rmax;
    if (shear_on) {
      const double sh = shear_rate(C, vxc, (double)s.vx[c + py] + vbg_p, inf);
      if (sh > smax) smax = sh;
    }
  }
  if (inf) smax = HUGE_VAL;
  int anybad = bad;
  block_reduce2(rmax, Max(), 0.0, smax, Max(), 0.0, red, &anybad);
  if (tid == 0) {
    ringrate[blockIdx.x] = rmax;
    ringshear[blockIdx.x] = smax;
    if (anybad) atomicOr(err, 1);
  }
}

// dt from the slots into the device word: one workgroup, every wave a share of
// the slots.
__device__ __forceinline__ void dt_final_body(const DtSlots &in, const DevWords &w) {
  __shared__ double red[2 * MAXW];
  double rmax, smax;
  slot_extremes(in, threadIdx.x, blockDim.x, rmax, smax);
  block_reduce2(rmax, Max(), 0.0, smax, Max(), 0.0, red);
  bool bad;
  const double dt = dt_of_extremes(in, rmax, smax, &bad);
  if (threadIdx.x == 0) {
    if (bad) atomicOr(w.err, 2);
    *w.dt = dt;
  }
}
__global__ __launch_bounds__(1024) void k_dt_final(DtSlots in, DevWords w) { dt_final_body(in, w); }

// The slots' extremes by groups of consecutive slots, one block per group (a
// workgroup alone reads at the rate of its compute unit, 40 GB/s).
__global__ __launch_bounds__(256) void k_dt_groups(const double *__restrict__ rate, const double *__restrict__ shear,
                                                   int nslot, int per, double *__restrict__ out) {
  __shared__ double red[2 * MAXW];
  double rmax = 0.0, smax = 0.0;
  const int r1 = min(nslot, ((int)blockIdx.x + 1) * per);
#pragma unroll 4
  for (int r = blockIdx.x * per + threadIdx.x; r < r1; r += 256) {
    const double a = rate[r], b = shear[r];
    rmax = a > rmax ? a : rmax;
    smax = b > smax ? b : smax;
  }
  block_reduce2(rmax, Max(), 0.0, smax, Max(), 0.0, red);
  if (threadIdx.x == 0) {
    out[blockIdx.x] = rmax;
    out[DT_GROUPS + blockIdx.x] = smax;
  }
}

// multi-mesh forms (ManyGrid)
template <typename R>
struct CflArgs {
  Mesh m;
  StateT<R> s;
  double *v0, *ringrate, *ringshear;
  int *err;
  unsigned nb;
};
// (a wave per ring whatever the mesh: a batch has rings enough)
template <bool ADI, typename R>
__global__ __launch_bounds__(CFL_BS1) void k_cfl_ring_many(const void *args, const uint2 *tab) {
  const uint2 t = many_block(tab);
  if (t.x == MANY_NONE) return;
  const CflArgs<R> a = many_args<CflArgs<R>>(args, t.x);
  cfl_body<1, true, false, ADI, R>(a.m, a.s, a.v0, a.ringrate, a.ringshear, a.err, t.y, a.nb);
}
struct DtArgs {
  DtSlots in;
  DevWords w;
};
__global__ __launch_bounds__(256) void k_dt_final_many(const void *args, const uint2 *tab) {
  const uint2 t = many_block(tab);
  if (t.x == MANY_NONE) return;
  const DtArgs a = many_args<DtArgs>(args, t.x);
  dt_final_body(a.in, a.w);
}

// The split of Eq. 29, one thread per ring, with dt given by value or, if
// dtp is not null, read from the device.
__global__ __launch_bounds__(256) void k_split(Mesh m, const double *__restrict__ v0, const double *__restrict__ dtp,
                                               double dtv, int32_t *__restrict__ N, double *__restrict__ xi) {
#pragma clang fp contract(off)
  int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= m.nring) return;
  const double dt = dtp ? *dtp : dtv;
  int j = m.j0 + r % m.ny, k = m.k0 + r / m.ny;
  double D = (v0[r] * dt) / m.DX(j, k);
  double rn = round(D);
  N[r] = (int32_t)rn;
  xi[r] = D - rn;
}

} // namespace

void launch_set_dt(Launch &L, const DevWords &w, double dt) {
  prof_begin(L, K_SET_DT);
  k_set_dt<<<1, 1, 0, L.s>>>(w, dt);
  prof_end(L, K_SET_DT);
}

template <typename R>
void launch_cfl(Launch &L, const Mesh &m, const StateT<R> &s, int with_cfl, double *v0, double *ringrate,
                double *ringshear, int *err) {
  prof_begin(L, K_CFL);
  auto go = [&](auto d3, auto adi) {
    constexpr bool D3 = decltype(d3)::value, ADI = decltype(adi)::value;
    if (m.cseg > 1) { // rings in segments
      const unsigned nb = (unsigned)m.nring * (unsigned)m.cseg;
      k_bulk_seg<R><<<nb, 256, 0, L.s>>>(m, s);
      k_cfl_seg<D3, ADI, R><<<nb, 256, 0, L.s>>>(m, s, with_cfl, v0, ringrate, ringshear, err);
      return;
    }
    const bool wave = cfl_wave(m, sizeof(R));
    const unsigned per = wave ? CFL_BS1 / 64 : 1, nb = ((unsigned)m.nring + per - 1) / per;
    const size_t lds = (size_t)per * cfl_vlen(m.nx) * sizeof(R);
    auto w = [&](auto wt) {
      constexpr int W = decltype(wt)::value, BS = W == 1 ? CFL_BS1 : 256;
      if (with_cfl) k_cfl_ring<W, true, D3, ADI, R><<<nb, BS, lds, L.s>>>(m, s, v0, ringrate, ringshear, err);
      else k_cfl_ring<W, false, false, false, R><<<nb, BS, lds, L.s>>>(m, s, v0, ringrate, ringshear, err);
    };
    if (wave) w(std::integral_constant<int, 1>{});
    else w(std::integral_constant<int, 4>{});
  };
  auto by_eos = [&](auto d3) {
    if (m.eos == FARGO_ADIABATIC) go(d3, std::true_type{});
    else go(d3, std::false_type{});
  };
  if (m.d3) by_eos(std::true_type{});
  else by_eos(std::false_type{});
  prof_end(L, K_CFL);
}

template void launch_cfl<double>(Launch &, const Mesh &, const StateT<double> &, int, double *, double *, double *,
                                 int *);
template void launch_cfl<float>(Launch &, const Mesh &, const StateT<float> &, int, double *, double *, double *,
                                int *);

DtIn launch_dt(Launch &L, const Mesh &m, const DevWords &w, const double *ringrate, const double *ringshear,
               double *scratch, bool in_word) {
  DtIn in{ringrate, ringshear, m.nring * m.cseg};
  if (in.nslot <= DT_SLOTS && !m.d3 && !in_word) return in;
  prof_begin(L, K_DT_FINAL);
  // by groups first where one workgroup would read for longer than a second
  // launch takes (17280 slots: 8.7 us alone, 9.4 by groups; 73728: 30 and 9.4)
  if (in.nslot > 20000) {
    const int per = (in.nslot + DT_GROUPS - 1) / DT_GROUPS;
    k_dt_groups<<<DT_GROUPS, 256, 0, L.s>>>(ringrate, ringshear, in.nslot, per, scratch);
    in = DtIn{scratch, scratch + DT_GROUPS, DT_GROUPS};
  }
  k_dt_final<<<1, in.nslot > 64 ? 1024 : 64, 0, L.s>>>(dt_slots(m, in), w);
  prof_end(L, K_DT_FINAL);
  return DtIn{nullptr, nullptr, 0};
}

void launch_split(Launch &L, const Mesh &m, const double *v0, double dt, int32_t *N, double *xi) {
  prof_begin(L, K_SPLIT);
  k_split<<<(m.nring + 255) / 256, 256, 0, L.s>>>(m, v0, nullptr, dt, N, xi);
  prof_end(L, K_SPLIT);
}

template <typename R>
size_t cfl_args_bytes() { return sizeof(CflArgs<R>); }

template <typename R>
unsigned cfl_args(const Mesh &m, const StateT<R> &s, double *v0, double *ringrate, double *ringshear, int *err,
                  void *dst) {
  const unsigned nb = (unsigned)((m.nring + CFL_BS1 / 64 - 1) / (CFL_BS1 / 64));
  *(CflArgs<R> *)dst = CflArgs<R>{m, s, v0, ringrate, ringshear, err, nb};
  return nb;
}

template <typename R>
void launch_cfl_many(Launch &L, const Mesh &m0, const ManyGrid &g, int nxmax) {
  prof_begin(L, K_CFL);
  const size_t sh = (size_t)(CFL_BS1 / 64) * cfl_vlen(nxmax) * sizeof(R);
  if (m0.eos == FARGO_ADIABATIC) k_cfl_ring_many<true, R><<<g.nblk, CFL_BS1, sh, L.s>>>(g.args, g.tab);
  else k_cfl_ring_many<false, R><<<g.nblk, CFL_BS1, sh, L.s>>>(g.args, g.tab);
  prof_end(L, K_CFL);
}

size_t dt_final_args_bytes() { return sizeof(DtArgs); }

unsigned dt_final_args(const Mesh &m, const DevWords &w, const double *ringrate, const double *ringshear, void *dst) {
  *(DtArgs *)dst = DtArgs{dt_slots(m, DtIn{ringrate, ringshear, m.nring}), w};
  return 1;
}

void launch_dt_final_many(Launch &L, const ManyGrid &g) {
  prof_begin(L, K_DT_FINAL);
  k_dt_final_many<<<g.nblk, 256, 0, L.s>>>(g.args, g.tab);
  prof_end(L, K_DT_FINAL);
}

template unsigned cfl_args<double>(const Mesh &, const StateT<double> &, double *, double *, double *, int *, void *);
template unsigned cfl_args<float>(const Mesh &, const StateT<float> &, double *, double *, double *, int *, void *);
template size_t cfl_args_bytes<double>();
template size_t cfl_args_bytes<float>();
template void launch_cfl_many<double>(Launch &, const Mesh &, const ManyGrid &, int);
template void launch_cfl_many<float>(Launch &, const Mesh &, const ManyGrid &, int);

} // namespace fargo
