// Box 7: source step (Sect. 3.3), boxes 7a, 7b and 7c fused in one pass.
//   7a  pressure and potential gradients on the owned faces, centrifugal
//       terms as squares of four-point arithmetic averages (Eq. 12 and its
//       generalisation); Jacobi: every face reads only v^n.  The pressure
//       term uses the arithmetic mean of the two face densities (Eq. 20),
//       which makes it momentum conserving (Eqs. 21-25).
//   7b  von Neumann-Richtmyer artificial viscosity per direction,
//       q = C^2 rho dv^2 where dv < 0, its gradient in the same conservative
//       form, and the heating -q dv / L.
//   7c  compressional heating of a gamma-law gas, time-centred:
//       e <- e (1 - a)/(1 + a), a = dt (gamma - 1) div(v) / 2.
// A zone owns its lower X, Y and Z faces (the lower Y/Z boundary face only in
// a periodic direction); faces that are not owned keep v^n.  Results go to
// separate arrays (v'', e''), so the pass reads the state while it writes.
//
// Layout of the work on 3D meshes (2D meshes: k_source2): a workgroup takes a
// tile of TX x TY zones of one (X, Y) plane and marches through the Z planes.  For each plane the tile and a halo
// of two zones in X and Y are staged in LDS; the v' of every X and Y face of
// the tile (and of the halo faces its stencil needs) is computed once and
// kept in LDS (with the reciprocal of its density sum where room is left),
// then each zone forms q on its neighbours and its v'' and e''.  Along Z each
// thread keeps a sliding window of its own column in registers (planes
// k-1 .. k+2), which also
// supplies the tile's interior values to LDS, so each interior value is read
// from memory once.  Geometric lengths enter through reciprocal tables.
//
// The field type F is double, or float for the FP32-bulk state; arithmetic is
// carried out in F, geometric factors are rounded to F where they are used.
// An FP32 v_x is a deviation from its ring's FP64 background vb: the X-face
// update acts on it unchanged, and each centrifugal term splits into the
// square of the background (vb + R Omega), formed in FP64 together with the
// potential gradient it nearly cancels and rounded once, and the FP32 terms
// of the deviation.
#include <type_traits>

#include "fargo_internal.h"

namespace fargo {

namespace {

constexpr int TX = 64, SX = TX + 4; // tile width, with two halo zones on each side
// Tile height (one wave per tile row).  The Y halo of a tile is read once per
// tile, so taller tiles read less of it.  The FP64 3D march takes 16 rows
// (1024 threads, at most 128 registers a thread), or 12 where the spherical or
// adiabatic terms need more registers; FP32 marches take 8 (two workgroups per
// compute unit, three with neither an energy nor the spherical terms; measured
// slower with taller tiles).
template <typename F, int GEO, bool ADI>
constexpr int tile_rows() {
  if (sizeof(F) == 4) return 8;
  return ADI || GEO == FARGO_SPHERICAL ? 12 : 16;
}
template <typename F, int GEO, bool ADI>
constexpr int src_threads() { return 64 * tile_rows<F, GEO, ADI>(); }
// minimum waves per SIMD: one workgroup of the FP64 march per compute unit,
// at least four waves of the others
template <typename F, int GEO, bool ADI>
constexpr int src_waves() {
  return sizeof(F) == 8 ? src_threads<F, GEO, ADI>() / 256 : 4;
}

template <typename F>
__device__ inline F qvisc(F c2, F rho, F dv) { return dv < F(0) ? c2 * rho * dv * dv : F(0); }

template <typename F, int TY, bool SPH, bool KI>
struct Lds {
  // staging of a plane (NB planes in flight; density one more)
  static constexpr int SY = TY + 4, NB = 2, NR = NB + 1;
  F R[NR][SY][SX];      // density
  F P[NB][SY][SX];      // pressure
  double Ph[NB][SY][SX]; // potential (FP64 in every mode)
  F VX[NB][SY][SX];     // v_x on the lower X face of each zone slot
  F VY[NB][SY][TX];     // v_y on the lower Y face of each zone slot
  F VT[SPH ? NB : 1][SPH ? SY : 1][SPH ? TX : 1]; // spherical: v_theta on the zone's two Z faces, summed
  // v' of the faces of a plane (NB planes in flight)
  F AX[NB][TY][SX];     // v'_x of X faces of the tile rows
  F AY[NB][SY][TX];     // v'_y of Y faces
  F IX[KI ? NB : 1][KI ? TY : 1][KI ? SX : 1]; // KI: 1 / ((rho_i + rho_{i-1}) dX) on the X faces
  F IY[KI ? NB : 1][KI ? SY : 1][KI ? TX : 1]; // KI: 1 / ((rho_j + rho_{j-1}) h_y) on the Y faces
  double DX[NB][TY];    // 1 / dX of the tile rows, for the halo X faces
};
constexpr size_t LDS_CU = 160 * 1024;
// The reciprocals of the faces' density sums are kept in LDS where they fit
// beside the rest, else formed again by the zones that use them (the same bits);
// formed again also where a compute unit then holds one workgroup more: FP32
// without the spherical terms and, for its registers (73, with an energy 97),
// without an energy.  2048 x 768 x 96: 1.85 to 1.47 ms; where no workgroup is
// gained it costs (501 x 167 x 43 spherical 72 to 77 us).
template <typename F, int TY, bool SPH, bool ADI>
constexpr bool keep_inv() {
  constexpr size_t with = sizeof(Lds<F, TY, SPH, true>), without = sizeof(Lds<F, TY, SPH, false>);
  return with <= LDS_CU && (sizeof(F) == 8 || ADI || LDS_CU / without == LDS_CU / with);
}

// An explicit register move.  The march keeps a window of plane records in
// registers and rotates it once per plane; moving the newest record out of its
// registers before the next plane's loads are issued lets those loads write
// the same registers, instead of temporaries whose copy into the window would
// wait for the loads to arrive.
template <typename T>
__device__ inline T vmove(T x) {
  T y;
  if constexpr (sizeof(T) == 8) asm("v_mov_b64 %0, %1" : "=v"(y) : "v"(x));
  else asm("v_mov_b32 %0, %1" : "=v"(y) : "v"(x));
  return y;
}

// A value the compiler is to keep in vector registers (every lane of a wave
// holding the same value), which leaves the scalar registers to the values
// that change along the march.
template <typename T>
__device__ inline T vreg(T x) {
  asm("" : "+v"(x));
  return x;
}

// one zone's values in one plane
template <typename F>
struct Zv {
  F rho, q; // q: sound speed (isothermal) or internal energy (adiabatic)
  double pot;
  F vz, vx, vxp; // vxp: v_x on the next X face
};

// Ghost rows that carry v^n and e into v'' and e'': those of FIXED sides (box
// 9 fills the others), and next to the Y sides those that box 7d reads first.
// Y ghost rows of planes [ka, kb) (extended over FIXED Z sides), then the Z
// ghost planes of rows [jt, jt + h); y0, y1: whether the Y sides belong to it.
__host__ __device__ inline bool ghost_rows(const Mesh &m, int side) { // of a Y side
  return m.visc || m.bc[side] == FARGO_BC_FIXED;
}
struct GhostRows {
  int jn, kn, nyl, nyr, nzl, nzr, kl, nk;
  __host__ __device__ GhostRows(const Mesh &m, bool y0, bool y1, int ka, int kb) : jn(m.jn), kn(m.kn) {
    nyl = y0 && ghost_rows(m, 0) ? NGH : 0;
    nyr = nyl + (y1 && ghost_rows(m, 1) ? NGH : 0);
    nzl = m.d3 && ka == m.k0 && m.bc[2] == FARGO_BC_FIXED ? NGH : 0;
    nzr = nzl + (m.d3 && kb == m.kn && m.bc[3] == FARGO_BC_FIXED ? NGH : 0);
    kl = ka - nzl;
    nk = kb + (nzr - nzl) - kl;
  }
  __host__ __device__ int rows(int jt, int h) const { return nyr * nk + nzr * h; }
  __device__ void row(int t, int jt, int h, int &j, int &k) const {
    if (t < nyr * nk) {
      const int q = t % nyr;
      j = q < nyl ? q : jn + q - nyl;
      k = kl + t / nyr;
    } else {
      t -= nyr * nk;
      const int q = t % nzr;
      j = jt + t / nzr;
      k = q < nzl ? q : kn + q - nzl;
    }
  }
};
template <typename F, bool D3, bool ADI>
__device__ inline void carry_ghost(const StateT<F> &s, unsigned o, F *__restrict__ vx2, F *__restrict__ vy2,
                                   F *__restrict__ vz2, F *__restrict__ e2) {
  const F a = s.vx[o], b = s.vy[o], d = D3 ? s.vz[o] : F(0), e = ADI ? s.e[o] : F(0);
  vx2[o] = a;
  vy2[o] = b;
  if (D3) vz2[o] = d;
  if (ADI) e2[o] = e;
}

// A plane goes through three phases: staging into LDS (S), v' of its faces
// (F), and the zones (Z).  The march is software-pipelined over planes: one
// barrier interval runs Z(k), F(k+1) and S(k+2) on separate buffers, so each
// plane costs one barrier and the three phases overlap.
// The geometry and the equation of state are template parameters: fewer
// run-time conditions leave more scalar registers for the march.
template <typename F, int GEO, bool ADI>
__device__ __forceinline__ void source_body(Mesh m, StateT<F> s, DevWords dw, F *__restrict__ vx2, F *__restrict__ vy2, F *__restrict__ vz2,
                                                  F *__restrict__ e2, int nbx, int nby, int zlen, int ghosts,
                                                  unsigned bid_, unsigned nbk_) {
  constexpr int TY = tile_rows<F, GEO, ADI>();
  constexpr bool KI = keep_inv<F, TY, GEO == FARGO_SPHERICAL, ADI>();
  __shared__ Lds<F, TY, GEO == FARGO_SPHERICAL, KI> L;
  static_assert(sizeof(L) <= LDS_CU, "source step tile exceeds the LDS of a compute unit");
  // the row is the wave index: uniform, so that geometric factors of the
  // row come through scalar loads, which do not stall behind the prefetches
  const int tid = threadIdx.x, r = __builtin_amdgcn_readfirstlane(tid >> 6), c = tid & 63;
  // Tiles in groups of G tile rows, Y fastest within a group.  The 16-row
  // FP64 march takes groups of 4: the 32 workgroups an XCD runs at once then
  // cover a patch 8 tiles wide and 4 tall, so that the X halo zones a tile
  // reads (each a 128-byte line of its neighbour's row) are mostly a running
  // neighbour's own, still in L2 (2.60 to 2.36 ms on the 2048 x 768 x 96 disk).
  // The FP32 march takes groups of 4 as well:
  // 29 % fewer bytes fetched, about as fast.  The 12-row march keeps Y fastest
  // over the whole mesh (G = nby), which measured faster.
  const int G = TY == 16 || sizeof(F) == 4 ? 4 : nby;
  const unsigned Lc = xcd_remap(bid_, nbk_), ntile = (unsigned)(nbx * nby), gsz = (unsigned)(G * nbx);
  const unsigned zc = Lc / ntile, Lb = Lc % ntile;
  const unsigned grp = Lb / gsz, idx = Lb % gsz, gy = (unsigned)min(G, nby - (int)grp * G);
  const int ty = (int)(grp * (unsigned)G + idx % gy), tx = (int)(idx / gy);
  const int i0 = tx * TX, jt0 = m.j0 + ty * TY;
  // the workgroup's active planes
  const int k0 = m.k0 + (int)zc * zlen, kn = min(k0 + zlen, m.kn);
  const int w = min(TX, m.nx - i0), h = min(TY, m.jn - jt0);
  const bool act = r < h && c < w;
  const int i = i0 + c, j = jt0 + r;
  constexpr bool adi = ADI;
  constexpr bool sph = GEO == FARGO_SPHERICAL, cyl = GEO == FARGO_CYLINDRICAL;
  const F dt = vreg((F)*dw.dt);
  const F c2 = vreg((F)(m.cvnr * m.cvnr)), om = vreg((F)m.omega), gm1 = vreg((F)(m.gamma - 1.0));
  const unsigned plane = (unsigned)m.plane();
  // geometric factors of the thread's row (the products with the plane
  // factors are those of Mesh::Sx, Sy, Sz and Vinv); rows past the tile
  // read the last active row
  const int jg = min(j, m.jn - 1);
  const double g_sxj = vreg(m.g.sxj(jg)), g_syj = vreg(m.g.syj(jg)), g_syj1 = vreg(m.g.syj(jg + 1)),
               g_szj = vreg(m.g.szj(jg)), g_invVj = vreg(m.g.invVj(jg)), g_invLy = vreg(m.g.inv_Ly(jg)),
               g_iymed = vreg(m.g.inv_ymed(jg)), g_ymed = vreg(m.g.ymed(jg));

  // storage column of X slot sl (i0 - 2 + sl, periodic) and row of Y slot t
  auto xcol = [&](int sl) {
    int x = i0 - 2 + sl;
    if (m.nx >= 2) return x < 0 ? x + m.nx : (x >= m.nx ? x - m.nx : x);
    return 0;
  };
  auto yrow = [&](int t) {
    int y = jt0 - 2 + t;
    if (m.yper()) y = y < m.j0 ? y + m.ny : (y >= m.jn ? y - m.ny : y);
    return y;
  };
  auto yowned = [&](int f) { return f >= m.ylo() && f < m.jn; };
  auto zowned = [&](int f) { return f >= m.zlo() && f < m.kn; };
  // Loads keep raw field values and derived ones are formed where they are
  // used, so that a prefetched load is not waited for when it is issued.
  auto pres = [&](F rho, F q) { return adi ? gm1 * q : q * q * rho; };
  auto loadz = [&](int k, Zv<F> &z) {
    const unsigned o = m.o32(i, j, k);
    const int ip = i + 1 == m.nx ? 0 : i + 1;
    z.rho = s.rho[o];
    z.q = adi ? s.e[o] : s.cs[o];
    z.pot = s.pot[o];
    z.vz = s.vz[o];
    z.vx = s.vx[o];
    z.vxp = sph ? s.vx[o - (unsigned)i + (unsigned)ip] : F(0);
  };
  // v'_z on face p between planes below(p) (zb) and p (z0); v^n if not owned.
  // iz receives 1 / ((rho + rho_below) h_z) for the viscous term.
  auto vz1 = [&](int p, const Zv<F> &zb, const Zv<F> &z0, F &iz) {
    iz = F(0);
    if (!zowned(p)) return z0.vz;
    const double ihzd = sph ? m.g.inv_dzmed(p) * g_iymed : m.g.inv_dzmed(p);
    iz = (F)ihzd / (z0.rho + zb.rho);
    F gradP = F(2) * (pres(z0.rho, z0.q) - pres(zb.rho, zb.q)) * iz;
    F gradPhi = (F)((z0.pot - zb.pot) * ihzd);
    F src = F(0);
    if constexpr (sizeof(F) == 4) {
      if (sph) {
        // an FP32 v_x is a deviation d from the ring's background: with W the
        // mean background of the two rings, vt^2 = W^2 + (2 W + d) d, and the
        // W^2 part, which the potential and pressure gradients nearly cancel,
        // is formed with the potential gradient in FP64 and rounded once
        const F W = (F)(0.5 * (m.bg(BG_VT, jg, p) + m.bg(BG_VT, jg, m.kbelow(p))));
        const F d = F(0.25) * ((z0.vx + z0.vxp) + (zb.vx + zb.vxp));
        const F base = (F)(m.bg(BG_CZ, jg, p) - (z0.pot - zb.pot) * ihzd);
        src = (F(2) * W + d) * d * (F)m.g.cotz(p) * (F)g_iymed + base;
      } else {
        src = -gradPhi;
      }
      return z0.vz - dt * gradP + dt * src;
    } else {
      if (sph) { // inertial azimuthal velocity v_x + R Omega of the two rings
        const F o0 = (F)(g_ymed * m.g.sinz(p)) * om, o1 = (F)(g_ymed * m.g.sinz(m.kbelow(p))) * om;
        F vt = F(0.25) * ((z0.vx + o0) + (z0.vxp + o0) + (zb.vx + o1) + (zb.vxp + o1));
        src = vt * vt * (F)m.g.cotz(p) * (F)g_iymed;
      }
      return z0.vz - dt * (gradP + gradPhi) + dt * src;
    }
  };
  const bool per = m.zper();
  auto pl = [&](int p) { return per ? m.k0 + (p - m.k0 + 2 * m.nz) % m.nz : p; };

  // The halo zone this thread stages, if any (fixed over the march):
  // role 1, Y halo rows 0, 1, h+2, h+3 over the tile's columns (with v_y and,
  // in spherical geometry, the summed v_theta); role 2, X halo slots 0, 1,
  // w+2, w+3 of the tile rows; role 3, v_x on the X face after the last
  // column, in the Y halo rows.
  int role = 0, ht = 0, hsl = 0;
  if (tid < 256) {
    const int q = tid >> 6;
    ht = q < 2 ? q : h + q;
    hsl = c + 2;
    role = c < w ? 1 : 0;
  } else if (tid < 256 + 4 * TY) {
    const int q = tid - 256, rr = q >> 2, a = q & 3;
    ht = rr + 2;
    hsl = a < 2 ? a : w + a;
    role = rr < h ? 2 : 0;
  } else if (tid < 256 + 4 * TY + 4) {
    const int q = tid - 256 - 4 * TY;
    ht = q < 2 ? q : h + q;
    hsl = w + 2;
    role = 3;
  }
  const unsigned hbase = role ? m.o32(xcol(hsl), yrow(ht), 0) : 0u;
  const bool hvy = role == 1 && ht != 0, hvt = role == 1 && sph;
  // what staging takes from memory besides the window: own v_y and the halo
  struct Halo {
    F vy, hr, hq, hx, hy, ht0, ht1;
    double hp;
  };
  auto load_halo = [&](int kk, Halo &n) {
    if (act) n.vy = s.vy[m.o32(i, j, kk)];
    if (role) {
      const unsigned o = hbase + (unsigned)kk * plane;
      n.hx = s.vx[o];
      if (role != 3) {
        n.hr = s.rho[o];
        n.hq = adi ? s.e[o] : s.cs[o];
        n.hp = s.pot[o];
      }
      if (hvy) n.hy = s.vy[o];
      if (hvt) {
        const int kp = m.kabove(kk);
        n.ht0 = s.vz[o];
        n.ht1 = s.vz[o + (unsigned)(kp - kk) * plane];
      }
    }
  };
  // S: stage plane kk into buffers sb (and rb for the density); interior from
  // the window record z (vt = summed v_theta of the zone), halo from hv
  auto stage = [&](int kk, int sb, int rb, const Zv<F> &z, F vt, const Halo &hv) {
    F(*R)[SX] = L.R[rb];
    if (c == 0 && r < h) L.DX[sb][r] = m.g.inv_dxlen((size_t)kk * m.nyg + jt0 + r);
    if (act) {
      R[r + 2][c + 2] = z.rho;
      L.P[sb][r + 2][c + 2] = pres(z.rho, z.q);
      L.Ph[sb][r + 2][c + 2] = z.pot;
      L.VX[sb][r + 2][c + 2] = z.vx;
      if (sph) L.VT[sb][r + 2][c] = vt;
      L.VY[sb][r + 2][c] = hv.vy;
    }
    if (role) {
      L.VX[sb][ht][hsl] = hv.hx;
      if (role != 3) {
        R[ht][hsl] = hv.hr;
        L.P[sb][ht][hsl] = pres(hv.hr, hv.hq);
        L.Ph[sb][ht][hsl] = hv.hp;
      }
      if (hvy) L.VY[sb][ht][hsl - 2] = hv.hy;
      if (hvt) L.VT[sb][ht][hsl - 2] = hv.ht0 + hv.ht1;
    }
  };
  // F: 7a on the X and Y faces of plane kk (staged in sb, rb) into face buffer sb
  auto faces = [&](int kk, int sb, int rb) {
    F(*R)[SX] = L.R[rb];
    auto xface = [&](int rr, int sl, double idXd) {
      const int t = rr + 2;
      const F inv = (F)idXd / (R[t][sl] + R[t][sl - 1]);
      const F gradP = F(2) * (L.P[sb][t][sl] - L.P[sb][t][sl - 1]) * inv;
      const F gradPhi = (F)((L.Ph[sb][t][sl] - L.Ph[sb][t][sl - 1]) * idXd);
      L.AX[sb][rr][sl] = L.VX[sb][t][sl] - dt * (gradP + gradPhi);
      if constexpr (KI) L.IX[sb][rr][sl] = inv;
    };
    auto yface = [&](int t, int cc) {
      const int f = yrow(t), sl = cc + 2;
      if (!yowned(f)) {
        L.AY[sb][t][cc] = L.VY[sb][t][cc];
        if constexpr (KI) L.IY[sb][t][cc] = F(0);
        return;
      }
      const double ihd = m.g.inv_hy(f);
      const F inv = (F)ihd / (R[t][sl] + R[t - 1][sl]);
      const F gradP = F(2) * (L.P[sb][t][sl] - L.P[sb][t - 1][sl]) * inv;
      const F gradPhi = (F)((L.Ph[sb][t][sl] - L.Ph[sb][t - 1][sl]) * ihd);
      F src = F(0);
      if constexpr (sizeof(F) == 4) {
        // an FP32 v_x is a deviation d from the ring's background: with W the
        // mean background of the two rings, v^2 = W^2 + (2 W + d) d; the W^2
        // part, which gravity cancels to order h^2 in a disk, is formed with
        // the potential gradient in FP64 and rounded once
        if (cyl || sph) {
          const int ya = yrow(t - 1);
          const F W = (F)(0.5 * (m.bg(BG_VT, f, kk) + m.bg(BG_VT, ya, kk)));
          const F d = F(0.25) * ((L.VX[sb][t][sl] + L.VX[sb][t][sl + 1]) + (L.VX[sb][t - 1][sl] + L.VX[sb][t - 1][sl + 1]));
          src = (F(2) * W + d) * d;
          if (sph) {
            const F wv = F(0.25) * (L.VT[sb][t][cc] + L.VT[sb][t - 1][cc]);
            src += wv * wv;
          }
          src = src * (F)m.g.inv_ymin(f) +
                (F)(m.bg(BG_CY, f, kk) - (L.Ph[sb][t][sl] - L.Ph[sb][t - 1][sl]) * ihd);
        } else {
          src = -gradPhi;
        }
        L.AY[sb][t][cc] = L.VY[sb][t][cc] - dt * gradP + dt * src;
      } else {
        if (cyl || sph) {
          const int ya = yrow(t - 1);
          const F ot = (F)(sph ? m.g.ymed(f) * m.g.sinz(kk) : m.g.ymed(f)) * om;
          const F oa = (F)(sph ? m.g.ymed(ya) * m.g.sinz(kk) : m.g.ymed(ya)) * om;
          const F vt0 = (L.VX[sb][t][sl] + ot) + (L.VX[sb][t][sl + 1] + ot);
          const F vt1 = (L.VX[sb][t - 1][sl] + oa) + (L.VX[sb][t - 1][sl + 1] + oa);
          const F v = F(0.25) * (vt0 + vt1);
          src = v * v;
          if (sph) {
            const F wv = F(0.25) * (L.VT[sb][t][cc] + L.VT[sb][t - 1][cc]);
            src += wv * wv;
          }
          src *= (F)m.g.inv_ymin(f);
        }
        L.AY[sb][t][cc] = L.VY[sb][t][cc] - dt * (gradP + gradPhi) + dt * src;
      }
      if constexpr (KI) L.IY[sb][t][cc] = inv;
    };
    if (act) {
      xface(r, c + 2, m.g.inv_dxlen((size_t)kk * m.nyg + jt0 + r));
      yface(r + 2, c);
    }
    // the halo faces: the last three waves take the extra Y-face rows and
    // wave 4 the extra X faces, since waves 0-3 stage the Y-halo rows (the
    // barrier waits for the most loaded wave)
    if (r >= TY - 3) {
      const int e = r - (TY - 3), t = e == 0 ? 1 : h + 1 + e;
      if (c < w) yface(t, c);
    } else if (r == 4 && c < 3 * TY) {
      const int rr = c / 3, a = c % 3, sl = a == 0 ? 1 : w + 1 + a;
      if (rr < h) xface(rr, sl, L.DX[sb][rr]);
    }
  };
  // Z: 7b and 7c for the zones of plane kk (faces in sb, density in rb); zd
  // gives the Z part: bz1/bz2 (v'' of faces kk and above(kk)), qz and dvz
  struct ZPart {
    F bz1, bz2, qz, dvz;
  };
  auto zones = [&](int kk, int sb, int rb, const ZPart &zp, F e_old) {
    F(*R)[SX] = L.R[rb];
    const int t = r + 2, sl = c + 2;
    const unsigned o = m.o32(i, j, kk);
    // X: faces sl-1 .. sl+2, zones sl-1 .. sl+1
    const F a0 = L.AX[sb][r][sl - 1], a1 = L.AX[sb][r][sl], a2 = L.AX[sb][r][sl + 1], a3 = L.AX[sb][r][sl + 2];
    const F r1 = R[t][sl - 1], r2 = R[t][sl], r3 = R[t][sl + 1];
    const F dvx = a2 - a1;
    const F qx = qvisc(c2, r2, dvx), qxm = qvisc(c2, r1, a1 - a0), qxp = qvisc(c2, r3, a3 - a2);
    const double idX = m.g.inv_dxlen((size_t)kk * m.nyg + j);
    // the reciprocals of the two X faces, as the faces' pass forms them
    const F ix1 = KI ? L.IX[sb][r][sl] : (F)idX / (r2 + r1);
    const F ix2 = KI ? L.IX[sb][r][sl + 1] : (F)idX / (r3 + r2);
    const F bx1 = a1 - dt * F(2) * (qx - qxm) * ix1;
    const F bx2 = a2 - dt * F(2) * (qxp - qx) * ix2;
    vx2[o] = bx1;
    F heat = qx * dvx * (F)idX;
    const double syk = m.g.syk(kk);
    F flux = (F)(g_sxj * m.g.sxk(kk)) * (bx2 - bx1);
    // Y: faces t-1 .. t+2, zones t-1 .. t+1
    const F b0 = L.AY[sb][t - 1][c], b1 = L.AY[sb][t][c], b2 = L.AY[sb][t + 1][c], b3 = L.AY[sb][t + 2][c];
    const F s1 = R[t - 1][sl], s3 = R[t + 1][sl];
    const F dvy = b2 - b1;
    const F qy = qvisc(c2, r2, dvy);
    F by1 = b1, by2 = b2;
    if (yowned(j)) {
      const F iy = KI ? L.IY[sb][t][c] : (F)m.g.inv_hy(j) / (r2 + s1);
      by1 = b1 - dt * F(2) * (qy - qvisc(c2, s1, b1 - b0)) * iy;
    }
    const int ju = yrow(t + 1);
    if (yowned(ju)) {
      const F iy = KI ? L.IY[sb][t + 1][c] : (F)m.g.inv_hy(ju) / (s3 + r2);
      by2 = b2 - dt * F(2) * (qvisc(c2, s3, b3 - b2) - qy) * iy;
    }
    vy2[o] = by1;
    heat += qy * dvy * (F)g_invLy;
    flux += (F)(g_syj1 * syk) * by2 - (F)(g_syj * syk) * by1;
    vz2[o] = zp.bz1;
    const F iLz = sph ? (F)(m.g.inv_dz(kk) * g_iymed) : (F)m.g.inv_dz(kk);
    heat += zp.qz * zp.dvz * iLz;
    flux += (F)(g_szj * m.g.szk(kk + 1)) * zp.bz2 - (F)(g_szj * m.g.szk(kk)) * zp.bz1;
    if (adi) {
      const F e1 = e_old - dt * heat;
      const F a = F(0.5) * dt * gm1 * ((F)(g_invVj / syk) * flux);
      e2[o] = e1 * (F(1) - a) / (F(1) + a);
    }
  };

  // ---- 3D march over the workgroup's active planes k0 .. kn-1
  // Z window of the thread's column at the top of interval kk:
  //   Z1, Z2 = records of planes kk+1, kk+2; vzk = v_z of plane kk;
  //   A[0..2] = v'_z of faces kk .. kk+2, IZ likewise; Q[0..2] = q_z of
  //   zones kk-1 .. kk+1
  Zv<F> Z1{}, Z2{}, Zn{};
  F vzk = F(0), A[3] = {}, IZ[3] = {}, Q[3] = {}, e_cur = F(0);
  Halo hv{}, hn{};
  if (act) {
    Zv<F> a, b, z0;
    F Am1, IZm1, A0, IZ0, A1, IZ1, A2, IZ2;
    loadz(pl(k0 - 2), a);
    loadz(pl(k0 - 1), b);
    loadz(k0, z0);
    loadz(pl(k0 + 1), Z1);
    loadz(pl(k0 + 2), Z2);
    Am1 = vz1(pl(k0 - 1), a, b, IZm1);
    A0 = vz1(k0, b, z0, IZ0);
    A1 = vz1(pl(k0 + 1), z0, Z1, IZ1);
    A2 = vz1(pl(k0 + 2), Z1, Z2, IZ2);
    (void)IZm1;
    A[0] = A0;
    A[1] = A1;
    A[2] = A2;
    IZ[0] = IZ0;
    IZ[1] = IZ1;
    IZ[2] = IZ2;
    Q[0] = qvisc(c2, b.rho, A0 - Am1);
    Q[1] = qvisc(c2, z0.rho, A1 - A0);
    Q[2] = qvisc(c2, Z1.rho, A2 - A1);
    vzk = z0.vz;
    e_cur = z0.q;
    // prologue: S(k0), then F(k0) with S(k0+1)
    load_halo(k0, hv);
    stage(k0, 0, 0, z0, z0.vz + Z1.vz, hv);
  } else {
    load_halo(k0, hv);
    stage(k0, 0, 0, Zv<F>{}, F(0), hv);
  }
  __syncthreads();
  faces(k0, 0, 0);
  load_halo(pl(k0 + 1), hv);
  stage(k0 + 1, 1, 1, Z1, Z1.vz + Z2.vz, hv);
  // prefetch for interval k0: record of plane k0+3, halo of plane k0+2
  if (act) loadz(pl(k0 + 3), Zn);
  if (k0 + 2 < kn) load_halo(k0 + 2, hn);
  __syncthreads();

  int sb = 0, rb = 0; // buffers of plane kk
#pragma unroll 1
  for (int kk = k0; kk < kn; kk++) {
    const int sb1 = sb ^ 1, rb1 = rb == 2 ? 0 : rb + 1, rb2 = rb1 == 2 ? 0 : rb1 + 1;
    // Z(kk)
    if (act) {
      ZPart zp;
      const int ka = pl(kk + 1);
      zp.bz1 = zowned(kk) ? A[0] - dt * F(2) * (Q[1] - Q[0]) * IZ[0] : vzk;
      zp.bz2 = zowned(ka) ? A[1] - dt * F(2) * (Q[2] - Q[1]) * IZ[1] : Z1.vz;
      zp.qz = Q[1];
      zp.dvz = A[1] - A[0];
      zones(kk, sb, rb, zp, e_cur);
    }
    // F(kk+1), S(kk+2)
    if (kk + 1 < kn) faces(kk + 1, sb1, rb1);
    if (kk + 2 < kn) stage(kk + 2, sb, rb2, Z2, Z2.vz + Zn.vz, hn);
    // advance the window and prefetch for interval kk+1
    if (kk + 1 < kn) {
      if (act) {
        F A3, IZ3;
        A3 = vz1(pl(kk + 3), Z2, Zn, IZ3);
        const F Q3 = qvisc(c2, Z2.rho, A3 - A[2]);
        vzk = Z1.vz;
        e_cur = Z1.q;
        Z1 = Z2;
        Z2.rho = vmove(Zn.rho);
        Z2.q = vmove(Zn.q);
        Z2.pot = vmove(Zn.pot);
        Z2.vz = vmove(Zn.vz);
        Z2.vx = vmove(Zn.vx);
        Z2.vxp = sph ? vmove(Zn.vxp) : F(0);
        A[0] = A[1];
        A[1] = A[2];
        A[2] = A3;
        IZ[0] = IZ[1];
        IZ[1] = IZ[2];
        IZ[2] = IZ3;
        Q[0] = Q[1];
        Q[1] = Q[2];
        Q[2] = Q3;
        // unconditional (plane kk+4 <= kn+2 is at worst a ghost plane), so
        // that the load writes the window register itself
        loadz(pl(kk + 4), Zn);
      }
      if (kk + 3 < kn) load_halo(kk + 3, hn);
    }
    __syncthreads();
    sb = sb1;
    rb = rb1;
  }
  if (!ghosts) return;
  // the ghost rows next to the tile's, a row of its columns per wave
  const GhostRows G_(m, ty == 0, ty == nby - 1, k0, kn);
  for (int t = r; t < G_.rows(jt0, h); t += TY) {
    int jg_, kg_;
    G_.row(t, jt0, h, jg_, kg_);
    if (c < w) carry_ghost<F, true, ADI>(s, m.o32(i, jg_, kg_), vx2, vy2, vz2, e2);
  }
}
template <typename F, int GEO, bool ADI>
__global__ __launch_bounds__((src_threads<F, GEO, ADI>()), (src_waves<F, GEO, ADI>())) void k_source(
    Mesh m, StateT<F> s, DevWords dw, F *__restrict__ vx2, F *__restrict__ vy2, F *__restrict__ vz2,
    F *__restrict__ e2, int nbx, int nby, int zlen, int ghosts) {
  source_body<F, GEO, ADI>(m, s, dw, vx2, vy2, vz2, e2, nbx, nby, zlen, ghosts, blockIdx.x, gridDim.x);
}

// The ghost rows alone, one block per row.
template <typename F, bool ADI>
__global__ __launch_bounds__(256) void k_source_ghosts(Mesh m, StateT<F> s, F *__restrict__ vx2, F *__restrict__ vy2,
                                                       F *__restrict__ vz2, F *__restrict__ e2) {
  const GhostRows G(m, true, true, m.k0, m.kn);
  int j, k;
  G.row((int)blockIdx.x, m.j0, m.ny, j, k);
  for (int i = threadIdx.x; i < m.nx; i += blockDim.x) carry_ghost<F, true, ADI>(s, m.o32(i, j, k), vx2, vy2, vz2, e2);
}

// tile rows of the source step's launch on a 3D mesh
template <typename F>
int src_rows(const Mesh &m) {
  const bool tall = m.geo != FARGO_SPHERICAL && m.eos != FARGO_ADIABATIC;
  return tall ? tile_rows<F, FARGO_CARTESIAN, false>() : tile_rows<F, FARGO_SPHERICAL, true>();
}

// ------------------------------------------------------------------------
// 2D meshes.  A wave walks a chunk of rows outwards over 64 columns, one per
// lane: neighbours along X come by DPP lane moves, the row below and the faces
// and terms that the next rows need stay in registers, and each face is formed
// once.  Two lanes below and one above (two with an energy, which takes the
// upper X face's final velocity) are halo.  Nothing goes through LDS and no wave
// waits for another; the loads of four rows are in flight.  Bound by memory on
// large meshes: 3072 x 1024 zones in FP64 47 + 8 (LDS tiles of 64 x 8 zones and a
// launch for the ghost rows) to 34.7 us, 5.1 TB/s of its 7 words a zone; the
// batch of 256 disks in FP32 770 + 9 to 534 us (4.2 TB/s), of 48 in FP64 239 + 7
// to 186; 633 x 211 zones 7.2 to 6.5, 384 x 128 6.1 to 5.5.
// ------------------------------------------------------------------------
template <typename F>
struct Source2 {
  Mesh m;
  StateT<F> s;
  DtIn in;
  DevWords dw;
  F *vx2, *vy2, *e2;
  int nseg, chunk, nchunk; // segments of a row, rows of a chunk, chunks
};
template <bool ADI>
constexpr int src2_cols() { return WAVE - (ADI ? 4 : 3); }
// The most rows of a chunk (which reads three or four beside its own), of one
// mesh and of the meshes of a batch.  One mesh: 32 rows, or as many chunks as
// make whole rounds of one wave per SIMD (3072 x 1024: 34.7 us; at most 16 rows
// 38; as many chunks as waves fit 38); 633 x 211: 6.5 us (twice the waves 7.0).
// A batch of 256 disks in FP32, which fills the chip at any length: 534 us at 16
// rows, 559 at 24, 573 at 32, 537 at 8.
constexpr int SRC2_ROWS = 32, SRC2_MANY = 16;
constexpr long SRC2_WAVES = 4L * CHIP_CUS;

template <typename F, bool CYL, bool ADI>
__device__ __forceinline__ void source2_body(const Source2<F> &A, unsigned bid_, unsigned nbk_) {
// Contraction is off: the rows of a turn of the march are compiled apart, and
// the same rounding in all keeps the result independent of the chunk length.
#pragma clang fp contract(off)
  const Mesh &m = A.m;
  const int lane = threadIdx.x & (WAVE - 1);
  // wave-uniform, so that the rows' constants come through scalar loads
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
  const int gw = (int)xcd_remap(bid_, nbk_) * (int)(blockDim.x / WAVE) + wave;
  const int seg = gw % A.nseg, ch = gw / A.nseg;
  const int a0 = m.j0 + ch * A.chunk, a1 = min(a0 + A.chunk, m.jn), n = m.nx;
  const int z = seg * src2_cols<ADI>() + lane - 2;
  const int i = n > 1 ? (z < 0 ? z + n : (z >= n ? z % n : z)) : 0;
  const bool useful = lane >= 2 && lane < 2 + src2_cols<ADI>() && z < n;
  // rows a0 - 2 .. last are read; past the last the read is of the last again
  const int last = ADI ? a1 + 1 : a1;
  auto yrow = [&](int t) {
    int y = min(t, last);
    if (m.yper()) y = y < m.j0 ? y + m.ny : (y >= m.jn ? y - m.ny : y);
    return y;
  };
  struct Row {
    F rho, q, vx, vy;
    double pot;
  };
  auto ld = [&](int t, Row &w) {
    const unsigned c = m.o32(i, yrow(t), 0);
    w.rho = A.s.rho[c];
    w.q = ADI ? A.s.e[c] : A.s.cs[c];
    w.pot = A.s.pot[c];
    w.vx = A.s.vx[c];
    w.vy = A.s.vy[c];
  };
  Row W[4];
  const bool live = ch < A.nchunk;
  if (live) {
#pragma unroll
    for (int q = 0; q < 4; q++) ld(a0 - 2 + q, W[q]);
  }
  // dt: the device word, or, on meshes of few rings, formed here from the
  // time-step pass's slots by the first wave of every workgroup, which saves a
  // launch of one workgroup (DT_SLOTS); the first workgroup leaves it in the
  // word for the kernels that follow
  __shared__ double dt_sh;
  F dt;
  if (A.in.nslot > 0) {
    if (wave == 0) {
      const DtSlots sl = dt_slots(m, A.in);
      // all slots read at once, the last one again past the end: a loop waits
      // for memory up to four times (2 us)
      constexpr int P = DT_SLOTS / WAVE;
      double rr[P], ss[P], rmax = 0.0, smax = 0.0;
#pragma unroll
      for (int q = 0; q < P; q++) {
        const int x = min(lane + q * WAVE, sl.nslot - 1);
        rr[q] = sl.rate[x];
        ss[q] = sl.shear[x];
      }
#pragma unroll
      for (int q = 0; q < P; q++) {
        rmax = rr[q] > rmax ? rr[q] : rmax;
        smax = ss[q] > smax ? ss[q] : smax;
      }
      rmax = lane63(wave_reduce_dpp(rmax, Max(), 0.0));
      smax = lane63(wave_reduce_dpp(smax, Max(), 0.0));
      bool bad;
      const double d = dt_of_extremes(sl, rmax, smax, &bad);
      if (lane == 0) {
        dt_sh = d;
        if (bid_ == 0) {
          if (bad) atomicOr(A.dw.err, 2);
          *A.dw.dt = d;
        }
      }
    }
    __syncthreads();
    dt = (F)dt_sh;
  } else {
    dt = (F)*A.dw.dt;
  }
  if (!live) return;
  const F c2 = (F)(m.cvnr * m.cvnr), om = (F)m.omega, gm1 = (F)(m.gamma - 1.0), dt2 = dt * F(2);
  const double syk = m.g.syk(0), sxk = m.g.sxk(0);
  auto yowned = [&](int f) { return f >= m.ylo() && f < m.jn; };
  auto pres = [&](F rho, F q) { return ADI ? gm1 * q : q * q * rho; };
  // a row's constants, read a row ahead
  struct Geo {
    double ihd, idX, ymed, iymin, vb, cb;
  };
  auto geo = [&](int t) {
    const int y = yrow(t);
    Geo g{};
    g.ihd = m.g.inv_hy(y);
    g.idX = m.g.inv_dxlen((size_t)y);
    if (CYL) {
      g.iymin = m.g.inv_ymin(y);
      if (sizeof(F) == 8) {
        g.ymed = m.g.ymed(y);
      } else {
        g.vb = m.bg(BG_VT, y, 0);
        g.cb = m.bg(BG_CY, y, 0);
      }
    }
    return g;
  };
  // v_x of the zone's two X faces, summed, with the frame velocity in FP64
  auto vsum = [&](F vx, const Geo &g) {
    const F vxn = from_next_lane(vx);
    if constexpr (CYL && sizeof(F) == 8) {
      const F o = (F)g.ymed * om;
      return (vx + o) + (vxn + o);
    } else {
      return vx + vxn;
    }
  };
  Geo gn = geo(a0 - 1);
  const Geo g0 = geo(a0 - 2);
  // of the row below: density, pressure, potential, summed v_x, mean background,
  // storage row
  F rho_s = W[0].rho, p_s = pres(W[0].rho, W[0].q), vt_s = vsum(W[0].vx, g0);
  double pot_s = W[0].pot, vb_s = g0.vb;
  int y_s = yrow(a0 - 2);
  // v'_y of its lower face, 1 / ((rho + rho below) h) there; q_y of the zone below it
  F b_s = F(0), iy_s = F(0), q_s = F(0);
  // ADI, [0] of the row below, [1] of the row two below: what X adds to heating
  // and divergence, the energy; of the row two below: v''_y of its lower face,
  // q_y and the velocity step of it
  F hx[2] = {}, fx[2] = {}, eo[2] = {}, by_s = F(0), dv_s = F(0);
  auto row = [&](int t, Row &w) {
    const int y = yrow(t);
    const F rho = w.rho, q = w.q, vx = w.vx, vy = w.vy;
    const double pot = w.pot;
    ld(t + 4, w);
    const Geo g = gn;
    gn = geo(t + 1);
    const F p = pres(rho, q), vt = vsum(vx, g);
    // Y: v' of the row's lower face, then 7b on the face below
    const double ihd = g.ihd;
    const F iy = (F)ihd / (rho + rho_s);
    const F gradP = F(2) * (p - p_s) * iy;
    F b;
    if constexpr (CYL && sizeof(F) == 4) {
      // an FP32 v_x is a deviation d from the ring's background: with W the
      // mean background of the two rings, v^2 = W^2 + (2 W + d) d; the W^2
      // part, which gravity cancels to order h^2 in a disk, is formed with
      // the potential gradient in FP64 and rounded once
      const F Wb = (F)(0.5 * (g.vb + vb_s)), d = F(0.25) * (vt + vt_s);
      const F src = (F(2) * Wb + d) * d * (F)g.iymin + (F)(g.cb - (pot - pot_s) * ihd);
      b = vy - dt * gradP + dt * src;
    } else {
      F acc = gradP + (F)((pot - pot_s) * ihd);
      if constexpr (CYL) {
        const F v = F(0.25) * (vt + vt_s);
        acc = acc - v * v * (F)g.iymin;
      }
      b = vy - dt * acc;
    }
    if (!yowned(y)) b = vy;
    const F dv = b - b_s, qy = qvisc(c2, rho_s, dv);
    F by = b_s;
    if (yowned(y_s)) by = b_s - dt2 * (qy - q_s) * iy_s;
    if (t > a0 && t <= a1 && useful) A.vy2[m.o32(i, t - 1, 0)] = by;
    // X: faces and zones of the row
    F heat = F(0), flux = F(0);
    if (t >= a0 && t < a1) {
      const double idX = g.idX;
      const F ix = (F)idX / (rho + from_prev_lane(rho));
      const F gp = F(2) * (p - from_prev_lane(p)) * ix;
      const F a = vx - dt * (gp + (F)((pot - from_prev_lane(pot)) * idX));
      const F dvx = from_next_lane(a) - a, qx = qvisc(c2, rho, dvx);
      const F bx = a - dt2 * (qx - from_prev_lane(qx)) * ix;
      if (useful) A.vx2[m.o32(i, t, 0)] = bx;
      if constexpr (ADI) {
        heat = qx * dvx * (F)idX;
        flux = (F)(m.g.sxj(y) * sxk) * (from_next_lane(bx) - bx);
      }
    }
    if constexpr (ADI) {
      // 7c of the row two below: [1] its X part, by_s and by its Y faces
      if (t >= a0 + 2) {
        const int j = t - 2;
        const F ht = hx[1] + q_s * dv_s * (F)m.g.inv_Ly(j);
        const F fl = fx[1] + ((F)(m.g.syj(j + 1) * syk) * by - (F)(m.g.syj(j) * syk) * by_s);
        const F e1 = eo[1] - dt * ht;
        const F al = F(0.5) * dt * gm1 * ((F)(m.g.invVj(j) / syk) * fl);
        if (useful) A.e2[m.o32(i, j, 0)] = e1 * (F(1) - al) / (F(1) + al);
      }
      hx[1] = hx[0];
      fx[1] = fx[0];
      eo[1] = eo[0];
      hx[0] = heat;
      fx[0] = flux;
      eo[0] = q;
      by_s = by;
      dv_s = dv;
    }
    rho_s = rho;
    p_s = p;
    vt_s = vt;
    pot_s = pot;
    y_s = y;
    vb_s = g.vb;
    b_s = b;
    iy_s = iy;
    q_s = qy;
  };
  ld(a0 + 2, W[0]);
#pragma unroll 1
  for (int t = a0 - 1; t <= last; t++) {
    row(t, W[1]);
    if (++t > last) break;
    row(t, W[2]);
    if (++t > last) break;
    row(t, W[3]);
    if (++t > last) break;
    row(t, W[0]);
  }
  // the ghost rows that keep v^n and e, all read before the first is written
  // (waves of their own for them, last in the launch, took 8 us longer on 3072 x
  // 1024 zones)
  auto carry = [&](int j0) {
    F v[NGH][3];
#pragma unroll
    for (int g = 0; g < NGH; g++) {
      const unsigned c = m.o32(i, j0 + g, 0);
      v[g][0] = A.s.vx[c];
      v[g][1] = A.s.vy[c];
      v[g][2] = ADI ? A.s.e[c] : F(0);
    }
    if (!useful) return;
#pragma unroll
    for (int g = 0; g < NGH; g++) {
      const unsigned c = m.o32(i, j0 + g, 0);
      A.vx2[c] = v[g][0];
      A.vy2[c] = v[g][1];
      if (ADI) A.e2[c] = v[g][2];
    }
  };
  if (ch == 0 && ghost_rows(m, 0)) carry(0);
  if (ch == A.nchunk - 1 && ghost_rows(m, 1)) carry(m.jn);
}
template <typename F, bool CYL, bool ADI>
__global__ __launch_bounds__(256) void k_source2(Source2<F> A) {
  source2_body<F, CYL, ADI>(A, blockIdx.x, gridDim.x);
}

// multi-mesh form (ManyGrid)
template <typename F>
struct Source2Args {
  Source2<F> A;
  unsigned nb, pad_;
};
template <typename F, bool CYL, bool ADI>
__global__ __launch_bounds__(256) void k_source2_many(const void *args, const uint2 *tab) {
  const uint2 t = many_block(tab);
  if (t.x == MANY_NONE) return;
  const Source2Args<F> a = many_args<Source2Args<F>>(args, t.x);
  source2_body<F, CYL, ADI>(a.A, t.y, a.nb);
}

inline int src2_segs(const Mesh &m) {
  const int u = m.eos == FARGO_ADIABATIC ? src2_cols<true>() : src2_cols<false>();
  return (m.nx + u - 1) / u;
}
// the step over 2D mesh m with chunks of at most `rows` rows, more to share out
// over `slots` waves (0: as they are), and its blocks
template <typename F>
Source2<F> source2_of(const Mesh &m, const StateT<F> &s, const DtIn &in, const DevWords &w, F *vx2, F *vy2, F *e2,
                      long slots, int rows, unsigned &nb) {
  Source2<F> A{m, s, in, w, vx2, vy2, e2, src2_segs(m), 0, 0};
  const int nch = slots ? fill_chunks(m.ny, rows, 1, A.nseg, slots, 4) : (m.ny + rows - 1) / rows;
  A.chunk = (m.ny + nch - 1) / nch;
  A.nchunk = (m.ny + A.chunk - 1) / A.chunk;
  nb = (unsigned)(((long)A.nseg * A.nchunk + 3) / 4);
  return A;
}

// go(cylindrical, adiabatic) with the compile-time constants of 2D mesh m
template <class GO>
void source2_form(const Mesh &m, const GO &go) {
  const bool cyl = m.geo == FARGO_CYLINDRICAL;
  if (m.eos == FARGO_ADIABATIC) {
    if (cyl) go(std::true_type{}, std::true_type{});
    else go(std::false_type{}, std::true_type{});
  } else {
    if (cyl) go(std::true_type{}, std::false_type{});
    else go(std::false_type{}, std::false_type{});
  }
}
} // namespace

template <typename F>
void launch_source(Launch &L, const Mesh &m, const StateT<F> &s, const DtIn &in, const DevWords &w, F *vx2, F *vy2,
                   F *vz2, F *e2) {
  prof_begin(L, K_SRC);
  const int nbx = (m.nx + TX - 1) / TX, nby = (m.ny + src_rows<F>(m) - 1) / src_rows<F>(m);
  auto go2 = [&](auto cyl, auto adi) {
    unsigned nb;
    const Source2<F> A = source2_of(m, s, in, w, vx2, vy2, e2, SRC2_WAVES, SRC2_ROWS, nb);
    k_source2<F, decltype(cyl)::value, decltype(adi)::value><<<nb, 256, 0, L.s>>>(A);
  };
  auto go = [&](auto geo, auto adi) {
    constexpr bool ADI = decltype(adi)::value;
    constexpr int GEO = decltype(geo)::value;
    const int ng = GhostRows(m, true, true, m.k0, m.kn).rows(m.j0, m.ny);
    // the march in chunks of planes where the tiles alone leave compute units
    // idle, or a last round of workgroups nearly empty (a chunk reads five
    // planes beside its own).  Box of 160 x 144 x 120 zones, 36 tiles: 311
    // to 64 us; 501 x 167 x 43 FP32 spherical, 168 tiles on 512 slots: 147
    // to 67 us; 1536 x 512 x 128, 1032 tiles on 256 slots: 2.52 to 2.42 ms;
    // 2048 x 768 x 96, 1536 tiles: unchanged.
    static const long slots = block_slots(k_source<F, GEO, ADI>, src_threads<F, GEO, ADI>());
    unsigned nb = (unsigned)nbx * (unsigned)nby;
    const int nzc = fill_chunks(m.nz, m.nz, 4, (long)nb, slots, 4);
    const int zlen = (m.nz + nzc - 1) / nzc;
    nb *= (unsigned)((m.nz + zlen - 1) / zlen);
    // The tiles at a side take its ghost rows along where a launch costs more
    // than the tail they add (2048 x 768 x 96, 1536 tiles: 69 us against 14 alone)
    const bool here = nb <= 2 * CHIP_CUS;
    k_source<F, GEO, ADI><<<nb, src_threads<F, GEO, ADI>(), 0, L.s>>>(m, s, w, vx2, vy2, vz2, e2, nbx, nby, zlen,
                                                                      here ? 1 : 0);
    if (!here && ng > 0) k_source_ghosts<F, ADI><<<(unsigned)ng, 256, 0, L.s>>>(m, s, vx2, vy2, vz2, e2);
  };
  auto by_eos = [&](auto geo) {
    if (m.eos == FARGO_ADIABATIC) go(geo, std::true_type{});
    else go(geo, std::false_type{});
  };
  if (!m.d3) source2_form(m, go2);
  else if (m.geo == FARGO_SPHERICAL) by_eos(std::integral_constant<int, FARGO_SPHERICAL>{});
  else if (m.geo == FARGO_CYLINDRICAL) by_eos(std::integral_constant<int, FARGO_CYLINDRICAL>{});
  else by_eos(std::integral_constant<int, FARGO_CARTESIAN>{});
  prof_end(L, K_SRC);
}

template void launch_source<double>(Launch &, const Mesh &, const StateT<double> &, const DtIn &, const DevWords &,
                                    double *, double *, double *, double *);
template void launch_source<float>(Launch &, const Mesh &, const StateT<float> &, const DtIn &, const DevWords &,
                                   float *, float *, float *, float *);

template <typename F>
size_t source_args_bytes() { return sizeof(Source2Args<F>); }

template <typename F>
int source_rows(const std::vector<Mesh> &ms) {
  return fill_chunk_length(ms, SRC2_MANY, SRC2_WAVES, 4, [](const Mesh &m) { return src2_segs(m); });
}

template <typename F>
unsigned source_args(const Mesh &m, const StateT<F> &s, const DevWords &w, F *vx2, F *vy2, F *e2, int rows, void *dst) {
  unsigned nb;
  const Source2<F> A = source2_of(m, s, DtIn{}, w, vx2, vy2, e2, 0L, rows, nb);
  *(Source2Args<F> *)dst = Source2Args<F>{A, nb, 0};
  return nb;
}

// 2D meshes of one geometry and equation of state (those of m0)
template <typename F>
void launch_source_many(Launch &L, const Mesh &m0, const ManyGrid &g) {
  prof_begin(L, K_SRC);
  source2_form(m0, [&](auto cyl, auto adi) {
    k_source2_many<F, decltype(cyl)::value, decltype(adi)::value><<<g.nblk, 256, 0, L.s>>>(g.args, g.tab);
  });
  prof_end(L, K_SRC);
}

#define FARGO_SOURCE_MANY(F)                                                                                        \
  template size_t source_args_bytes<F>();                                                                          \
  template int source_rows<F>(const std::vector<Mesh> &);                                                          \
  template unsigned source_args<F>(const Mesh &, const StateT<F> &, const DevWords &, F *, F *, F *, int, void *); \
  template void launch_source_many<F>(Launch &, const Mesh &, const ManyGrid &);
FARGO_SOURCE_MANY(double)
FARGO_SOURCE_MANY(float)
#undef FARGO_SOURCE_MANY

} // namespace fargo
