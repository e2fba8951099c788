// Box 7d: kinematic viscosity, cylindrical 2D (phi, r), App. B: the stress
// components of Eq. 73 (tau_phiphi and tau_rr at zone centres, tau_rphi on
// the zone's lower edge in both X and Y, Fig. "stress") and their divergence
// (Eq. 76).  Every component comes from the velocities after box 7b (Jacobi);
// v_phi is updated on the X faces of active zones and v_r on the owned Y
// faces, with the face density of Eq. 20; ghost zones carry v'' over.  On an
// edge, rho and nu are the means of the four zones sharing it and v_phi / r
// is the mean of v_phi / r on the two X faces it joins.  The field type F is
// double or float.
#include "fargo_internal.h"

namespace fargo {

namespace {

template <typename F>
struct Visc {
  Mesh m;
  StateT<F> s;
  const F *vx, *vy;
  const double *dt;
  F *vx3, *vy3;
  int nseg, chunk, nchunk; // segments of a row, rows of a chunk, chunks
};

// One pass.  A wave walks a chunk of rows outwards over 64 columns, one per
// lane: the rows j - 1, j and j + 1 and the components of the row below stay in
// registers, the neighbours along X come by DPP lane moves, and each component
// is formed once.  The first and last lane are halo, so a wave updates
// VISC_U = 62 columns.  Each field is read once and each result written once: 6
// words a zone, where two passes through the three components took 13 (the
// batch of 256 disks in FP32, 70.7 M zones: 1172 to 408 us, 4.2 TB/s; of 48 in
// FP64: 455 to 174 us, 3.9 TB/s; 633 x 211 zones: 9.0 to 5.7 us).
constexpr int VISC_U = WAVE - 2;
constexpr int VISC_ROWS = 32; // the most rows of a chunk (a chunk reads two beside its own)

template <typename F>
__device__ __forceinline__ void visc_body(const Visc<F> &V, unsigned bid_, unsigned nbk_) {
  const Mesh &m = V.m;
  const int lane = threadIdx.x & (WAVE - 1);
  // wave-uniform, so that the rows' constants come through scalar loads
  const int gw = (int)xcd_remap(bid_, nbk_) * (int)(blockDim.x / WAVE) +
                 __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
  const int seg = gw % V.nseg, ch = gw / V.nseg;
  if (ch >= V.nchunk) return;
  const int a0 = m.j0 + ch * V.chunk, a1 = min(a0 + V.chunk, m.jn), n = m.nx;
  const int z = seg * VISC_U + lane - 1;
  const int i = z < 0 ? z + n : (z >= n ? z % n : z);
  const bool useful = lane >= 1 && lane <= VISC_U && z < n;
  const F dt = (F)*V.dt;
  const double idphi = 1.0 / m.dx, syk = m.g.syk(0), sxk = m.g.sxk(0);
  struct Row {
    F rho, nu, vx, vy;
  };
  auto ld = [&](int j, Row &r) {
    const unsigned c = m.o32(i, j, 0);
    r.rho = V.s.rho[c];
    r.nu = V.s.nu[c];
    r.vx = V.vx[c];
    r.vy = V.vy[c];
  };
  // (Contraction is off in the components: a chunk forms its first ones before
  // the loop and the others inside it, and the same rounding in both places
  // keeps the result independent of the chunk length.)
  // tau_phiphi and tau_rr of row j from its velocities and v_r on its upper face
  auto diag = [&](int j, const Row &r, F vyn, F &tpp, F &trr) {
#pragma clang fp contract(off)
    const F dvx = from_next_lane(r.vx) - r.vx;
    const F div = (F)m.Vinv(j, 0) *
                  ((F)(m.g.sxj(j) * sxk) * dvx + ((F)(m.g.syj(j + 1) * syk) * vyn - (F)(m.g.syj(j) * syk) * r.vy));
    const F rn = r.rho * r.nu, ur = F(0.5) * (r.vy + vyn), d3 = F(2) / F(3) * div;
    tpp = -rn * (F(2) * (dvx * (F)(m.g.inv_ymed(j) * idphi) + ur * (F)m.g.inv_ymed(j)) - d3);
    trr = -rn * (F(2) * (vyn - r.vy) * (F)m.g.inv_Ly(j) - d3);
  };
  // tau_rphi on the lower edges of row j (u) above row j - 1 (d); pu and pd are
  // rho and nu of the zones before
  struct Prev {
    F rho, nu;
  };
  auto prev = [&](const Row &r) { return Prev{from_prev_lane(r.rho), from_prev_lane(r.nu)}; };
  auto edge = [&](int j, const Row &u, const Prev &pu, const Row &d, const Prev &pd) {
#pragma clang fp contract(off)
    const F rho4 = F(0.25) * (u.rho + pu.rho + d.rho + pd.rho), nu4 = F(0.25) * (u.nu + pu.nu + d.nu + pd.nu);
    F shear = (u.vx - d.vx) * (F)m.g.inv_hy(j) -
              F(0.5) * (u.vx * (F)m.g.inv_ymed(j) + d.vx * (F)m.g.inv_ymed(j - 1));
    // an FP32 v_phi is a deviation from its ring's background: the same two
    // terms of the background, formed in FP64 and rounded once
    if constexpr (sizeof(F) == 4) shear += (F)m.bg(BG_KV, j, 0);
    return -rho4 * nu4 * (shear + (u.vy - from_prev_lane(u.vy)) * (F)(m.g.inv_ymin(j) * idphi));
  };
  auto carry = [&](int j) { // a ghost row
    const unsigned c = m.o32(i, j, 0);
    const F a = V.vx[c], b = V.vy[c];
    if (useful) {
      V.vx3[c] = a;
      V.vy3[c] = b;
    }
  };
  if (ch == 0)
    for (int j = 0; j < m.j0; j++) carry(j);
  Row S, C, N, X;
  ld(a0 - 1, S);
  ld(a0, C);
  ld(a0 + 1, X);
  F tpp_s, trr_s;
  diag(a0 - 1, S, C.vy, tpp_s, trr_s);
  Prev pC = prev(C);
  F trp = edge(a0, C, pC, S, prev(S));
  F rho_s = S.rho;
#pragma unroll 1
  for (int j = a0; j < a1; j++) {
    N = X;
    if (j + 2 <= a1) ld(j + 2, X);
    F tpp, trr;
    diag(j, C, N.vy, tpp, trr);
    const Prev pN = prev(N);
    const F trp_n = edge(j + 1, N, pN, C, pC);
    const F tpp_w = from_prev_lane(tpp), trp_e = from_next_lane(trp);
    const unsigned c = m.o32(i, j, 0);
    const double a = m.g.ymin(j), b = m.g.ymin(j + 1), ir = m.g.inv_ymed(j), ia = m.g.inv_ymin(j);
    // v_phi on the X face of zone (i, j)
    const F rx = F(0.5) * (C.rho + pC.rho);
    const F divx = ((F)(b * b) * trp_n - (F)(a * a) * trp) * (F)(ir * ir * m.g.inv_Ly(j)) +
                   (tpp - tpp_w) * (F)(ir * idphi);
    const F vxn = C.vx - dt * divx / rx;
    // v_r on the Y face of zone (i, j), if the step owns it
    F vyn = C.vy;
    if (j >= m.ylo()) {
      const F ry = F(0.5) * (C.rho + rho_s);
      const F divy = ((F)m.g.ymed(j) * trr - (F)m.g.ymed(j - 1) * trr_s) * (F)(ia * m.g.inv_hy(j)) +
                     (trp_e - trp) * (F)(ia * idphi) - F(0.5) * (tpp + tpp_s) * (F)ia;
      vyn = C.vy - dt * divy / ry;
    }
    if (useful) {
      V.vx3[c] = vxn;
      V.vy3[c] = vyn;
    }
    rho_s = C.rho;
    tpp_s = tpp;
    trr_s = trr;
    trp = trp_n;
    C = N;
    pC = pN;
  }
  if (ch == V.nchunk - 1)
    for (int j = m.jn; j < m.nyg; j++) carry(j);
}

template <typename F>
__global__ __launch_bounds__(256) void k_visc(Visc<F> V) {
  visc_body<F>(V, blockIdx.x, gridDim.x);
}

// multi-mesh form (ManyGrid)
template <typename F>
struct ViscArgs {
  Visc<F> V;
  unsigned nb, pad_;
};
template <typename F>
__global__ __launch_bounds__(256) void k_visc_many(const void *args, const uint2 *tab) {
  const uint2 t = many_block(tab);
  if (t.x == MANY_NONE) return;
  const ViscArgs<F> a = many_args<ViscArgs<F>>(args, t.x);
  visc_body<F>(a.V, t.y, a.nb);
}

// the pass over mesh m with chunks of at most `rows` rows, as many as `slots`
// waves can share (0: no more than that takes), and its blocks
template <typename F>
Visc<F> visc_of(const Mesh &m, const StateT<F> &s, const F *vx2, const F *vy2, F *vx3, F *vy3, const double *dt,
                long slots, int rows, unsigned &nb) {
  Visc<F> V{m, s, vx2, vy2, dt, vx3, vy3, (m.nx + VISC_U - 1) / VISC_U, 0, 0};
  int nch = slots ? fill_chunks(m.ny, rows, 1, V.nseg, slots, 2) : (m.ny + rows - 1) / rows;
  V.chunk = (m.ny + nch - 1) / nch;
  V.nchunk = (m.ny + V.chunk - 1) / V.chunk;
  nb = (unsigned)(((long)V.nseg * V.nchunk + 3) / 4);
  return V;
}

} // namespace

template <typename F>
void launch_visc(Launch &L, const Mesh &m, const StateT<F> &s, const F *vx2, const F *vy2, F *vx3, F *vy3,
                 const double *dt) {
  static const long slots = 4 * block_slots(k_visc<F>, 256);
  unsigned nb;
  const Visc<F> V = visc_of(m, s, vx2, vy2, vx3, vy3, dt, slots, VISC_ROWS, nb);
  prof_begin(L, K_VISC);
  k_visc<F><<<nb, 256, 0, L.s>>>(V);
  prof_end(L, K_VISC);
}

template <typename F>
size_t visc_args_bytes() { return sizeof(ViscArgs<F>); }

template <typename F>
int visc_rows(const std::vector<Mesh> &ms) {
  static const long slots = 4 * block_slots(k_visc_many<F>, 256);
  return fill_chunk_length(ms, VISC_ROWS, slots, 2, [](const Mesh &m) { return (m.nx + VISC_U - 1) / VISC_U; });
}

template <typename F>
unsigned visc_args(const Mesh &m, const StateT<F> &s, const F *vx2, const F *vy2, F *vx3, F *vy3, const double *dt,
                   int rows, void *dst) {
  unsigned nb;
  const Visc<F> V = visc_of(m, s, vx2, vy2, vx3, vy3, dt, 0L, rows, nb);
  *(ViscArgs<F> *)dst = ViscArgs<F>{V, nb, 0};
  return nb;
}

template <typename F>
void launch_visc_many(Launch &L, const ManyGrid &g) {
  prof_begin(L, K_VISC);
  k_visc_many<F><<<g.nblk, 256, 0, L.s>>>(g.args, g.tab);
  prof_end(L, K_VISC);
}

#define FARGO_VISC(F)                                                                                               \
  template void launch_visc<F>(Launch &, const Mesh &, const StateT<F> &, const F *, const F *, F *, F *,          \
                               const double *);                                                                    \
  template size_t visc_args_bytes<F>();                                                                            \
  template int visc_rows<F>(const std::vector<Mesh> &);                                                            \
  template unsigned visc_args<F>(const Mesh &, const StateT<F> &, const F *, const F *, F *, F *, const double *,  \
                                 int, void *);                                                                        \
  template void launch_visc_many<F>(Launch &, const ManyGrid &);
FARGO_VISC(double)
FARGO_VISC(float)
#undef FARGO_VISC

} // namespace fargo
