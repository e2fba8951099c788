// Boxes 2 and 9: boundary conditions in the three ghost layers of Y and Z
// (Sect. 4.1).  X is periodic through index arithmetic and has no ghosts.
//
// Per side: PERIODIC copies the opposite edge; REFLECT mirrors zone-centred
// fields and tangential velocities, makes the normal velocity antisymmetric
// and sets the boundary face to zero; OUTFLOW copies the edge zone and the
// first interior face; FIXED writes nothing.  The Y sides are filled over every
// Z row before the Z sides over every Y column (corners consistent).  An FP32
// v_x (a deviation from its ring's background) is copied with the difference of
// the two rings' backgrounds.
#include "fargo_internal.h"

namespace fargo {

namespace {

template <typename R>
struct Cen {
  R *p[4];
  int n;
  int ivx; // index of v_x in p (-1 if absent)
};

__device__ inline size_t at(const Mesh &m, int dir, int i, int a, int b) {
  return dir == 1 ? m.idx(i, a, b) : m.idx(i, b, a);
}

// Both sides of a direction in one launch: a block of a row of zones for each
// row b of the other direction, side and layer, where layer 0 is the boundary
// face and 1 .. nlay the ghost layers outwards.  Only ghosts and boundary
// faces are written and only zones and faces inside are read (the values the
// boundary faces take are formed where a ghost face mirrors one), so the
// layers of a side, and the sides, need no order.  (Faces, then ghosts, side
// after side, were eight launches of some 5 us each on a small mesh for what
// are two now.)
template <typename R>
__global__ __launch_bounds__(256) void k_bc(Mesh m, int dir, int side0, int nside, int nlay, int nib, Cen<R> cen,
                                            R *vn) {
  const int lo = dir == 1 ? m.j0 : m.k0, hi = dir == 1 ? m.jn : m.kn, s0 = dir == 1 ? 0 : 2;
  unsigned t = blockIdx.x;
  const int i = (int)(t % (unsigned)nib) * (int)blockDim.x + (int)threadIdx.x;
  t /= (unsigned)nib;
  const int layer = (int)(t % (unsigned)(nlay + 1));
  t /= (unsigned)(nlay + 1);
  const int side = side0 + (int)(t % (unsigned)nside), b = (int)(t / (unsigned)nside);
  if (i >= m.nx) return;
  const int kind = m.bc[s0 + side];
  auto v = [&](int f) { return vn[at(m, dir, i, f, b)]; };
  // the boundary face of a side, once set
  auto bface = [&](int sd) {
    const int k = m.bc[s0 + sd];
    if (k == FARGO_BC_REFLECT) return R(0);
    if (k == FARGO_BC_OUTFLOW) return v(sd == 0 ? lo + 1 : hi - 1);
    if (k == FARGO_BC_PERIODIC) return v(lo); // owned below, its image above
    return v(sd == 0 ? lo : hi);
  };
  if (layer == 0) {
    if (kind == FARGO_BC_PERIODIC && side == 0) return; // the lower face is owned by the step
    vn[at(m, dir, i, side == 0 ? lo : hi, b)] = bface(side);
    return;
  }
  const int g = layer - 1;
  int dst, src, fdst = -1, fsrc = -1;
  R sgn = R(1);
  if (side == 0) {
    dst = lo - 1 - g;
    fdst = lo - 1 - g;
    if (kind == FARGO_BC_PERIODIC) { src = hi - 1 - g; fsrc = hi - 1 - g; }
    else if (kind == FARGO_BC_REFLECT) { src = lo + g; fsrc = lo + 1 + g; sgn = R(-1); }
    else { src = lo; fsrc = lo; }
  } else {
    dst = hi + g;
    if (g < NGH - 1) fdst = hi + 1 + g;
    if (kind == FARGO_BC_PERIODIC) { src = lo + g; fsrc = lo + 1 + g; }
    else if (kind == FARGO_BC_REFLECT) { src = hi - 1 - g; fsrc = hi - 1 - g; sgn = R(-1); }
    else { src = hi - 1; fsrc = hi; }
  }
  const size_t d = at(m, dir, i, dst, b), s = at(m, dir, i, src, b);
  R c[4];
#pragma unroll
  for (int q = 0; q < 4; q++)
    if (q < cen.n) c[q] = cen.p[q][s];
  R f = R(0);
  if (fdst >= 0) f = sgn * (fsrc == lo ? bface(0) : fsrc == hi ? bface(1) : v(fsrc));
  if constexpr (sizeof(R) == 4) {
    // FP32 v_x is a deviation from the ring's background: the ghost takes the
    // source's full velocity, so the two backgrounds' difference is added
    const int jd = dir == 1 ? dst : b, kd = dir == 1 ? b : dst;
    const int js = dir == 1 ? src : b, ks = dir == 1 ? b : src;
    const R off = (R)(m.bg(BG_V, js, ks) - m.bg(BG_V, jd, kd));
#pragma unroll
    for (int q = 0; q < 4; q++)
      if (q == cen.ivx) c[q] += off;
  }
#pragma unroll
  for (int q = 0; q < 4; q++)
    if (q < cen.n) cen.p[q][d] = c[q];
  if (fdst >= 0) vn[at(m, dir, i, fdst, b)] = f;
}

template <typename R>
void one_dir(Launch &L, const Mesh &m, int dir, int nlay, const Cen<R> &cen, R *vn) {
  const int s0 = dir == 1 ? 0 : 2;
  const bool f0 = m.bc[s0] == FARGO_BC_FIXED, f1 = m.bc[s0 + 1] == FARGO_BC_FIXED;
  if (f0 && f1) return;
  int nib, bs;
  row_blocks(m.nx, nib, bs);
  const int nside = f0 || f1 ? 1 : 2, nb = dir == 1 ? m.nzg : m.nyg;
  const unsigned blocks = (unsigned)nib * (unsigned)nb * (unsigned)(nside * (nlay + 1));
  prof_begin(L, K_BC);
  k_bc<R><<<blocks, bs, 0, L.s>>>(m, dir, f0 ? 1 : 0, nside, nlay, nib, cen, vn);
  prof_end(L, K_BC);
}

} // namespace

// Box 9 (post) refills copies that one step reads: the density's ghosts, which
// box 2 has filled and box 7 does not change, are left, and so is the third
// layer, which no sweep reads (a face of it on the upper sides comes with the
// second).
template <typename R>
void launch_bc(Launch &L, const Mesh &m, R *rho, R *e, R *vx, R *vy, R *vz, bool post) {
  const int nlay = post ? 2 : NGH;
  Cen<R> cy{};
  if (!post) cy.p[cy.n++] = rho;
  if (e) cy.p[cy.n++] = e;
  cy.ivx = cy.n;
  cy.p[cy.n++] = vx;
  if (m.d3) cy.p[cy.n++] = vz;
  one_dir(L, m, 1, nlay, cy, vy);
  if (!m.d3) return;
  Cen<R> cz{};
  if (!post) cz.p[cz.n++] = rho;
  if (e) cz.p[cz.n++] = e;
  cz.ivx = cz.n;
  cz.p[cz.n++] = vx;
  cz.p[cz.n++] = vy;
  one_dir(L, m, 2, nlay, cz, vz);
}

template void launch_bc<double>(Launch &, const Mesh &, double *, double *, double *, double *, double *, bool);
template void launch_bc<float>(Launch &, const Mesh &, float *, float *, float *, float *, float *, bool);

} // namespace fargo
