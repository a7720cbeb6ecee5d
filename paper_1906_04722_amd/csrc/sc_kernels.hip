// sc_kernels.hip -- gfx950 kernels of the two-component Shan-Chen D3Q19
// update (Montella et al., Sec. 2.1, Eq. 1-5) on one pore-throat subdomain.
//
// Storage: shifted FP32 populations g = f - w_k rho_ref of numbered nodes, each
// population of 32 consecutive numbers one 128-byte line (numberings, index
// map and ghost planes in sc_internal.h).  The update is a pull scheme: buffer
// `src` holds the post-collision state of step t-1 at each node's own
// position; pulling g_k from x - e_k gives the pre-collision state f(x, t) of
// Eq. 1: pull + half-way bounce-back, moments (Eq. 2-3), the cohesion force
// (Eq. 4) from the 18 neighbours' densities, the adhesion force from the
// node's cut links, the velocity shift, BGK relaxation toward the component
// equilibria (Eq. 1) and the store of the post-collision state.
#include <algorithm>
#include <cmath>
#include <mutex>
#include <type_traits>

#include "geom.h"
#include "sc_internal.h"

// Multiply-adds are fused only where one source expression reads a * b + c,
// never across statements, so every kernel that shares the arithmetic below
// (both steps, the reduction, the export) rounds it identically.
#pragma clang fp contract(on)

namespace sc {

// ---- D3Q19: rest; +x,-x,+y,-y,+z,-z; twelve edges, opposite pairs adjacent
__host__ __device__ constexpr int ex(int k) {
  constexpr int t[19] = {0, 1, -1, 0, 0, 0, 0, 1, -1, 1, -1, 1, -1, 1, -1, 0, 0, 0, 0};
  return t[k];
}
__host__ __device__ constexpr int ey(int k) {
  constexpr int t[19] = {0, 0, 0, 1, -1, 0, 0, 1, -1, -1, 1, 0, 0, 0, 0, 1, -1, 1, -1};
  return t[k];
}
__host__ __device__ constexpr int ez(int k) {
  constexpr int t[19] = {0, 0, 0, 0, 0, 1, -1, 0, 0, 0, 0, 1, -1, -1, 1, 1, -1, -1, 1};
  return t[k];
}
__host__ __device__ constexpr int opp(int k) { return k == 0 ? 0 : ((k & 1) ? k + 1 : k - 1); }
__host__ __device__ constexpr float wf(int k) {
  return k == 0 ? 1.0f / 3.0f : (k <= 6 ? 1.0f / 18.0f : 1.0f / 36.0f);
}
__host__ __device__ constexpr double wd(int k) {
  return k == 0 ? 1.0 / 3.0 : (k <= 6 ? 1.0 / 18.0 : 1.0 / 36.0);
}

// ---- node addressing ------------------------------------------------------

// global-memory views of the buffers: loads and stores then take a uniform
// 64-bit base and a 32-bit per-lane offset
typedef const __attribute__((address_space(1))) char gcchar;
typedef __attribute__((address_space(1))) char gchar;
typedef const __attribute__((address_space(1))) uint32_t gcu32;
typedef const __attribute__((address_space(1))) float gcfloat;
typedef __attribute__((address_space(1))) float gfloat;

// Numbers of a node's D3Q19 neighbours: the nine rows (y + dy, z + dz) of the
// index map around it, three of x - 1 .. x + 1 where D3Q19 has them all.
struct Near {
  uint32_t r[5][3];  // rows (0, 0), (-1, 0), (1, 0), (0, -1), (0, 1) of (dy, dz)
  uint32_t c[4];     // x itself in rows (-1, -1), (1, -1), (-1, 1), (1, 1)
};
// number of the node at x + (DX, DY, DZ)
template <int DX, int DY, int DZ>
__device__ __forceinline__ uint32_t near_at(const Near &n) {
  static_assert(DX * DX + DY * DY + DZ * DZ <= 2, "a D3Q19 neighbour");
  if constexpr (DY != 0 && DZ != 0)
    return n.c[(DY > 0 ? 1 : 0) + (DZ > 0 ? 2 : 0)];
  else
    return n.r[DZ != 0 ? (DZ < 0 ? 3 : 4) : (DY != 0 ? (DY < 0 ? 1 : 2) : 0)][1 + DX];
}

// the map element at map + off is position (x - 1, y - 1, z - 1); px, pp: row
// and plane strides of the map.  (Written out row by row: an index that is
// constant only after unrolling can keep a Near in memory.)
template <class Off, int DY, int DZ>
__device__ __forceinline__ gcchar *near_row(const uint32_t *map, Off off, uint32_t px, size_t pp) {
  return (gcchar *)(map + (size_t)(1 + DZ) * pp + (size_t)((uint32_t)(1 + DY) * px)) +
         (size_t)(Off)(off * (Off)4);
}
template <class Off>
__device__ __forceinline__ void load_near(const uint32_t *map, Off off, uint32_t px, size_t pp,
                                          Near &n) {
#define NEAR_ROW(i, DY, DZ)                                       \
  {                                                               \
    gcchar *row = near_row<Off, DY, DZ>(map, off, px, pp);        \
    n.r[i][0] = *(gcu32 *)row;                                    \
    n.r[i][1] = *(gcu32 *)(row + 4);                              \
    n.r[i][2] = *(gcu32 *)(row + 8);                              \
  }
  NEAR_ROW(0, 0, 0)
  NEAR_ROW(1, -1, 0)
  NEAR_ROW(2, 1, 0)
  NEAR_ROW(3, 0, -1)
  NEAR_ROW(4, 0, 1)
#undef NEAR_ROW
  n.c[0] = *(gcu32 *)(near_row<Off, -1, -1>(map, off, px, pp) + 4);
  n.c[1] = *(gcu32 *)(near_row<Off, 1, -1>(map, off, px, pp) + 4);
  n.c[2] = *(gcu32 *)(near_row<Off, -1, 1>(map, off, px, pp) + 4);
  n.c[3] = *(gcu32 *)(near_row<Off, 1, 1>(map, off, px, pp) + 4);
}

// Element of population 0 of node i within its buffer, and the same in bytes
// where a buffer is small enough for 32 bits (one full-rate 24-bit
// multiply-add; i >> 5 < 2^24 there).
__device__ __forceinline__ size_t node_elem(uint32_t i) {
  return (size_t)(i >> 5) * (size_t)(kQ * kLine) + (size_t)(i & 31u);
}
__device__ __forceinline__ uint32_t node_bytes(uint32_t i) {
  return __umul24(i >> 5, (uint32_t)(4 * (kQ - 1) * kLine)) + (i << 2);
}

// Pull the pre-collision populations f(x,t) - w_k rho_ref of the fluid node
// with number i: g_k from x - e_k, or the reflected g_opp(k) of the node
// itself when x - e_k is solid or beyond a wall (half-way bounce-back).  m
// receives the cut links (bits 1..18).  WIDE: 64-bit addresses per lane; else
// one uniform base and 32-bit byte offsets, kept one line above the start so
// that the reflected slot of the first node does not go below zero.
template <bool WIDE, int K>
__device__ __forceinline__ void pull_rec(const float *src, uint32_t i, const Near &n, uint32_t &m,
                                         float (&v)[2][19]) {
  constexpr int o = opp(K);
  const uint32_t s = near_at<-ex(K), -ey(K), -ez(K)>(n);
  const bool cut = K != 0 && s == kNoNode;
  if (K != 0) m |= cut ? 1u << K : 0u;
  // selects, not branches: the 38 loads issue back to back
  const uint32_t j = cut ? i : s;
  const int shift = cut ? (o - K) * 4 * kLine : 0;
  gcchar *p;
  if constexpr (WIDE)
    p = (gcchar *)(src + node_elem(j)) + shift;
  else
    p = (gcchar *)src - 4 * kLine + (size_t)(node_bytes(j) + (uint32_t)(4 * kLine + shift));
  v[0][K] = *(gcfloat *)(p + K * 4 * kLine);
  v[1][K] = *(gcfloat *)(p + (19 + K) * 4 * kLine);
  if constexpr (K + 1 < 19) pull_rec<WIDE, K + 1>(src, i, n, m, v);
}

template <bool WIDE>
__device__ __forceinline__ void pull(const float *src, const Near &n, uint32_t &m,
                                     float (&v)[2][19]) {
  m = 0;
  pull_rec<WIDE, 0>(src, n.r[0][1], n, m, v);
}

// the same for the node at (x, y, z) of the box
__device__ __forceinline__ void pull_at(const Dom &d, int x, int y, int z, float (&v)[2][19]) {
  Near n;
  uint32_t m;
  const uint32_t px = (uint32_t)(d.nx + 2 * kPad);
  load_near<size_t>(d.map, map_pos(d.nx, d.ny, x - 1, y - 1, z - 1), px,
                    (size_t)px * (size_t)(d.ny + 2 * kPad), n);
  pull<true>(d.src, n, m, v);
}

// class of a box node: solid without a number, a bath on the first and last
// plane of a subdomain with baths
__device__ __forceinline__ uint32_t class_at(const Dom &d, int x, int y, int z) {
  if (d.map[map_pos(d.nx, d.ny, x, y, z)] == kNoNode) return kSolid;
  if (d.res && z == 0) return kResIn;
  if (d.res && z == d.nz - 1) return kResOut;
  return kFluid;
}

// Type of the density sums.  Populations are stored in FP32 (the HBM
// bytes); the 19-term density sums are FP64 (see collide() for the rest).
typedef double acc_t;

__device__ __forceinline__ acc_t sum19(const float (&a)[19]) {
  acc_t s = 0;
#pragma unroll
  for (int k = 0; k < 19; ++k) s += (acc_t)a[k];
  return s;
}

// BGK collision of one fluid node (Eq. 1 right-hand side) with the cohesion
// force of Eq. 4 (S = sum_k w_k rho(x + e_k) e_k of each component, from the
// density stencil) and the adhesion force toward solid neighbours, entering
// through the velocity shift u_eq = u' + tau F / rho.  v: pulled shifted
// populations in, post-collision shifted populations out.
//
// Precision: the densities (sum of the 19 populations) and the post-collision
// rest population are FP64; momenta, forces, velocities and the 18 moving
// equilibria are FP32.  The rest population is set to the FP64 density minus
// the 18 moving post-collision values, so the collision conserves each
// component's mass to FP64 rounding (the BGK update does so exactly), and
// FP32 rounding of the weights (their FP32 sum is not exactly 1) cannot bias
// the mass step after step.  Momenta are summed from opposite-pair
// differences.  drd: the FP64 sums of each component's 19 shifted
// populations, as taken when the node was pulled; m: the node's cut links (bits 1..18).
//
// It comes in parts, so that one lane can take both components of a node or
// one lane each.

// density shift, density and momentum of one component
__device__ __forceinline__ void moments(const Phys &P, double drd, const float (&v)[19], float &dr,
                                        float &rho, float (&j)[3]) {
  dr = (float)drd;
  rho = (float)((double)P.rho_ref + drd);
  float jx = 0.f, jy = 0.f, jz = 0.f;
#pragma unroll
  for (int k = 1; k < 19; ++k) {
    if (k > opp(k)) continue;
    const float dk = v[k] - v[opp(k)];
    if (ex(k)) jx += ex(k) > 0 ? dk : -dk;
    if (ey(k)) jy += ey(k) > 0 ? dk : -dk;
    if (ez(k)) jz += ez(k) > 0 ? dk : -dk;
  }
  j[0] = jx;
  j[1] = jy;
  j[2] = jz;
}

// adhesion direction: zero (the same +0 the sum gives) when no link is cut
__device__ __forceinline__ void adhesion(uint32_t m, float (&A)[3]) {
  A[0] = A[1] = A[2] = 0.f;
  if ((m & kLinkBits) == 0u) return;
#pragma unroll
  for (int k = 1; k < 19; ++k) {
    const float s = (float)((m >> opp(k)) & 1u) * wf(k);
    if (ex(k)) A[0] += ex(k) > 0 ? s : -s;
    if (ey(k)) A[1] += ey(k) > 0 ? s : -s;
    if (ez(k)) A[2] += ez(k) > 0 ? s : -s;
  }
}

// force on a component: S from the other component's densities
__device__ __forceinline__ void force(const Phys &P, float Gads, float rho, const float (&S)[3],
                                      const float (&A)[3], float (&F)[3]) {
#pragma unroll
  for (int a = 0; a < 3; ++a) F[a] = -P.G * rho * S[a] - Gads * rho * A[a];
}

// common velocity (quotients as products with three reciprocals)
__device__ __forceinline__ void velocity(const Phys &P, float rho0, float rho1,
                                         const float (&j0)[3], const float (&j1)[3],
                                         float (&up)[3]) {
  const float it0 = P.itau[0], it1 = P.itau[1];
  const float den = rho0 * it0 + rho1 * it1;
  const float iden = 1.0f / den;
#pragma unroll
  for (int a = 0; a < 3; ++a) up[a] = (j0[a] * it0 + j1[a] * it1) * iden;
}

// relaxation of one component
__device__ __forceinline__ void relax(float tc, float itc, const float (&up)[3],
                                      const float (&F)[3], double drd, float dr, float rho,
                                      float (&v)[19]) {
  float u[3];
  const float irho = 1.0f / rho;
#pragma unroll
  for (int a = 0; a < 3; ++a) u[a] = up[a] + tc * F[a] * irho;
  const float uu = u[0] * u[0] + u[1] * u[1] + u[2] * u[2];
  double rest = drd;
#pragma unroll
  for (int k = 1; k < 19; ++k) {
    float eu = 0.f;
    if (ex(k)) eu += ex(k) > 0 ? u[0] : -u[0];
    if (ey(k)) eu += ey(k) > 0 ? u[1] : -u[1];
    if (ez(k)) eu += ez(k) > 0 ? u[2] : -u[2];
    const float geq = wf(k) * (dr + rho * (3.f * eu + 4.5f * eu * eu - 1.5f * uu));
    const float g = v[k];
    const float gs = g - (g - geq) * itc;
    v[k] = gs;
    rest -= (double)gs;
  }
  v[0] = (float)rest;
}

__device__ __forceinline__ void collide(const Phys &P, uint32_t m, const float (&Sw)[3],
                                        const float (&Sn)[3], const double (&drd)[2],
                                        float (&v)[2][19]) {
  float dr[2], rho[2], j[2][3], A[3], F[2][3], up[3];
  moments(P, drd[0], v[0], dr[0], rho[0], j[0]);
  moments(P, drd[1], v[1], dr[1], rho[1], j[1]);
  adhesion(m, A);
  force(P, P.Gads[0], rho[0], Sn, A, F[0]);
  force(P, P.Gads[1], rho[1], Sw, A, F[1]);
  velocity(P, rho[0], rho[1], j[0], j[1], up);
  relax(P.tau[0], P.itau[0], up, F[0], drd[0], dr[0], rho[0], v[0]);
  relax(P.tau[1], P.itau[1], up, F[1], drd[1], dr[1], rho[1], v[1]);
}

// Store the post-collision populations of node i.  KEEP: through the caches as
// any store; else non-temporal.
template <bool WIDE, bool KEEP>
__device__ __forceinline__ void store_node(float *dst, uint32_t i, const float (&v)[2][19]) {
  gchar *p = WIDE ? (gchar *)(dst + node_elem(i)) : (gchar *)dst + (size_t)node_bytes(i);
#pragma unroll
  for (int c = 0; c < 2; ++c)
#pragma unroll
    for (int k = 0; k < 19; ++k) {
      gfloat *q = (gfloat *)(p + (19 * c + k) * 4 * kLine);
      if constexpr (KEEP)
        *q = v[c][k];
      else
        __builtin_nontemporal_store(v[c][k], q);
    }
}

// work lists are handed out so that each XCD (workgroups b = xcd mod 8) gets
// one contiguous range, keeping spatial neighbours in one L2
__device__ __forceinline__ int xcd_item(int n) {
  const int b = blockIdx.x, q = n >> 3, r = n & 7, xcd = b & 7, idx = b >> 3;
  return xcd * q + min(xcd, r) + idx;
}

// ---- two passes over the non-solid nodes --------------------------------------------
// k_dens writes each non-solid node's two densities, k_node pulls again, takes
// the 18-neighbour density stencil from that array, collides and stores.
//
// Bound: the rate at which the eight L2s exchange lines with the memory side
// (6.2 TB/s for a copy).  A step fetches 152 + 152 bytes of populations per
// node, 16 of positions and densities and the index map twice, and writes 160:
// 2.19 GB and 1.02 GB on the 256^3 packed sample (6.4 M of 16.8 M nodes), where
// 2.19 and 1.02 were counted.  Before, one fused pass
// in tiles over all nodes of the box refetched halo lines and moved partly used
// lines: 3.7 GB and 873-893 us a step on that sample, now 660; 40-sphere
// sample with membrane 113 -> 64 us (57 with kept stores), 96^3 throat 18.4 ->
// 12.9 us, 40^3 throat 11.4 (33 in the default tile shape) -> 6.5 us.
//
// Whole rows along x make a wavefront's 64 nodes pull runs of 3-4 lines per
// population; groups of 32 rows marched through z keep the lines that links to
// z + 1 and z - 1 share in the L2 until both have read them (raster order over
// whole planes: 2.86 GB fetched, 676 us; blocks of 8^3: 776 us).  Workgroups of
// one wavefront: those of two or four put a CU's wavefronts on the same SIMDs
// or leave CUs idle where the chip is not full (us a step with workgroups of
// 64 / 128 / 256: 1 k nodes 7.2 / 7.5 / 8.3, 41 k 8.4 / 10.1 / 8.9, 55 k 10.1
// / 11.5, 131 k 13.2 / 13.4 / 13.3), large ones do not care.
// Not faster: one kernel that keeps the densities of a block and its halo in
// LDS (929-1300 us on the sample: the halo's pulls cost twice the arithmetic),
// and the second pass trailing the first by a part that fits the 256 MB
// memory-side cache (690-950 us: the second read costs the same L2 misses).
__device__ __forceinline__ bool list_item(const Throat *__restrict__ throats,
                                          const TileRef *__restrict__ items, int nitems,
                                          const Throat *&T, uint32_t &i) {
  const int k = xcd_item(nitems);
  const TileRef it = items ? items[k] : TileRef{0, k};
  T = throats + it.throat;
  i = (uint32_t)it.tile * kListNodes + threadIdx.x;
  return T->active && i < T->n_live;
}

// bath of the node at map position pos: 0 inlet, 1 outlet, -1 none
__device__ __forceinline__ int bath_of(const Throat &T, uint32_t pos, size_t pp) {
  if (!T.res) return -1;
  if ((size_t)pos < (size_t)(1 + kPad) * pp) return 0;
  return (size_t)pos >= (size_t)(T.nz - 1 + kPad) * pp ? 1 : -1;
}

template <bool WIDE>
__device__ __forceinline__ void near_of(const Throat &T, uint32_t pos, uint32_t px, size_t pp,
                                        Near &n) {
  typedef typename std::conditional<WIDE, size_t, uint32_t>::type Off;
  load_near<Off>(T.map - pp - px - 1, (Off)pos, px, pp, n);
}

template <bool WIDE>
__global__ __launch_bounds__(kListNodes) void k_dens(const Throat *__restrict__ throats,
                                                     const TileRef *__restrict__ items,
                                                     int nitems, int parity) {
  const Throat *Tp;
  uint32_t i;
  if (!list_item(throats, items, nitems, Tp, i)) return;
  const Throat &T = *Tp;
  const uint32_t px = (uint32_t)(T.nx + 2 * kPad);
  const size_t pp = (size_t)px * (size_t)(T.ny + 2 * kPad);
  const uint32_t pos = *(gcu32 *)((gcchar *)T.pos + (size_t)i * 4);
  const int bath = bath_of(T, pos, pp);
  if (bath >= 0) {
    const bool in = bath == 0;
    T.rho[T.map[pos]] = make_float2(in ? T.P.rres[0][0] : T.P.rres[1][0],
                                    in ? T.P.rres[0][1] : T.P.rres[1][1]);
    return;
  }
  Near n;
  uint32_t m;
  float v[2][19];
  near_of<WIDE>(T, pos, px, pp, n);
  pull<WIDE>(T.g[parity], n, m, v);
  T.rho[n.r[0][1]] = make_float2((float)((acc_t)T.P.rho_ref + sum19(v[0])),
                                 (float)((acc_t)T.P.rho_ref + sum19(v[1])));
}

// densities of the neighbours x + e_k, zero where there is none
template <bool WIDE, int K>
__device__ __forceinline__ void stencil_rec(const float2 *rho, const Near &n, float2 (&r)[19]) {
  typedef typename std::conditional<WIDE, size_t, uint32_t>::type Off;
  const uint32_t s = near_at<ex(K), ey(K), ez(K)>(n);
  const bool none = s == kNoNode;
  gcchar *p = (gcchar *)rho + (size_t)((Off)(none ? n.r[0][1] : s) * (Off)8);
  r[K] = make_float2(*(gcfloat *)p, *(gcfloat *)(p + 4));
  if (none) r[K] = make_float2(0.f, 0.f);
  if constexpr (K + 1 < 19) stencil_rec<WIDE, K + 1>(rho, n, r);
}

template <bool WIDE, bool KEEP>
__global__ __launch_bounds__(kListNodes) void k_node(const Throat *__restrict__ throats,
                                                     const TileRef *__restrict__ items,
                                                     int nitems, int parity) {
  const Throat *Tp;
  uint32_t i;
  if (!list_item(throats, items, nitems, Tp, i)) return;
  const Throat &T = *Tp;
  const uint32_t px = (uint32_t)(T.nx + 2 * kPad);
  const size_t pp = (size_t)px * (size_t)(T.ny + 2 * kPad);
  const uint32_t pos = *(gcu32 *)((gcchar *)T.pos + (size_t)i * 4);
  const Phys P = T.P;
  const int bath = bath_of(T, pos, pp);
  if (bath >= 0) {
    const float gw = bath == 0 ? P.gres[0][0] : P.gres[1][0];
    const float gn = bath == 0 ? P.gres[0][1] : P.gres[1][1];
    float v[2][19];
#pragma unroll
    for (int k = 0; k < 19; ++k) {
      v[0][k] = wf(k) * gw;
      v[1][k] = wf(k) * gn;
    }
    store_node<WIDE, KEEP>(T.g[parity ^ 1], T.map[pos], v);
    return;
  }
  Near n;
  uint32_t m;
  float v[2][19];
  float2 r[19];
  near_of<WIDE>(T, pos, px, pp, n);
  pull<WIDE>(T.g[parity], n, m, v);
  stencil_rec<WIDE, 1>(T.rho, n, r);
  float Sw[3] = {0, 0, 0}, Sn[3] = {0, 0, 0};
#pragma unroll
  for (int k = 1; k < 19; ++k) {
    const float a = wf(k) * r[k].x, bb = wf(k) * r[k].y;
    if (ex(k)) { Sw[0] += ex(k) > 0 ? a : -a; Sn[0] += ex(k) > 0 ? bb : -bb; }
    if (ey(k)) { Sw[1] += ey(k) > 0 ? a : -a; Sn[1] += ey(k) > 0 ? bb : -bb; }
    if (ez(k)) { Sw[2] += ez(k) > 0 ? a : -a; Sn[2] += ez(k) > 0 ? bb : -bb; }
  }
  const double ds[2] = {sum19(v[0]), sum19(v[1])};
  collide(P, m, Sw, Sn, ds, v);
  store_node<WIDE, KEEP>(T.g[parity ^ 1], n.r[0][1], v);
}

// ---- the two passes with a lane per component ---------------------------------------
// For subdomains that leave the chip with a wavefront or less per SIMD, where a
// step is the time of one wavefront through both kernels: lanes l and l + 32
// share a node and take one component each, half the loads, sums and
// relaxation per wavefront and twice the wavefronts.  They exchange density
// and momentum for the common velocity, and each reads the other component's
// densities for its force.  Same arithmetic, same bits.

// the 32-bit value of lanes l and l + 32, in both
__device__ __forceinline__ void both(float x, float &x0, float &x1) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false,
                                                  false);
  x0 = __uint_as_float(r[0]);
  x1 = __uint_as_float(r[1]);
}

template <int K>
__device__ __forceinline__ void pull_one(const float *src, uint32_t cofs, uint32_t i,
                                         const Near &n, uint32_t &m, float (&v)[19]) {
  constexpr int o = opp(K);
  const uint32_t s = near_at<-ex(K), -ey(K), -ez(K)>(n);
  const bool cut = K != 0 && s == kNoNode;
  if (K != 0) m |= cut ? 1u << K : 0u;
  const uint32_t j = cut ? i : s;
  const uint32_t shift = cofs + (uint32_t)(cut ? (o - K) * 4 * kLine : 0);
  v[K] = *(gcfloat *)((gcchar *)src - 4 * kLine + (size_t)(node_bytes(j) + shift) + K * 4 * kLine);
  if constexpr (K + 1 < 19) pull_one<K + 1>(src, cofs, i, n, m, v);
}

template <int K>
__device__ __forceinline__ void stencil_one(const float2 *rho, uint32_t cofs, const Near &n,
                                            float (&r)[19]) {
  const uint32_t s = near_at<ex(K), ey(K), ez(K)>(n);
  const bool none = s == kNoNode;
  r[K] = *(gcfloat *)((gcchar *)rho + (size_t)((none ? n.r[0][1] : s) * 8u + cofs));
  if (none) r[K] = 0.f;
  if constexpr (K + 1 < 19) stencil_one<K + 1>(rho, cofs, n, r);
}

// a workgroup takes half an item; c: this lane's component
__device__ __forceinline__ bool split_item(const Throat *__restrict__ throats,
                                           const TileRef *__restrict__ items, int nitems,
                                           const Throat *&T, uint32_t &i, int &c) {
  const int half = xcd_item(2 * nitems);
  const TileRef it = items ? items[half >> 1] : TileRef{0, half >> 1};
  T = throats + it.throat;
  i = (uint32_t)it.tile * kListNodes + (uint32_t)(half & 1) * 32u + (threadIdx.x & 31u);
  c = (int)(threadIdx.x >> 5);
  return T->active && i < T->n_live;
}

__global__ __launch_bounds__(kListNodes) void k_dens_split(const Throat *__restrict__ throats,
                                                           const TileRef *__restrict__ items,
                                                           int nitems, int parity) {
  const Throat *Tp;
  uint32_t i;
  int c;
  if (!split_item(throats, items, nitems, Tp, i, c)) return;
  const Throat &T = *Tp;
  const uint32_t px = (uint32_t)(T.nx + 2 * kPad);
  const size_t pp = (size_t)px * (size_t)(T.ny + 2 * kPad);
  const uint32_t pos = *(gcu32 *)((gcchar *)T.pos + (size_t)i * 4);
  const int bath = bath_of(T, pos, pp);
  float *rho = (float *)T.rho;
  if (bath >= 0) {
    const float w = bath == 0 ? T.P.rres[0][0] : T.P.rres[1][0];
    const float nw = bath == 0 ? T.P.rres[0][1] : T.P.rres[1][1];
    rho[2 * T.map[pos] + c] = c ? nw : w;
    return;
  }
  Near n;
  uint32_t m = 0;
  float v[19];
  near_of<false>(T, pos, px, pp, n);
  pull_one<0>(T.g[parity], (uint32_t)(4 * kLine) + (uint32_t)c * (19 * 4 * kLine), n.r[0][1], n, m,
              v);
  rho[2 * n.r[0][1] + c] = (float)((acc_t)T.P.rho_ref + sum19(v));
}

__global__ __launch_bounds__(kListNodes) void k_node_split(const Throat *__restrict__ throats,
                                                           const TileRef *__restrict__ items,
                                                           int nitems, int parity) {
  const Throat *Tp;
  uint32_t i;
  int c;
  if (!split_item(throats, items, nitems, Tp, i, c)) return;
  const Throat &T = *Tp;
  const uint32_t px = (uint32_t)(T.nx + 2 * kPad);
  const size_t pp = (size_t)px * (size_t)(T.ny + 2 * kPad);
  const uint32_t pos = *(gcu32 *)((gcchar *)T.pos + (size_t)i * 4);
  const Phys P = T.P;
  const int bath = bath_of(T, pos, pp);
  const uint32_t cofs = (uint32_t)c * (19 * 4 * kLine);
  uint32_t own;
  float v[19];
  if (bath >= 0) {
    const float gw = bath == 0 ? P.gres[0][0] : P.gres[1][0];
    const float gn = bath == 0 ? P.gres[0][1] : P.gres[1][1];
    const float g = c ? gn : gw;
#pragma unroll
    for (int k = 0; k < 19; ++k) v[k] = wf(k) * g;
    own = T.map[pos];
  } else {
    Near n;
    uint32_t m = 0;
    float r[19];
    near_of<false>(T, pos, px, pp, n);
    own = n.r[0][1];
    pull_one<0>(T.g[parity], (uint32_t)(4 * kLine) + cofs, own, n, m, v);
    stencil_one<1>(T.rho, (uint32_t)(1 - c) * 4u, n, r);
    float S[3] = {0, 0, 0};
#pragma unroll
    for (int k = 1; k < 19; ++k) {
      const float a = wf(k) * r[k];
      if (ex(k)) S[0] += ex(k) > 0 ? a : -a;
      if (ey(k)) S[1] += ey(k) > 0 ? a : -a;
      if (ez(k)) S[2] += ez(k) > 0 ? a : -a;
    }
    const double drd = sum19(v);
    float dr, rho, rho0, rho1, j[3], j0[3], j1[3], A[3], F[3], up[3];
    moments(P, drd, v, dr, rho, j);
    both(rho, rho0, rho1);
#pragma unroll
    for (int a = 0; a < 3; ++a) both(j[a], j0[a], j1[a]);
    adhesion(m, A);
    force(P, c ? P.Gads[1] : P.Gads[0], rho, S, A, F);
    velocity(P, rho0, rho1, j0, j1, up);
    relax(c ? P.tau[1] : P.tau[0], c ? P.itau[1] : P.itau[0], up, F, drd, dr, rho, v);
  }
  gchar *p = (gchar *)T.g[parity ^ 1] + (size_t)(node_bytes(own) + cofs);
#pragma unroll
  for (int k = 0; k < 19; ++k) __builtin_nontemporal_store(v[k], (gfloat *)(p + k * 4 * kLine));
}

// ---- tiled step over the brick numbering ------------------------------------------
// Map (X, Y, Z), which may lie one node beyond the box, to a node index:
// wrapped on periodic axes, -1 beyond a wall.  Coordinates further out (the
// unused halo slots of a ragged tile) also give -1.
__device__ __forceinline__ long long node_of(const Dom &d, int X, int Y, int Z) {
  if (X < -1 || X > d.nx || Y < -1 || Y > d.ny || Z < -1 || Z > d.nz) return -1;
  if (X < 0 || X >= d.nx) {
    if (!(d.per & 1)) return -1;
    X = X < 0 ? X + d.nx : X - d.nx;
  }
  if (Y < 0 || Y >= d.ny) {
    if (!(d.per & 2)) return -1;
    Y = Y < 0 ? Y + d.ny : Y - d.ny;
  }
  if (Z < 0 || Z >= d.nz) {
    if (!(d.per & 4)) return -1;
    Z = Z < 0 ? Z + d.nz : Z - d.nz;
  }
  return (long long)X + (long long)d.nx * ((long long)Y + (long long)d.ny * Z);
}

__device__ __forceinline__ int wrap(int c, int n) { return c < 0 ? c + n : (c >= n ? c - n : c); }

// Pull from bricks.  Addresses are the start of plane Z - 1 (uniform across a
// tile) plus a 32-bit byte offset per lane: the offset of a node is the sum of
// an x part and a y part (brick_x, brick_y); with P the elements of a plane,
// population q of the node itself is at P + y(Y) + x(X) + 32 q, of the source
// node at (1 - ez) P + y(Ys) + x(Xs) + 32 q.  The second component's
// populations follow 19 * 32 later.  Xs and Ys are taken modulo nx and ny:
// across a periodic face that is the wrapped neighbour, across a wall the link
// is cut and the offset unused.
template <int K>
__device__ __forceinline__ void brick_dir(gcchar *b0, gcchar *b1, uint32_t m, uint32_t own,
                                         uint32_t s, float (&v)[2][19]) {
  constexpr int o = opp(K);
  const bool cut = (m >> K) & 1u;
  const uint32_t off = cut ? own + (uint32_t)(o * kBN) : s + (uint32_t)(K * kBN);
  v[0][K] = *(const __attribute__((address_space(1))) float *)(b0 + (size_t)(off * 4u));
  v[1][K] = *(const __attribute__((address_space(1))) float *)(b1 + (size_t)(off * 4u));
}

// source offset of direction K: planes, then the y and x parts of x - e_k
// (index 0: coordinate - 1, 1: itself, 2: + 1)
template <int K>
__device__ __forceinline__ uint32_t src_index(uint32_t P, const uint32_t (&py)[3],
                                              const uint32_t (&px)[3]) {
  return (uint32_t)(1 - ez(K)) * P + py[1 - ey(K)] + px[1 - ex(K)];
}

template <int K>
__device__ __forceinline__ void brick_rec(gcchar *b0, gcchar *b1, uint32_t m, uint32_t own,
                                         uint32_t P, const uint32_t (&py)[3],
                                         const uint32_t (&px)[3], float (&v)[2][19]) {
  brick_dir<K>(b0, b1, m, own, src_index<K>(P, py, px), v);
  if constexpr (K + 1 < 19) brick_rec<K + 1>(b0, b1, m, own, P, py, px, v);
}

__device__ __forceinline__ void brick_pull(const Dom &d, uint32_t m, int X, int Y, int Z,
                                     float (&v)[2][19]) {
  const uint32_t P = (uint32_t)brick_plane(d.nx, d.ny);
  gcchar *b0 = (gcchar *)(d.src + (size_t)P * (size_t)Z);
  gcchar *b1 = b0 + (size_t)(19 * kBN * 4);
  uint32_t px[3], py[3];
  px[0] = brick_x(X == 0 ? d.nx - 1 : X - 1);
  px[1] = brick_x(X);
  px[2] = brick_x(X == d.nx - 1 ? 0 : X + 1);
  py[0] = brick_y(Y == 0 ? d.ny - 1 : Y - 1, d.nx);
  py[1] = brick_y(Y, d.nx);
  py[2] = brick_y(Y == d.ny - 1 ? 0 : Y + 1, d.nx);
  // The offsets do not depend on Z (the base does), so a z-marching loop
  // would otherwise keep all 38 of them live in registers across planes;
  // these opaque moves make them cheap per-plane arithmetic instead.
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    asm volatile("" : "+v"(px[i]));
    asm volatile("" : "+v"(py[i]));
  }
  const uint32_t own = P + py[1] + px[1];
  brick_rec<0>(b0, b1, m, own, P, py, px, v);
}

// mask word of a node as the march sees it: solid beyond a wall
__device__ __forceinline__ uint32_t mask_at(const Dom &d, int X, int Y, int Z) {
  const long long n = node_of(d, X, Y, Z);
  return n < 0 ? kSolid << kTypeShift : ((gcu32 *)d.mask)[n];
}

// the pulls of a fluid node (others keep v undefined)
__device__ __forceinline__ void pull_fluid(const Dom &d, uint32_t m, int X, int Y, int Z,
                                           float (&v)[2][19]) {
  if (m >> kTypeShift == kFluid) brick_pull(d, m, X, Y, wrap(Z, d.nz), v);
}

// Density seen by the interaction sums: zero on solid nodes and beyond walls,
// the imposed value on bath nodes, Eq. 2 on fluid nodes, whose pulled
// populations are v.  ds: the two FP64 sums of a fluid node's shifted
// populations (zero otherwise), for its collision.
__device__ __forceinline__ float2 density_of(const Phys &P, uint32_t m, const float (&v)[2][19],
                                             double (&ds)[2]) {
  ds[0] = ds[1] = 0.0;
  const uint32_t t = m >> kTypeShift;
  if (t == kSolid) return make_float2(0.f, 0.f);
  if (t == kResIn) return make_float2(P.rres[0][0], P.rres[0][1]);
  if (t == kResOut) return make_float2(P.rres[1][0], P.rres[1][1]);
  ds[0] = sum19(v[0]);
  ds[1] = sum19(v[1]);
  return make_float2((float)((acc_t)P.rho_ref + ds[0]), (float)((acc_t)P.rho_ref + ds[1]));
}

// Store the post-collision populations of the node at (X, Y, Z) (the ghost
// planes of z-periodic subdomains are refreshed by k_ghost after the step).
__device__ __forceinline__ void brick_store(const Dom &d, int X, int Y, int Z,
                                           const float (&v)[2][19]) {
  const size_t P = brick_plane(d.nx, d.ny);
  uint32_t own = brick_y(Y, d.nx) + brick_x(X);
  asm volatile("" : "+v"(own));  // per-plane offsets, as in pull()
  gchar *b = (gchar *)(d.dst + P * (size_t)(Z + 1));
#pragma unroll
  for (int c = 0; c < 2; ++c)
#pragma unroll
    for (int k = 0; k < 19; ++k)
      __builtin_nontemporal_store(
          v[c][k], (__attribute__((address_space(1))) float *)(
                       b + (size_t)((own + (uint32_t)((19 * c + k) * kBN)) * 4u)));
}

// A workgroup owns a TX x TY column of nodes and marches it through a
// z-segment, software-pipelined over three planes.  Entering iteration Z, the
// thread holds its own nodes of planes Z and Z+1 in registers, the mask words
// of plane Z+2, and the LDS density ring holds planes Z-1..Z+1.  It
//   1. issues the loads of plane Z+3's mask words and the pulls of plane Z+2
//      for its halo node and its own node,
//   2. collides plane Z with the 18-neighbour density stencil while those are
//      in flight,
//   3. sums the pulls into the ring (plane Z+2), stores plane Z (see kLateNodes)
//      and moves the planes down,
//   4. synchronises the workgroup.
// Every population is read from memory once per step (halo pulls re-read
// neighbour tiles' lines, which are normally still in L2).
//
// Bound: the lines exchanged between L2 and memory, and how much of a plane
// the L2s can hold until the neighbouring tiles have read it.  So the tile is
// as large as the registers allow, 512 threads of up to 256 registers (a CU's
// two wavefronts per SIMD), and no population waits in LDS.  All fluid, us a
// step, against tiles of 256 threads with the middle plane in LDS and three
// workgroups a CU (1.58 times the populations fetched into the L2s, 1.14 now):
// 256^3 1137 / 1325 (304 B a node: 4.5 TB/s), 192^3 554 / 672.  Halo and own
// pulls one after the other: 1238 and 610; mask words through generic addresses
// behind the pulls: 1152 and 570.
template <int TX, int TY>
__device__ __forceinline__ void halo_slot(int h, int &hx, int &hy) {
  constexpr int HR = 2 * (TX + 2);
  if (h < HR) {
    hx = h % (TX + 2) - 1;
    hy = h < TX + 2 ? -1 : TY;
  } else {
    const int u = h - HR;
    hx = u < TY ? -1 : TX;
    hy = u % TY;
  }
}

// Up to this many nodes of the box plane Z is stored behind the sums of plane
// Z+2, whose wait for the pulls would wait for the stores as well; beyond, ahead
// of them: there the step is bound by lines, and tiles that wait more stay
// closer together.  Time behind over ahead: 144^3 0.96, 192^3 0.98, 224^3 0.98,
// 248^3 (14.5 x 2^20) 0.985, 256 x 256 x 224 0.995, 384 x 384 x 96 0.99, 128 x 128
// x 768 0.99, 512 x 512 x 16 and x 32 0.99 and 1.01; at 2^24 by shape, 256^3
// 0.995, 512 x 512 x 64 and 128 x 128 x 1024 1.015; 288^3 1.005, 320^3 1.01, 384^3
// 1.02, 256 x 256 x 512 1.045.  The line lies below 2^24, where nearly every
// shape still gains.
constexpr uint32_t kLateNodes = 15u << 20;
template <int TX, int TY>
__global__ __launch_bounds__(TX *TY) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_step(
    const Throat *__restrict__ throats, const TileRef *__restrict__ tiles, int ntiles,
    int parity) {
  constexpr int NT = TX * TY;
  constexpr int H = 2 * (TX + 2) + 2 * TY;  // halo ring of one plane
  static_assert(NT >= H, "tile too small for its halo");
  __shared__ float2 ring[4][TY + 2][TX + 2];
  // lanes follow the storage bricks: 32 consecutive lanes own one 8 x 4
  // brick, so each population load or store of a wavefront is whole lines
  static_assert(TX % kBX == 0 && TY % kBY == 0, "tiles are whole bricks");
  const int tid = threadIdx.x;
  const int tb = tid / kBN;
  const int tx = (tb % (TX / kBX)) * kBX + tid % kBX;
  const int ty = (tb / (TX / kBX)) * kBY + (tid / kBX) % kBY;
  const TileRef tr = tiles[xcd_item(ntiles)];
  const Throat &T = throats[tr.throat];
  if (!T.active) return;
  Dom d;
  d.src = T.g[parity];
  d.dst = T.g[parity ^ 1];
  d.mask = T.mask;
  d.N = T.N;
  d.nx = T.nx;
  d.ny = T.ny;
  d.nz = T.nz;
  d.per = T.per;
  const Phys P = T.P;
  const int ntx = T.ntx, nty = T.nty, lz = T.lz;
  const bool late = T.N <= kLateNodes;
  const int tix = tr.tile % ntx, tiy = (tr.tile / ntx) % nty, tiz = tr.tile / (ntx * nty);
  const int x0 = tix * TX, y0 = tiy * TY, z0 = tiz * lz;
  const int z1 = min(z0 + lz, d.nz);
  const int x = x0 + tx, y = y0 + ty;
  const bool own = x < d.nx && y < d.ny;
  // the first H threads also pull one halo node each (the halo instructions
  // are then issued by as few wavefronts as possible)
  const bool halo = tid < H;
  int hx = 0, hy = 0;
  if (halo) halo_slot<TX, TY>(tid, hx, hy);
  const int X = wrap(x, d.nx), Y = wrap(y, d.ny);
  const int XH = wrap(x0 + hx, d.nx), YH = wrap(y0 + hy, d.ny);

  float cur[2][19], mid[2][19], nxt[2][19], hv[2][19];
  uint32_t mcur, mmid, mnxt, mh = kSolid << kTypeShift;
  // FP64 population sums of the own node at planes Z, Z+1, Z+2 (for collide)
  double dcur[2], dmid[2], dnxt[2], dh[2];

  // prologue: densities of planes z0-1 .. z0+1, populations of z0 and z0+1
  auto own_plane = [&](int Z, uint32_t &m, float (&v)[2][19], double (&ds)[2]) {
    m = mask_at(d, x, y, Z);
    pull_fluid(d, m, X, Y, Z, v);
    ring[Z & 3][ty + 1][tx + 1] = density_of(P, m, v, ds);
  };
  auto halo_plane = [&](int Z) {
    if (!halo) return;
    mh = mask_at(d, x0 + hx, y0 + hy, Z);
    pull_fluid(d, mh, XH, YH, Z, hv);
    ring[Z & 3][hy + 1][hx + 1] = density_of(P, mh, hv, dh);
  };
  own_plane(z0 - 1, mcur, cur, dcur);
  halo_plane(z0 - 1);
  own_plane(z0, mcur, cur, dcur);
  halo_plane(z0);
  own_plane(z0 + 1, mmid, mid, dmid);
  halo_plane(z0 + 1);
  mnxt = mask_at(d, x, y, min(z0 + 2, z1));
  if (halo) mh = mask_at(d, x0 + hx, y0 + hy, min(z0 + 2, z1));
  __syncthreads();

  for (int Z = z0; Z < z1; ++Z) {
    const bool ahead = Z + 2 <= z1;  // plane Z+2 is needed (density halo or next own)
    const int Z3 = min(Z + 3, z1);
    uint32_t mnxt3 = mask_at(d, x, y, Z3);
    uint32_t mh3 = halo ? mask_at(d, x0 + hx, y0 + hy, Z3) : mh;
    if (ahead) {
      pull_fluid(d, mh, XH, YH, Z + 2, hv);
      pull_fluid(d, mnxt, X, Y, Z + 2, nxt);
    }
    if (own) {
      const uint32_t t = mcur >> kTypeShift;
      if (t == kFluid) {
        float Sw[3] = {0, 0, 0}, Sn[3] = {0, 0, 0};
#pragma unroll
        for (int k = 1; k < 19; ++k) {
          const float2 rn = ring[(Z + ez(k)) & 3][ty + 1 + ey(k)][tx + 1 + ex(k)];
          const float a = wf(k) * rn.x, bb = wf(k) * rn.y;
          if (ex(k)) { Sw[0] += ex(k) > 0 ? a : -a; Sn[0] += ex(k) > 0 ? bb : -bb; }
          if (ey(k)) { Sw[1] += ey(k) > 0 ? a : -a; Sn[1] += ey(k) > 0 ? bb : -bb; }
          if (ez(k)) { Sw[2] += ez(k) > 0 ? a : -a; Sn[2] += ez(k) > 0 ? bb : -bb; }
        }
        collide(P, mcur, Sw, Sn, dcur, cur);
      } else if (t == kResIn || t == kResOut) {
        const int i = t == kResIn ? 0 : 1;
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
          for (int k = 0; k < 19; ++k) cur[c][k] = wf(k) * P.gres[i][c];
      }
      if (!late && t != kSolid) brick_store(d, x, y, Z, cur);
    }
    if (ahead) {
      if (halo) ring[(Z + 2) & 3][hy + 1][hx + 1] = density_of(P, mh, hv, dh);
      ring[(Z + 2) & 3][ty + 1][tx + 1] = density_of(P, mnxt, nxt, dnxt);
    }
    // (the opaque moves put the wait for the mask words ahead of the stores)
    asm volatile("" : "+v"(mnxt3), "+v"(mh3));
    if (late && own && mcur >> kTypeShift != kSolid) brick_store(d, x, y, Z, cur);
#pragma unroll
    for (int c = 0; c < 2; ++c) {
#pragma unroll
      for (int k = 0; k < 19; ++k) {
        cur[c][k] = mid[c][k];
        mid[c][k] = nxt[c][k];
      }
      dcur[c] = dmid[c];
      dmid[c] = dnxt[c];
    }
    mcur = mmid;
    mmid = mnxt;
    mnxt = mnxt3;
    mh = mh3;
    __syncthreads();
  }
}

bool schedule_valid(const Sched &s) {
  if (s.tx == kListTx) return true;  // two passes
  if (s.lz < 1) return false;
  for (int i = 0; i < kNumShapes; ++i)
    if (s.tx == kShapes[i][0] && s.ty == kShapes[i][1]) return true;
  return false;
}

template <int TX, int TY>
static hipError_t step_as(const Throat *th, const TileRef *tiles, int ntiles, int parity,
                          hipStream_t st) {
  if (ntiles <= 0) return hipSuccess;
  hipLaunchKernelGGL((k_step<TX, TY>), dim3((unsigned)ntiles), dim3(TX * TY), 0, st, th, tiles,
                     ntiles, parity);
  return hipGetLastError();
}

// Ghost planes of z-periodic subdomains in bricks: plane 0 of buffer g[which]
// is copied to plane nz, plane nz - 1 to plane -1 (two contiguous runs of one
// padded plane each).  Grid: x over the run, y over the listed subdomains.
__global__ __launch_bounds__(256) void k_ghost(const Throat *__restrict__ throats,
                                               const int *__restrict__ ids, int which) {
  const Throat &T = throats[ids[blockIdx.y]];
  if (!T.active) return;
  float *g = T.g[which];
  const size_t P = brick_plane(T.nx, T.ny);
  for (size_t i = blockIdx.x * (size_t)256 + threadIdx.x; i < P; i += (size_t)gridDim.x * 256) {
    g[P * (size_t)(T.nz + 1) + i] = g[P + i];
    g[i] = g[P * (size_t)T.nz + i];
  }
}

hipError_t launch_ghost(const Throat *th, const int *zper_ids, int n_zper, int which,
                        hipStream_t st) {
  if (n_zper <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_ghost, dim3(1024, (unsigned)n_zper), dim3(256), 0, st, th, zper_ids, which);
  return hipGetLastError();
}

// Both buffers of the populations, in bytes of listed nodes, for which k_node
// stores through the caches: where the next step reads lines just stored from
// the 256 MB memory-side cache, and the L2s (8 x 4 MB) hold too few of them for
// the choice to matter there.  The limits are the measured crossovers; the upper
// one lies above that cache, which still keeps most of the lines.  Step time, cached against non-temporal: up to 10 MB 0.97-0.98, 17-34
// MB 1.01-1.06, 69-80 MB 0.95-0.97, 102 MB 0.95, 133-156 MB 0.92, 212 MB 0.89,
// 242 MB 0.93-0.97, 269 MB 0.91-0.95, from 335 MB on 1.01-1.13.
constexpr long long kKeepLo = 48ll << 20, kKeepHi = 288ll << 20;
static bool keep_stores(long long items) {
  const long long bytes = items * kListNodes * 2 * 38 * 4;
  return bytes >= kKeepLo && bytes <= kKeepHi;
}

// Where the two passes take a lane per component, by items (whole wavefronts)
// and SIMDs: up to half an item per SIMD, where a step is one wavefront's time,
// and again just above one per SIMD, where whole items put two wavefronts on
// some SIMDs and half ones three halves.  Time with a lane per component over a
// lane per node, open boxes of 64 x 32 nodes a plane and four-sphere throats: 16
// to 375 items 0.89-0.94, 480 0.97, 512 0.98, 544 1.02, 1024 1.03; 1056 0.96,
// 1096 0.98, 1152 0.97, 1184 0.99, 1216 1.00, 1248 1.04, 1280 1.01, 1536 1.03.
// Above the next multiples several wavefronts share each SIMD either way and
// nothing is left to gain: 2080 1.02, 2176 1.00, 2304 1.01, 2560 0.99, 3104
// 1.02, 4128 1.11.
constexpr int kSimds = 256 * 4;
static bool split_lanes(int items) {
  return items <= kSimds / 2 || (items > kSimds && items <= kSimds + 3 * kSimds / 16);
}

static hipError_t step_body(const Throat *th, const TileRef *tiles, int ntiles, int tx, int ty,
                            bool wide, int parity, hipStream_t st) {
  if (tx == kListTx) {
    if (ntiles <= 0) return hipSuccess;
    const dim3 grid((unsigned)ntiles), block(kListNodes);
    if (wide) {
      hipLaunchKernelGGL(k_dens<true>, grid, block, 0, st, th, tiles, ntiles, parity);
      hipLaunchKernelGGL((k_node<true, false>), grid, block, 0, st, th, tiles, ntiles, parity);
    } else if (split_lanes(ntiles)) {
      const dim3 halves(2 * (unsigned)ntiles);
      hipLaunchKernelGGL(k_dens_split, halves, block, 0, st, th, tiles, ntiles, parity);
      hipLaunchKernelGGL(k_node_split, halves, block, 0, st, th, tiles, ntiles, parity);
    } else {
      hipLaunchKernelGGL(k_dens<false>, grid, block, 0, st, th, tiles, ntiles, parity);
      if (keep_stores(ntiles))
        hipLaunchKernelGGL((k_node<false, true>), grid, block, 0, st, th, tiles, ntiles, parity);
      else
        hipLaunchKernelGGL((k_node<false, false>), grid, block, 0, st, th, tiles, ntiles, parity);
    }
    return hipGetLastError();
  }
  if (tx == 32) {
    if (ty == 4) return step_as<32, tile_rows(4)>(th, tiles, ntiles, parity, st);
    return step_as<32, tile_rows(8)>(th, tiles, ntiles, parity, st);
  }
  if (tx == 16) {
    if (ty == 4) return step_as<16, tile_rows(4)>(th, tiles, ntiles, parity, st);
    return step_as<16, tile_rows(8)>(th, tiles, ntiles, parity, st);
  }
  if (tx == 8) return step_as<8, tile_rows(8)>(th, tiles, ntiles, parity, st);
  return step_as<64, tile_rows(4)>(th, tiles, ntiles, parity, st);
}

hipError_t launch_step(const Throat *th, const TileRef *tiles, int ntiles, int tx, int ty,
                       bool wide, int parity, hipStream_t st, const int *zper_ids, int n_zper) {
  if (!schedule_valid(Sched{tx, ty, 1})) return hipErrorInvalidValue;
  const hipError_t e = step_body(th, tiles, ntiles, tx, ty, wide, parity, st);
  // (the two passes pull across a periodic face by number)
  if (e != hipSuccess || ntiles <= 0 || n_zper <= 0) return e;
  return launch_ghost(th, zper_ids, n_zper, parity ^ 1, st);
}

void brick_map(const uint8_t *types, int nx, int ny, int nz, std::vector<uint8_t> &live) {
  const int nbx = (nx + kBX - 1) / kBX, nby = (ny + kBY - 1) / kBY;
  live.assign((size_t)nbx * nby * nz, 0);
  for (int z = 0; z < nz; ++z)
    for (int y = 0; y < ny; ++y) {
      const uint8_t *row = types + (size_t)nx * ((size_t)y + (size_t)ny * z);
      uint8_t *b = live.data() + (size_t)nbx * ((size_t)(y / kBY) + (size_t)nby * z);
      for (int x = 0; x < nx; ++x)
        if (row[x] != kSolid) b[x / kBX] = 1;
    }
}

void list_tiles(const uint8_t *live, int nx, int ny, int nz, int tx, int ty, int lz, int throat,
                std::vector<TileRef> &out) {
  const int nbx = (nx + kBX - 1) / kBX, nby = (ny + kBY - 1) / kBY;
  const int bpx = tx / kBX, bpy = ty / kBY;  // patches per tile side
  const int ntx = (nx + tx - 1) / tx, nty = (ny + ty - 1) / ty, ntz = (nz + lz - 1) / lz;
  // liveness of each (x-tile, y-tile) cell of every plane, then of every z-segment
  std::vector<uint8_t> cell((size_t)ntx * nty * nz, 0);
  for (int z = 0; z < nz; ++z)
    for (int by = 0; by < nby; ++by) {
      const uint8_t *b = live + (size_t)nbx * ((size_t)by + (size_t)nby * z);
      uint8_t *c = cell.data() + (size_t)ntx * ((size_t)(by / bpy) + (size_t)nty * z);
      for (int bx = 0; bx < nbx; ++bx)
        if (b[bx]) c[bx / bpx] = 1;
    }
  for (int tz = 0; tz < ntz; ++tz)
    for (int tyi = 0; tyi < nty; ++tyi)
      for (int txi = 0; txi < ntx; ++txi) {
        bool any = false;
        for (int z = tz * lz; z < std::min(nz, (tz + 1) * lz) && !any; ++z)
          any = cell[(size_t)txi + (size_t)ntx * ((size_t)tyi + (size_t)nty * z)] != 0;
        if (any) out.push_back(TileRef{throat, txi + ntx * (tyi + nty * tz)});
      }
}

void list_items(size_t n_live, int throat, std::vector<TileRef> &out) {
  for (size_t c = 0; c * kListNodes < n_live; ++c) out.push_back(TileRef{throat, (int)c});
}

// ---- numbering ---------------------------------------------------------------------
// one wavefront per row
__global__ __launch_bounds__(256) void k_row_counts(const uint8_t *types, int nx, uint32_t rows,
                                                    uint32_t *counts) {
  const uint32_t row = blockIdx.x * 4u + (threadIdx.x >> 6);
  if (row >= rows) return;
  const uint8_t *t = types + (size_t)row * nx;
  uint32_t n = 0;
  for (int x0 = 0; x0 < nx; x0 += 64) {
    const int x = x0 + (int)(threadIdx.x & 63);
    n += (uint32_t)__popcll(__ballot(x < nx && t[x] != kSolid));
  }
  if ((threadIdx.x & 63) == 0) counts[row] = n;
}

hipError_t launch_row_counts(const uint8_t *types, int nx, int ny, int nz, uint32_t *counts,
                             hipStream_t st) {
  const uint32_t rows = (uint32_t)ny * (uint32_t)nz;
  hipLaunchKernelGGL(k_row_counts, dim3((rows + 3) / 4), dim3(256), 0, st, types, nx, rows, counts);
  return hipGetLastError();
}

size_t number_rows(uint32_t *rows, int ny, int nz) {
  size_t n = 0;
  for (int Y = 0; Y < ny; Y += kGroupY)
    for (int z = 0; z < nz; ++z)
      for (int y = Y; y < std::min(Y + kGroupY, ny); ++y) {
        uint32_t &r = rows[(size_t)z * ny + y];
        const uint32_t c = r;
        r = (uint32_t)n;
        n += c;
      }
  return n;
}

// one wavefront per row: the row's nodes take consecutive list places from
// its first one
__global__ __launch_bounds__(256) void k_number(const uint8_t *types, int nx, int ny, int nz,
                                                uint32_t nrows, const uint32_t *rows, int bricks,
                                                uint32_t *map, uint32_t *pos) {
  const uint32_t row = blockIdx.x * 4u + (threadIdx.x >> 6);
  if (row >= nrows) return;
  const uint8_t *t = types + (size_t)row * nx;
  const int y = (int)(row % (uint32_t)ny), z = (int)(row / (uint32_t)ny);
  const int lane = (int)(threadIdx.x & 63);
  uint32_t base = rows[row];
  for (int x0 = 0; x0 < nx; x0 += 64) {
    const int x = x0 + lane;
    const bool live = x < nx && t[x] != kSolid;
    const unsigned long long bal = __ballot(live);
    if (live) {
      const uint32_t i = base + (uint32_t)__popcll(bal & ((1ull << lane) - 1ull));
      const size_t p = map_pos(nx, ny, x, y, z);
      map[p] = bricks ? brick_number(nx, ny, x, y, z) : i;
      pos[i] = (uint32_t)p;
    }
    base += (uint32_t)__popcll(bal);
  }
}

// solid nodes, and the two layers beyond the box
__global__ void k_number_rest(const uint8_t *types, int nx, int ny, int nz, int per,
                              uint32_t *map) {
  const size_t M = map_elems(nx, ny, nz);
  const int n[3] = {nx, ny, nz};
  for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < M;
       i += (size_t)gridDim.x * blockDim.x) {
    int c[3] = {(int)(i % (size_t)(nx + 2 * kPad)) - kPad,
                (int)((i / (size_t)(nx + 2 * kPad)) % (size_t)(ny + 2 * kPad)) - kPad,
                (int)(i / ((size_t)(nx + 2 * kPad) * (size_t)(ny + 2 * kPad))) - kPad};
    bool inside = true, none = false;
    for (int a = 0; a < 3; ++a)
      if (c[a] < 0 || c[a] >= n[a]) {
        inside = false;
        if (!((per >> a) & 1)) none = true;
        c[a] += c[a] < 0 ? n[a] : -n[a];
      }
    if (!none)
      none = types[(size_t)c[0] + (size_t)nx * ((size_t)c[1] + (size_t)ny * c[2])] == kSolid;
    if (none)
      map[i] = kNoNode;
    else if (!inside)
      map[i] = map[map_pos(nx, ny, c[0], c[1], c[2])];
  }
}

static hipError_t number_rest(const uint8_t *types, int nx, int ny, int nz, int per, uint32_t *map,
                              hipStream_t st) {
  const size_t M = map_elems(nx, ny, nz);
  const unsigned grid = (unsigned)std::min<size_t>((M + 255) / 256, 65536);
  hipLaunchKernelGGL(k_number_rest, dim3(grid), dim3(256), 0, st, types, nx, ny, nz, per, map);
  return hipGetLastError();
}

hipError_t launch_number(const uint8_t *types, int nx, int ny, int nz, int per,
                         const uint32_t *rows, bool bricks, uint32_t *map, uint32_t *pos,
                         hipStream_t st) {
  const uint32_t nrows = (uint32_t)ny * (uint32_t)nz;
  hipLaunchKernelGGL(k_number, dim3((nrows + 3) / 4), dim3(256), 0, st, types, nx, ny, nz, nrows,
                     rows, bricks ? 1 : 0, map, pos);
  return number_rest(types, nx, ny, nz, per, map, st);
}

// The compact number of the i-th listed node is i, its brick number follows
// from its coordinates: neither numbering needs the other's map.
__device__ __forceinline__ void coords_of(const Dom &d, uint32_t pos, int &x, int &y, int &z) {
  const uint32_t px = (uint32_t)(d.nx + 2 * kPad), py = (uint32_t)(d.ny + 2 * kPad);
  x = (int)(pos % px) - kPad;
  y = (int)(pos / px % py) - kPad;
  z = (int)(pos / px / py) - kPad;
}

__global__ __launch_bounds__(256) void k_renumber(Dom d, const uint32_t *pos, uint32_t n_live,
                                                  int bricks, uint32_t *map) {
  for (size_t i = blockIdx.x * (size_t)256 + threadIdx.x; i < n_live;
       i += (size_t)gridDim.x * 256) {
    int x, y, z;
    coords_of(d, pos[i], x, y, z);
    map[pos[i]] = bricks ? brick_number(d.nx, d.ny, x, y, z) : (uint32_t)i;
  }
}

hipError_t launch_renumber(const Dom &d, const uint8_t *types, const uint32_t *pos, uint32_t n_live,
                           bool bricks, uint32_t *map, hipStream_t st) {
  if (n_live)
    hipLaunchKernelGGL(k_renumber, dim3(std::min((n_live + 255) / 256, 65536u)), dim3(256), 0, st,
                       d, pos, n_live, bricks ? 1 : 0, map);
  return number_rest(types, d.nx, d.ny, d.nz, d.per, map, st);
}

__global__ __launch_bounds__(256) void k_move(Dom d, const uint32_t *pos, uint32_t n_live,
                                              int bricks, const float *src, float *dst) {
  for (size_t i = blockIdx.x * (size_t)256 + threadIdx.x; i < n_live;
       i += (size_t)gridDim.x * 256) {
    int x, y, z;
    coords_of(d, pos[i], x, y, z);
    const size_t c = node_elem((uint32_t)i), b = node_elem(brick_number(d.nx, d.ny, x, y, z));
    const size_t from = bricks ? c : b, to = bricks ? b : c;
    // the planes -1 and nz of z-periodic bricks repeat the planes nz - 1 and 0
    const size_t turn = brick_plane(d.nx, d.ny) * (size_t)d.nz;
    const bool ghosts = bricks && (d.per & 4);
    for (int q = 0; q < kQ; ++q) {
      const size_t o = (size_t)(q * kLine);
      const float v = src[from + o];
      dst[to + o] = v;
      if (ghosts && z == 0) dst[to + turn + o] = v;
      if (ghosts && z == d.nz - 1) dst[to - turn + o] = v;
    }
  }
}

hipError_t launch_move(const Dom &d, const uint32_t *pos, uint32_t n_live, bool bricks,
                       const float *src, float *dst, hipStream_t st) {
  if (n_live == 0) return hipSuccess;
  hipLaunchKernelGGL(k_move, dim3(std::min((n_live + 255) / 256, 65536u)), dim3(256), 0, st, d, pos,
                     n_live, bricks ? 1 : 0, src, dst);
  return hipGetLastError();
}

// number of every subdomain's probe node, whose map position info[t].probe holds
__global__ void k_probe_numbers(const Throat *throats, int n, RedInfo *info) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t < n) info[t].probe = throats[t].map[info[t].probe];
}

hipError_t launch_probe_numbers(const Throat *throats, int n, RedInfo *info, hipStream_t st) {
  hipLaunchKernelGGL(k_probe_numbers, dim3((unsigned)(n + 255) / 256), dim3(256), 0, st, throats,
                     n, info);
  return hipGetLastError();
}

__global__ void k_links(const uint8_t *types, Dom d, uint32_t *mask) {
  for (size_t n = blockIdx.x * (size_t)blockDim.x + threadIdx.x; n < d.N;
       n += (size_t)gridDim.x * blockDim.x) {
    const int x = (int)(n % d.nx), y = (int)((n / d.nx) % d.ny), z = (int)(n / ((size_t)d.nx * d.ny));
    uint32_t m = 0;
#pragma unroll
    for (int k = 1; k < 19; ++k)
      if (d.map[map_pos(d.nx, d.ny, x - ex(k), y - ey(k), z - ez(k))] == kNoNode) m |= 1u << k;
    mask[n] = m | ((uint32_t)types[n] << kTypeShift);
  }
}

hipError_t launch_links(const uint8_t *types, const Dom &d, uint32_t *mask, hipStream_t st) {
  const unsigned blocks = (unsigned)std::min<size_t>((d.N + 255) / 256, 65536);
  hipLaunchKernelGGL(k_links, dim3(blocks), dim3(256), 0, st, types, d, mask);
  return hipGetLastError();
}

// ---- geometry ----------------------------------------------------------------
// Node classes from spheres and the prism closure (predicates in geom.h).
// Spheres are binned on the host into cubic cells of kVoxCell nodes: a node
// tests only the spheres whose bounding box (widened by one node) meets its
// cell, in increasing sphere order, which classifies every node exactly as
// testing all spheres would.
__global__ void k_voxelize(const double *sph, const VoxBins bins, int prism, int i0, int i1,
                           int i2, int nx, int ny, int nz, int res_z, uint8_t *types) {
  const size_t N = (size_t)nx * ny * nz;
  for (size_t n = blockIdx.x * (size_t)blockDim.x + threadIdx.x; n < N;
       n += (size_t)gridDim.x * blockDim.x) {
    const int x = (int)(n % nx), y = (int)((n / nx) % ny), z = (int)(n / ((size_t)nx * ny));
    const int c = x / kVoxCell + bins.ncx * (y / kVoxCell + bins.ncy * (z / kVoxCell));
    bool solid = false;
    for (int j = bins.start[c]; j < bins.start[c + 1] && !solid; ++j)
      solid = geom::in_sphere(x, y, z, sph + 4 * bins.ids[j]);
    if (!solid && prism) solid = !geom::in_prism(sph + 4 * i0, sph + 4 * i1, sph + 4 * i2, x, y);
    uint8_t t = kFluid;
    if (solid) t = kSolid;
    else if (res_z && z == 0) t = kResIn;
    else if (res_z && z == nz - 1) t = kResOut;
    types[n] = t;
  }
}

void bin_spheres(const double *sph, int ns, int nx, int ny, int nz, std::vector<int> &start,
                 std::vector<int> &ids, int &ncx, int &ncy, int &ncz) {
  ncx = (nx + kVoxCell - 1) / kVoxCell;
  ncy = (ny + kVoxCell - 1) / kVoxCell;
  ncz = (nz + kVoxCell - 1) / kVoxCell;
  const int nn[3] = {nx, ny, nz};
  std::vector<std::vector<int>> cell((size_t)ncx * ncy * ncz);
  for (int i = 0; i < ns; ++i) {
    int lo[3], hi[3];
    bool empty = false;
    for (int a = 0; a < 3; ++a) {
      const double l = std::floor(sph[4 * i + a] - sph[4 * i + 3]) - 1.0;
      const double h = std::ceil(sph[4 * i + a] + sph[4 * i + 3]) + 1.0;
      if (h < 0.0 || l > nn[a] - 1.0) empty = true;
      lo[a] = (int)std::max(0.0, l) / kVoxCell;
      hi[a] = (int)std::min((double)(nn[a] - 1), h) / kVoxCell;
    }
    if (empty) continue;
    for (int cz = lo[2]; cz <= hi[2]; ++cz)
      for (int cy = lo[1]; cy <= hi[1]; ++cy)
        for (int cx = lo[0]; cx <= hi[0]; ++cx)
          cell[(size_t)cx + (size_t)ncx * ((size_t)cy + (size_t)ncy * cz)].push_back(i);
  }
  start.assign(cell.size() + 1, 0);
  ids.clear();
  for (size_t c = 0; c < cell.size(); ++c) {
    start[c] = (int)ids.size();
    ids.insert(ids.end(), cell[c].begin(), cell[c].end());
  }
  start[cell.size()] = (int)ids.size();
}

hipError_t launch_voxelize(const double *spheres, const VoxBins &bins, int prism, const int *ids,
                           int nx, int ny, int nz, int res_z, uint8_t *types, hipStream_t st) {
  const size_t N = (size_t)nx * ny * nz;
  const unsigned blocks = (unsigned)std::min<size_t>((N + 255) / 256, 65536);
  hipLaunchKernelGGL(k_voxelize, dim3(blocks), dim3(256), 0, st, spheres, bins, prism, ids[0],
                     ids[1], ids[2], nx, ny, nz, res_z, types);
  return hipGetLastError();
}

// ---- initial state ------------------------------------------------------------
// Post-collision values of a virtual step -1 chosen so that the first pull
// yields f(x,0) = f_eq(rho(x,0), u = 0) = w_k rho(x,0) on every fluid node:
// slot k of node y holds w_k rho(y + e_k), or w_k rho(y) when y + e_k is
// solid or beyond a wall (that slot is then only read back by y's own
// bounce-back).
__device__ __forceinline__ double rho0_of(const Dom &d, const double *rho_init, double maj,
                                          double mnr, int z_front, const double *rres, int x,
                                          int y, int z, int c) {
  if (d.res && z == 0) return rres[0 * 2 + c];
  if (d.res && z == d.nz - 1) return rres[1 * 2 + c];
  if (rho_init)
    return rho_init[(size_t)c * d.N + (size_t)x + (size_t)d.nx * ((size_t)y + (size_t)d.ny * z)];
  const bool nw = z <= z_front;
  return (c == 1) == nw ? maj : mnr;
}

__global__ void k_init(Dom d, double rho_ref, const double *rho_init, double maj, double mnr,
                       int z_front, const double *rres, float *g, unsigned long long *bad) {
  for (size_t n = blockIdx.x * (size_t)blockDim.x + threadIdx.x; n < d.N;
       n += (size_t)gridDim.x * blockDim.x) {
    const int x = (int)(n % d.nx), y = (int)((n / d.nx) % d.ny), z = (int)(n / ((size_t)d.nx * d.ny));
    const uint32_t i = d.map[map_pos(d.nx, d.ny, x, y, z)];
    if (i == kNoNode) continue;
    if (rho_init && class_at(d, x, y, z) == kFluid)
      for (int c = 0; c < 2; ++c) {
        const double r = rho_init[c * d.N + n];
        if (!(isfinite(r) && r > 0)) atomicMin(bad, (unsigned long long)(c * d.N + n));
      }
    float *slot = g + node_elem(i);
#pragma unroll
    for (int k = 0; k < 19; ++k) {
      int X = x + ex(k), Y = y + ey(k), Z = z + ez(k);
      const bool none = d.map[map_pos(d.nx, d.ny, X, Y, Z)] == kNoNode;
      X = none ? x : wrap(X, d.nx);
      Y = none ? y : wrap(Y, d.ny);
      Z = none ? z : wrap(Z, d.nz);
      for (int c = 0; c < 2; ++c) {
        const double r = rho0_of(d, rho_init, maj, mnr, z_front, rres, X, Y, Z, c);
        slot[(c * 19 + k) * kLine] = (float)(wd(k) * (r - rho_ref));
      }
    }
  }
}

hipError_t launch_init(const Dom &d, const Phys &P, const double *rho_init, double maj, double mnr,
                       int z_front, const double *rres_d, float *g, unsigned long long *bad,
                       hipStream_t st) {
  const unsigned blocks = (unsigned)std::min<size_t>((d.N + 255) / 256, 65536);
  hipLaunchKernelGGL(k_init, dim3(blocks), dim3(256), 0, st, d, (double)P.rho_ref, rho_init, maj,
                     mnr, z_front, rres_d, g, bad);
  return hipGetLastError();
}

// ---- checkpoint-file layout -----------------------------------------------------
// element `o` of the file layout: population q of box node (x, y, z); false
// for padding, unused ghost planes and solid nodes
__device__ __forceinline__ bool file_node(const Dom &d, size_t o, bool ghosts, uint32_t &i,
                                          int &q) {
  const size_t P = brick_plane(d.nx, d.ny);
  int z = (int)(o / P) - 1;
  const uint32_t r = (uint32_t)(o % P);
  const uint32_t brick = r / (uint32_t)(kQ * kBX * kBY), w = r % (uint32_t)(kQ * kBX * kBY);
  const uint32_t nbx = (uint32_t)(pad_x(d.nx) / kBX), l = w % (uint32_t)(kBX * kBY);
  q = (int)(w / (uint32_t)(kBX * kBY));
  const int x = (int)((brick % nbx) * kBX + l % kBX), y = (int)((brick / nbx) * kBY + l / kBX);
  if (x >= d.nx || y >= d.ny) return false;
  if (z < 0 || z >= d.nz) {
    if (!ghosts || !(d.per & 4)) return false;
    z = wrap(z, d.nz);
  }
  i = d.map[map_pos(d.nx, d.ny, x, y, z)];
  return i != kNoNode;
}

__global__ void k_to_file(Dom d, const float *g, size_t first, size_t count, float *out) {
  for (size_t o = blockIdx.x * (size_t)blockDim.x + threadIdx.x; o < count;
       o += (size_t)gridDim.x * blockDim.x) {
    uint32_t i;
    int q;
    out[o] = file_node(d, first + o, true, i, q) ? g[node_elem(i) + (size_t)(q * kLine)] : 0.f;
  }
}

__global__ void k_from_file(Dom d, const float *in, size_t first, size_t count, float *g) {
  for (size_t o = blockIdx.x * (size_t)blockDim.x + threadIdx.x; o < count;
       o += (size_t)gridDim.x * blockDim.x) {
    uint32_t i;
    int q;
    if (file_node(d, first + o, false, i, q)) g[node_elem(i) + (size_t)(q * kLine)] = in[o];
  }
}

hipError_t launch_to_file(const Dom &d, const float *g, size_t first, size_t count, float *out,
                          hipStream_t st) {
  const unsigned blocks = (unsigned)std::min<size_t>((count + 255) / 256, 65536);
  hipLaunchKernelGGL(k_to_file, dim3(blocks), dim3(256), 0, st, d, g, first, count, out);
  return hipGetLastError();
}

hipError_t launch_from_file(const Dom &d, const float *in, size_t first, size_t count, float *g,
                            hipStream_t st) {
  const unsigned blocks = (unsigned)std::min<size_t>((count + 255) / 256, 65536);
  hipLaunchKernelGGL(k_from_file, dim3(blocks), dim3(256), 0, st, d, in, first, count, g);
  return hipGetLastError();
}

// ---- read-back: pre-collision populations and densities in FP64 ------------
__global__ void k_export(Dom d, Phys P, const double *rres, double *f) {
  for (size_t n = blockIdx.x * (size_t)blockDim.x + threadIdx.x; n < d.N;
       n += (size_t)gridDim.x * blockDim.x) {
    const int x = (int)(n % d.nx), y = (int)((n / d.nx) % d.ny), z = (int)(n / ((size_t)d.nx * d.ny));
    const uint32_t t = class_at(d, x, y, z);
    float v[2][19];
    if (t == kFluid) pull_at(d, x, y, z, v);
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int k = 0; k < 19; ++k) {
        double o = 0.0;
        if (t == kFluid) o = wd(k) * (double)P.rho_ref + (double)v[c][k];
        else if (t == kResIn) o = wd(k) * rres[0 * 2 + c];
        else if (t == kResOut) o = wd(k) * rres[1 * 2 + c];
        f[(size_t)(c * 19 + k) * d.N + n] = o;
      }
  }
}

hipError_t launch_export(const Dom &d, const Phys &P, const double *rres_d, double *f,
                         hipStream_t st) {
  const unsigned blocks = (unsigned)std::min<size_t>((d.N + 255) / 256, 65536);
  hipLaunchKernelGGL(k_export, dim3(blocks), dim3(256), 0, st, d, P, rres_d, f);
  return hipGetLastError();
}

__global__ void k_density(Dom d, Phys P, const double *rres, double *rho) {
  for (size_t n = blockIdx.x * (size_t)blockDim.x + threadIdx.x; n < d.N;
       n += (size_t)gridDim.x * blockDim.x) {
    const int x = (int)(n % d.nx), y = (int)((n / d.nx) % d.ny), z = (int)(n / ((size_t)d.nx * d.ny));
    const uint32_t t = class_at(d, x, y, z);
    double r0 = 0.0, r1 = 0.0;
    if (t == kFluid) {
      float v[2][19];
      pull_at(d, x, y, z, v);
      r0 = (double)(float)((acc_t)P.rho_ref + sum19(v[0]));
      r1 = (double)(float)((acc_t)P.rho_ref + sum19(v[1]));
    } else if (t == kResIn) {
      r0 = rres[0];
      r1 = rres[1];
    } else if (t == kResOut) {
      r0 = rres[2];
      r1 = rres[3];
    }
    rho[n] = r0;
    rho[d.N + n] = r1;
  }
}

hipError_t launch_density(const Dom &d, const Phys &P, const double *rres_d, double *rho,
                          hipStream_t st) {
  const unsigned blocks = (unsigned)std::min<size_t>((d.N + 255) / 256, 65536);
  hipLaunchKernelGGL(k_density, dim3(blocks), dim3(256), 0, st, d, P, rres_d, rho);
  return hipGetLastError();
}

// ---- fixed staging array of the allocation-free density read-back ---------
// A file-scope device array, one copy per device for the life of the process.
// Host code never uses its name as an address (on the host the name is only a
// stand-in for the symbol): the device address of the current device's copy
// comes from hipGetSymbolAddress, taken once per device and kept.
static __device__ __align__(256) __attribute__((used)) double scratch[kScratchDoubles];

hipError_t scratch_address(double **out) {
  constexpr int kMaxDevices = 64;
  static std::mutex mu;
  static double *addr[kMaxDevices] = {};
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (!addr[dev]) {
    void *p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    addr[dev] = (double *)p;
  }
  *out = addr[dev];
  return hipSuccess;
}

// ---- FP64 reductions ------------------------------------------------------
// Two passes with a fixed summation order (a chunk's nodes strided over one
// workgroup, then an LDS tree; then a subdomain's chunks likewise), so results
// are bitwise reproducible and identical whether a subdomain is reduced alone or
// inside a batch.
constexpr int kRedThreads = 256;
constexpr int kRedVals = 3;

__device__ __forceinline__ void block_sum(double (&v)[kRedVals], double (*sh)[kRedThreads]) {
  const int t = threadIdx.x;
#pragma unroll
  for (int i = 0; i < kRedVals; ++i) sh[i][t] = v[i];
  __syncthreads();
  for (int s = kRedThreads / 2; s > 0; s >>= 1) {
    if (t < s)
#pragma unroll
      for (int i = 0; i < kRedVals; ++i) sh[i][t] += sh[i][t + s];
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < kRedVals; ++i) v[i] = sh[i][0];
}

__global__ __launch_bounds__(kRedThreads) void k_reduce_chunks(const Throat *__restrict__ th,
                                                               const RedChunk *__restrict__ chunks,
                                                               int nchunks,
                                                               const RedInfo *__restrict__ info,
                                                               int parity, double *partials,
                                                               double *probe_out) {
  __shared__ double sh[kRedVals][kRedThreads];
  const int item = xcd_item(nchunks);
  const RedChunk ch = chunks[item];
  const Throat &T = th[ch.throat];
  const uint32_t px = (uint32_t)(T.nx + 2 * kPad);
  const size_t pp = (size_t)px * (size_t)(T.ny + 2 * kPad);
  const float rho_ref = T.P.rho_ref;
  const RedInfo ri = info[ch.throat];
  double acc[kRedVals] = {0.0, 0.0, 0.0};
  for (uint32_t i = ch.first + threadIdx.x; i < ch.end; i += kRedThreads) {
    const uint32_t pos = T.pos[i];
    if (bath_of(T, pos, pp) >= 0) continue;
    Near n;
    uint32_t m;
    float v[2][19];
    near_of<true>(T, pos, px, pp, n);
    pull<true>(T.g[parity], n, m, v);
    const double a = (double)(float)((acc_t)rho_ref + sum19(v[0]));
    const double b = (double)(float)((acc_t)rho_ref + sum19(v[1]));
    acc[0] += a;
    acc[1] += b;
    acc[2] += ((a - b) / (a + b) + ri.phib) / (2.0 * ri.phib);
    if ((long long)n.r[0][1] == ri.probe) {
      probe_out[2 * ch.throat] = a;
      probe_out[2 * ch.throat + 1] = b;
    }
  }
  block_sum(acc, sh);
  if (threadIdx.x == 0)
    for (int i = 0; i < kRedVals; ++i) partials[(size_t)item * kRedVals + i] = acc[i];
}

__global__ __launch_bounds__(kRedThreads) void k_reduce_throats(const int *first, const int *count,
                                                                const double *partials,
                                                                double *sums) {
  __shared__ double sh[kRedVals][kRedThreads];
  const int t = blockIdx.x;
  double acc[kRedVals] = {0.0, 0.0, 0.0};
  for (int c = threadIdx.x; c < count[t]; c += kRedThreads)
    for (int i = 0; i < kRedVals; ++i) acc[i] += partials[(size_t)(first[t] + c) * kRedVals + i];
  block_sum(acc, sh);
  if (threadIdx.x == 0)
    for (int i = 0; i < kRedVals; ++i) sums[(size_t)t * kRedVals + i] = acc[i];
}

// A node per thread up to 2^18 nodes, where a chunk's time is its chain of
// loads (a check of 1 k to 94 k nodes takes 22-24 us, with four nodes a thread
// and a copy of the sums to the host 29), four beyond, where there are chunks
// enough to fill the chip and their partial sums are one workgroup's work.
void red_chunks(size_t n_live, int throat, std::vector<RedChunk> &out) {
  const size_t step = n_live <= ((size_t)1 << 18) ? kRedThreads : 4 * kRedThreads;
  for (size_t f = 0; f < n_live; f += step)
    out.push_back(RedChunk{throat, (uint32_t)f, (uint32_t)std::min(f + step, n_live)});
}

hipError_t launch_reduce_chunks(const Throat *th, const RedChunk *chunks, int nchunks,
                                const RedInfo *info, int parity, double *partials,
                                double *probe_out, hipStream_t st) {
  if (nchunks <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_reduce_chunks, dim3(nchunks), dim3(kRedThreads), 0, st, th, chunks,
                     nchunks, info, parity, partials, probe_out);
  return hipGetLastError();
}

hipError_t launch_reduce_throats(const int *first, const int *count, int n, const double *partials,
                                 double *sums, hipStream_t st) {
  hipLaunchKernelGGL(k_reduce_throats, dim3((unsigned)n), dim3(kRedThreads), 0, st, first, count,
                     partials, sums);
  return hipGetLastError();
}

void copy_chunks(int throat, size_t elems, std::vector<Chunk> &out) {
  const size_t n = elems / 4;
  for (size_t s = 0; s < n; s += kCopyChunk)
    out.push_back(Chunk{throat, (uint32_t)std::min<size_t>(kCopyChunk, n - s), s});
}

// ---- device-side drainage ramp (Sec. 2.2.2) ---------------------------------
// The same decisions as the host ramp of a single subdomain, taken for every
// subdomain of a batch between chunks of steps, so that the whole ramp runs
// as graph replays without host decisions per subdomain or per step.
__device__ __forceinline__ void set_inlet(Throat &T, const RampDev &R, double pc) {
  const double rin = R.rho_out + pc / R.dpc_drho;
  T.P.rres[0][1] = (float)rin;
  T.P.gres[0][1] = (float)(rin - R.rho_ref);
}

__global__ void k_ramp_begin(Throat *th, RampDev *rd, const double *pc, RampCfg cfg,
                             const double *sums, int n) {
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= n) return;
  RampDev R = rd[t];
  const double S = R.n_fluid ? sums[3 * t + 2] / (double)R.n_fluid : 0.0;
  R.phase = kPhaseRamp;
  R.point = 0;
  R.invaded_at = -1;
  R.n_bisect = 0;
  R.warn = 0;
  R.failed = 0;
  R.steps_pt = 0;
  R.total_steps = 0;
  R.S_old = S;
  R.S_stable = S;
  R.stable_pc = 0.0;
  R.req = kSaveStable;
  set_inlet(th[t], R, pc[(size_t)t * cfg.n_pc]);
  th[t].active = 1;
  rd[t] = R;
}

__device__ __forceinline__ void ramp_next_point(Throat &T, RampDev &R, const double *pcs,
                                                const RampCfg &cfg, double S_now) {
  R.point += 1;
  if (R.point >= cfg.n_pc) {
    R.phase = kPhaseDone;
    T.active = 0;
    return;
  }
  set_inlet(T, R, pcs[R.point]);
  R.S_old = S_now;
  R.steps_pt = 0;
}

__device__ __forceinline__ void ramp_trial(Throat &T, RampDev &R) {
  R.mid = 0.5 * (R.lo + R.hi);
  R.req |= kRestoreStable;
  set_inlet(T, R, R.mid);
  R.S_old = R.S_stable;
  R.steps_pt = 0;
}

// a subdomain whose state became non-finite: it stops, and the ramp points
// from `from` on are marked non-finite (none of them gets a result)
__device__ __forceinline__ void ramp_fail(Throat &T, RampDev &R, int *status, int from,
                                          int n_pc) {
  R.failed = 1;
  R.phase = kPhaseDone;
  T.active = 0;
  for (int j = from; j < n_pc; ++j) status[j] = 2;  // LBM_PT_NONFINITE
}

__global__ __launch_bounds__(256) void k_ramp_advance(Throat *th, RampDev *rd, const double *pc,
                                                      RampCfg cfg, const double *sums,
                                                      const double *probe, double *S_out,
                                                      long long *steps_out, int *status_out,
                                                      int n, int *n_active_out) {
  __shared__ int cnt[256];
  int active = 0;
  for (int t = threadIdx.x; t < n; t += blockDim.x) {
    RampDev R = rd[t];
    if (R.phase == kPhaseDone) continue;
    Throat &T = th[t];
    const double *pcs = pc + (size_t)t * cfg.n_pc;
    R.req = 0;  // the previous requests have been carried out
    const double S = R.n_fluid ? sums[3 * t + 2] / (double)R.n_fluid : 0.0;
    const bool inv = probe[2 * t + 1] > probe[2 * t];
    R.steps_pt += cfg.every;
    R.total_steps += cfg.every;
    const bool nonfin = !isfinite(S);
    const bool conv = fabs(S - R.S_old) < cfg.tol;
    if (!nonfin && !conv && R.steps_pt < cfg.cap) {
      R.S_old = S;
      rd[t] = R;
      ++active;
      continue;
    }
    const int st = nonfin ? 2 : (conv ? 0 : 1);
    if (R.phase == kPhaseRamp) {
      const int i = R.point;
      S_out[(size_t)t * cfg.n_pc + i] = S;
      steps_out[(size_t)t * cfg.n_pc + i] = R.steps_pt;
      status_out[(size_t)t * cfg.n_pc + i] = st;
      R.warn |= st == 1;
      if (nonfin) {
        ramp_fail(T, R, status_out + (size_t)t * cfg.n_pc, i + 1, cfg.n_pc);
      } else if (!inv) {
        R.req |= kSaveStable;
        R.S_stable = S;
        R.stable_pc = pcs[i];
        ramp_next_point(T, R, pcs, cfg, S);
      } else if (R.invaded_at >= 0) {
        ramp_next_point(T, R, pcs, cfg, S);
      } else {
        R.invaded_at = i;
        R.lo = i == 0 ? 0.0 : R.stable_pc;
        R.hi = pcs[i];
        if ((R.hi - R.lo) / R.hi > cfg.rel) {
          R.req |= kSaveMain;
          R.S_main = S;
          R.rho_in_main = pcs[i];
          R.phase = kPhaseBisect;
          ramp_trial(T, R);
        } else {
          ramp_next_point(T, R, pcs, cfg, S);
        }
      }
    } else {  // bisection run finished
      R.n_bisect += 1;
      if (nonfin) {
        // the ramp point being bisected keeps its status; the points after
        // it are never reached
        ramp_fail(T, R, status_out + (size_t)t * cfg.n_pc, R.point + 1, cfg.n_pc);
      } else {
        if (inv) {
          R.hi = R.mid;
        } else {
          R.lo = R.mid;
          R.req |= kSaveStable;
          R.S_stable = S;
        }
        const bool wide = (R.hi - R.lo) / R.hi > cfg.rel;
        if (wide && R.n_bisect < kMaxBisect) {
          ramp_trial(T, R);
        } else {
          R.warn |= wide;
          R.req |= kRestoreMain;
          R.phase = kPhaseRamp;
          ramp_next_point(T, R, pcs, cfg, R.S_main);
        }
      }
    }
    if (R.phase != kPhaseDone) ++active;
    rd[t] = R;
  }
  cnt[threadIdx.x] = active;
  __syncthreads();
  for (int s = blockDim.x / 2; s > 0; s >>= 1) {
    if (threadIdx.x < s) cnt[threadIdx.x] += cnt[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) n_active_out[0] = cnt[0];
}

typedef float v4f __attribute__((ext_vector_type(4)));

__global__ __launch_bounds__(256) void k_copy_requests(const Throat *__restrict__ th,
                                                       const RampDev *__restrict__ rd,
                                                       const Ckpt *__restrict__ ck,
                                                       const Chunk *__restrict__ chunks,
                                                       int parity) {
  const Chunk c = chunks[blockIdx.x];
  const int req = rd[c.throat].req;
  if (!req) return;
  v4f *g = (v4f *)th[c.throat].g[parity] + c.start;
  v4f *sa = (v4f *)ck[c.throat].stable + c.start, *ma = (v4f *)ck[c.throat].main + c.start;
  for (uint32_t o = threadIdx.x; o < c.count; o += blockDim.x) {
    const v4f v = g[o];
    if (req & kSaveStable) sa[o] = v;
    if (req & kSaveMain) ma[o] = v;
    if (req & kRestoreStable) g[o] = sa[o];
    if (req & kRestoreMain) g[o] = ma[o];
  }
}

hipError_t launch_ramp_begin(Throat *th, RampDev *rd, const double *pc, const RampCfg &cfg,
                             const double *sums, int n, hipStream_t st) {
  hipLaunchKernelGGL(k_ramp_begin, dim3((n + 255) / 256), dim3(256), 0, st, th, rd, pc, cfg, sums,
                     n);
  return hipGetLastError();
}

hipError_t launch_ramp_advance(Throat *th, RampDev *rd, const double *pc, const RampCfg &cfg,
                               const double *sums, const double *probe, double *S_out,
                               long long *steps_out, int *status_out, int n, int *n_active_out,
                               hipStream_t st) {
  hipLaunchKernelGGL(k_ramp_advance, dim3(1), dim3(256), 0, st, th, rd, pc, cfg, sums, probe,
                     S_out, steps_out, status_out, n, n_active_out);
  return hipGetLastError();
}

hipError_t launch_copy_requests(const Throat *th, const RampDev *rd, const Ckpt *ck,
                                const Chunk *chunks, int nchunks, int parity, hipStream_t st) {
  if (nchunks <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_copy_requests, dim3(nchunks), dim3(256), 0, st, th, rd, ck, chunks, parity);
  return hipGetLastError();
}

// ---- stream-copy probe: achievable HBM bandwidth on this device ----------
// one 16-byte element per thread, plain loads and stores (the fastest copy
// form measured on this device)
__global__ __launch_bounds__(256) void k_copy(const v4f *__restrict__ a, v4f *__restrict__ b,
                                              size_t n4) {
  const size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
  if (i < n4) b[i] = a[i];
}

hipError_t launch_copy(const float *a, float *b, size_t n_floats, hipStream_t st) {
  const size_t n4 = n_floats / 4;
  const size_t blocks = (n4 + 255) / 256;
  if (blocks > 0x7fffffff) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_copy, dim3((unsigned)blocks), dim3(256), 0, st, (const v4f *)a, (v4f *)b, n4);
  return hipGetLastError();
}

}  // namespace sc
