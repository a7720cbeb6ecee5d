// lbm_abi.cpp -- host side of the C interface declared in lbm_abi.h:
// argument validation, device memory, the step/reduction launches and the
// drainage ramp with bisection (Montella et al., Sec. 2.2.2).
#include "lbm_abi.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <climits>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <string>
#include <type_traits>
#include <vector>

#include "lbm_handle.h"
#include "sc_internal.h"

namespace {
thread_local std::string g_err;
std::atomic<unsigned long long> g_budget{0};  // bytes; 0 = no budget
}  // namespace

namespace lbmh {
void set_err(const char *fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  g_err = buf;
}

size_t subdomain_bytes(int nx, int ny, int nz, bool checkpoints) {
  // an upper bound: solid nodes hold no populations
  const size_t pop = sizeof(float) * sc::brick_elems(nx, ny, nz);
  const size_t N = (size_t)nx * ny * nz;
  return (checkpoints ? 4 : 2) * pop + 25 * N + ((size_t)1 << 20);
}

int check_budget(size_t need, const char *what) {
  const unsigned long long b = g_budget.load();
  if (b && need > b) {
    set_err("%s needs %zu bytes of device memory, over the budget of %llu bytes", what, need, b);
    return LBM_ENOMEM;
  }
  return LBM_OK;
}
}  // namespace lbmh

namespace {
using lbmh::set_err;

#define HIPCHK(call)                                                          \
  do {                                                                        \
    hipError_t e_ = (call);                                                   \
    if (e_ != hipSuccess) {                                                   \
      set_err("%s failed: %s", #call, hipGetErrorString(e_));                 \
      return LBM_EHIP;                                                        \
    }                                                                         \
  } while (0)

#define TRY(call)                                                             \
  do {                                                                        \
    int r_ = (call);                                                          \
    if (r_ < 0) return r_;                                                    \
  } while (0)

constexpr double kCs2 = 1.0 / 3.0;

bool finite_pos(double v) { return std::isfinite(v) && v > 0; }

}  // namespace

namespace {

void fill_phys(lbm_throat *h) {
  sc::Phys &P = h->P;
  for (int c = 0; c < 2; ++c) {
    P.tau[c] = (float)h->tau[c];
    P.itau[c] = (float)(1.0 / h->tau[c]);
    P.Gads[c] = (float)h->Gads[c];
  }
  P.G = (float)h->G;
  // populations are stored relative to w_k rho_minor: the minority phase,
  // where populations are smallest, is then held with the most absolute
  // precision
  const double ref = h->rho_minor;
  P.rho_ref = (float)ref;
  const double rr[2][2] = {{h->rho_minor, h->rho_in}, {h->rho_out, h->rho_minor}};
  for (int i = 0; i < 2; ++i)
    for (int c = 0; c < 2; ++c) {
      P.rres[i][c] = (float)rr[i][c];
      P.gres[i][c] = (float)(rr[i][c] - ref);
    }
}

// Tiles of 32 x 16 nodes (64 x 8 measured 1 % behind) in the length of
// z-segment that leaves the fewest planes to march: a CU holds one workgroup,
// so a launch is ceil(workgroups / 256) rounds of a segment and about eight
// planes' time to fill the pipeline.  us a step: 256^3 segments of 16, 32, 64,
// 128 planes 1274, 1216, 1185, 1150; 192^3 of 16, 32, 64, 128 617, 589, 567,
// 931 (144 workgroups, one of two segments short).
constexpr int kTileTx = 32, kTileTy = 8;
long long tile_columns(int nx, int ny) {
  const int rows = sc::tile_rows(kTileTy);
  return (long long)((nx + kTileTx - 1) / kTileTx) * ((ny + rows - 1) / rows);
}
sc::Sched default_schedule(int nx, int ny, int nz) {
  return sc::Sched{kTileTx, kTileTy, lbmh::tile_length({{tile_columns(nx, ny), nz}})};
}

// A subdomain starts in bricks, stepped in tiles, from this share of non-solid
// nodes among the lanes of its default tiles (32 x 16 nodes a plane) and
// kTileNodes nodes padded to bricks on; else in the two passes.  Time of the tiles
// over that of the two passes, all fluid or with cubic arrays of spheres: by
// size at full tiles 96^3 1.24, 112^3 1.18, 128^3 0.86, 160^3 0.80, 256^3 0.75;
// by share, 2 to 3 M nodes 0.90 0.90, 0.80 0.95-1.00, 0.76 1.02, 0.72 1.05-1.09,
// 0.65 1.16; 8 to 27 M 0.86 0.82-0.93, 0.78 0.96-1.02, 0.74 0.94, 0.69 0.99-1.05;
// thin boxes 40 x 40 x 1400 (0.52) 1.24, 33 x 65 x 1000 (0.42) 1.43, 8 x 8 x
// 33000 (0.13) 2.2.
constexpr double kTileFill = 0.75;

// the descriptor: buffers, sizes, tile grid, parameters
void fill_desc(lbm_throat *h) {
  sc::Throat &T = h->desc;
  T.g[0] = h->g[0];
  T.g[1] = h->g[1];
  T.map = h->map_d;
  T.pos = h->pos_d;
  T.rho = h->rho_d;
  T.n_live = (uint32_t)h->n_live;
  T.nx = h->nx;
  T.ny = h->ny;
  T.nz = h->nz;
  T.res = h->bc[2] == LBM_BC_RESERVOIR;
  T.active = 1;
  T.P = h->P;
  T.mask = h->mask_d;
  T.N = (uint32_t)h->N;
  T.per = h->per;
  const sc::Sched s = h->sched;
  const bool tiled = s.tx != sc::kListTx;
  T.ntx = tiled ? (h->nx + s.tx - 1) / s.tx : 0;
  const int rows = sc::tile_rows(s.ty);
  T.nty = tiled ? (h->ny + rows - 1) / rows : 0;
  T.lz = s.lz;
}

// refresh the device descriptor
int sync_desc(lbm_throat *h) {
  fill_desc(h);
  HIPCHK(hipMemcpyAsync(h->desc_d, &h->desc, sizeof(sc::Throat), hipMemcpyHostToDevice,
                        h->stream));
  return LBM_OK;
}

int upload_rres(lbm_throat *h) {
  const double rr[4] = {h->rho_minor, h->rho_in, h->rho_out, h->rho_minor};
  HIPCHK(hipMemcpyAsync(h->rres_d, rr, sizeof rr, hipMemcpyHostToDevice, h->stream));
  return LBM_OK;
}

sc::Dom dom(const lbm_throat *h, const float *src, float *dst) {
  sc::Dom d;
  d.src = src;
  d.dst = dst;
  d.map = h->map_d;
  d.mask = h->mask_d;
  d.N = h->N;
  d.nx = h->nx;
  d.ny = h->ny;
  d.nz = h->nz;
  d.per = h->per;
  d.res = h->bc[2] == LBM_BC_RESERVOIR;
  return d;
}

void fill_handle(const lbm_params *p, lbm_throat *h) {
  h->nx = p->nx;
  h->ny = p->ny;
  h->nz = p->nz;
  h->N = (size_t)p->nx * p->ny * p->nz;
  for (int a = 0; a < 3; ++a) h->bc[a] = p->bc[a];
  h->per = (p->bc[0] == LBM_BC_PERIODIC ? 1 : 0) | (p->bc[1] == LBM_BC_PERIODIC ? 2 : 0) |
           (p->bc[2] == LBM_BC_PERIODIC ? 4 : 0);
  for (int c = 0; c < 2; ++c) {
    h->tau[c] = p->tau[c];
    h->Gads[c] = p->G_ads[c];
  }
  h->G = p->G;
  h->rho_major = p->rho_major;
  h->rho_minor = p->rho_minor;
  h->rho_in = p->rho_in_nw;
  h->rho_out = p->rho_out_w;
  h->phib = (p->rho_major - p->rho_minor) / (p->rho_major + p->rho_minor);
  fill_phys(h);
}

int validate(const lbm_params *p) {
  if (!p) {
    set_err("params is NULL");
    return LBM_EINVAL;
  }
  if (p->nx < 3 || p->ny < 3 || p->nz < 3) {
    set_err("box %d x %d x %d: each side must be >= 3", p->nx, p->ny, p->nz);
    return LBM_EINVAL;
  }
  if ((long long)p->nx * p->ny * p->nz >= (1LL << 29)) {
    set_err("box of %lld nodes: at most 2^29 - 1 nodes per subdomain",
            (long long)p->nx * p->ny * p->nz);
    return LBM_EINVAL;
  }
  if ((long long)sc::pad_x(p->nx) * sc::pad_y(p->ny) > sc::kMaxPlaneNodes) {
    set_err("plane of %lld nodes (padded to %d x %d): at most %lld nodes per z-plane",
            (long long)p->nx * p->ny, sc::pad_x(p->nx), sc::pad_y(p->ny), sc::kMaxPlaneNodes);
    return LBM_EINVAL;
  }
  for (int a = 0; a < 3; ++a) {
    const int b = p->bc[a];
    const bool ok = b == LBM_BC_PERIODIC || b == LBM_BC_WALLS || (a == 2 && b == LBM_BC_RESERVOIR);
    if (!ok) {
      set_err("bc[%d] = %d is not a boundary kind allowed on that axis", a, b);
      return LBM_EINVAL;
    }
  }
  for (int c = 0; c < 2; ++c)
    if (!(std::isfinite(p->tau[c]) && p->tau[c] > 0.5)) {
      set_err("tau[%d] = %g must be finite and > 0.5", c, p->tau[c]);
      return LBM_EINVAL;
    }
  if (!std::isfinite(p->G) || !std::isfinite(p->G_ads[0]) || !std::isfinite(p->G_ads[1])) {
    set_err("interaction strengths must be finite");
    return LBM_EINVAL;
  }
  if (!finite_pos(p->rho_major) || !finite_pos(p->rho_minor) || !finite_pos(p->rho_in_nw) ||
      !finite_pos(p->rho_out_w)) {
    set_err("densities must be finite and > 0");
    return LBM_EINVAL;
  }
  if (p->n_spheres < 0 || (p->n_spheres > 0 && !p->spheres)) {
    set_err("sphere list invalid");
    return LBM_EINVAL;
  }
  for (int i = 0; i < p->n_spheres; ++i) {
    const lbm_sphere &s = p->spheres[i];
    if (!std::isfinite(s.c[0]) || !std::isfinite(s.c[1]) || !std::isfinite(s.c[2]) ||
        !finite_pos(s.r)) {
      set_err("sphere %d has a non-finite centre or a non-positive radius", i);
      return LBM_EINVAL;
    }
  }
  if (p->prism)
    for (int a = 0; a < 3; ++a)
      if (p->prism_ids[a] < 0 || p->prism_ids[a] >= p->n_spheres) {
        set_err("prism sphere id %d out of range", p->prism_ids[a]);
        return LBM_EINVAL;
      }
  return LBM_OK;
}

void release(lbm_throat *h) {
  if (!h) return;
  for (int i = 0; i < 2; ++i) {
    if (h->g[i]) (void)hipFree(h->g[i]);
    if (h->save[i]) (void)hipFree(h->save[i]);
    if (h->ev[i]) (void)hipEventDestroy(h->ev[i]);
    if (h->tev[i]) (void)hipEventDestroy(h->tev[i]);
  }
  for (void *p : {(void *)h->map_d, (void *)h->pos_d, (void *)h->rho_d, (void *)h->mask_d,
                  (void *)h->types_d, (void *)h->rres_d, (void *)h->partials,
                  (void *)h->chunks_d, (void *)h->redinfo_d, (void *)h->red_first_d,
                  (void *)h->red_count_d, (void *)h->desc_d, (void *)h->tiles_d,
                  (void *)h->zper_d})
    if (p) (void)hipFree(p);
  if (h->red_h) (void)hipHostFree(h->red_h);
  if (h->own_stream && h->stream) (void)hipStreamDestroy(h->stream);
  delete h;
}

hipError_t one_step(const lbm_throat *h, int parity) {
  // (the two passes over one subdomain take no list: its items are 0, 1, ...)
  const sc::TileRef *tiles = h->sched.tx == sc::kListTx ? nullptr : h->tiles_d;
  return sc::launch_step(h->desc_d, tiles, h->ntiles, h->sched.tx, h->sched.ty, lbmh::wide(h),
                         parity, h->stream, h->zper_d, h->n_zper);
}

int run_steps(lbm_throat *h, long long n) {
  for (long long i = 0; i < n; ++i) {
    const hipError_t e = one_step(h, h->cur);
    if (e != hipSuccess) {
      set_err("step launch failed: %s", hipGetErrorString(e));
      return LBM_EHIP;
    }
    h->cur = 1 - h->cur;
  }
  h->steps_done += n;
  return LBM_OK;
}

// FP64 masses, saturation and probe densities of the current state (the
// reduction the batched ramp uses too, so both give the same bits)
int reduce_now(lbm_throat *h, double out[5]) {
  HIPCHK(sc::launch_reduce_chunks(h->desc_d, h->chunks_d, h->nchunks, h->redinfo_d, h->cur,
                                  h->partials, h->red_h + 3, h->stream));
  HIPCHK(sc::launch_reduce_throats(h->red_first_d, h->red_count_d, 1, h->partials, h->red_h,
                                   h->stream));
  HIPCHK(hipStreamSynchronize(h->stream));
  for (int i = 0; i < 5; ++i) out[i] = h->red_h[i];
  out[2] = h->n_fluid ? out[2] / (double)h->n_fluid : 0.0;
  return LBM_OK;
}

int set_rho_in(lbm_throat *h, double r) {
  h->rho_in = r;
  fill_phys(h);
  TRY(sync_desc(h));
  return upload_rres(h);
}

int copy_state(lbm_throat *h, float *dst, const float *src) {
  HIPCHK(hipMemcpyAsync(dst, src, sizeof(float) * sc::pop_elems(h->n_numbers),
                        hipMemcpyDeviceToDevice, h->stream));
  return LBM_OK;
}

}  // namespace

namespace lbmh {
int describe(const lbm_params *p, lbm_throat *h) {
  TRY(validate(p));
  fill_handle(p, h);
  return LBM_OK;
}

Geometry::Geometry(const lbm_params &p) : sph(4 * (size_t)std::max(p.n_spheres, 1)) {
  for (int i = 0; i < p.n_spheres; ++i) {
    for (int a = 0; a < 3; ++a) sph[4 * i + a] = p.spheres[i].c[a];
    sph[4 * i + 3] = p.spheres[i].r;
  }
  sc::bin_spheres(sph.data(), p.n_spheres, p.nx, p.ny, p.nz, bin_start, bin_ids, ncx, ncy, ncz);
  if (bin_ids.empty()) bin_ids.push_back(0);
}

hipError_t Geometry::voxelize(const lbm_params &p, const double *sph_d, const int *start_d,
                              const int *ids_d, uint8_t *types_d, hipStream_t st) const {
  const sc::VoxBins bins{start_d, ids_d, ncx, ncy, ncz};
  int prism[3] = {0, 0, 0};
  for (int a = 0; a < 3 && p.prism; ++a) prism[a] = p.prism_ids[a];
  return sc::launch_voxelize(sph_d, bins, p.prism ? 1 : 0, prism, p.nx, p.ny, p.nz,
                             p.bc[2] == LBM_BC_RESERVOIR, types_d, st);
}

int check_rho_init(const lbm_throat *h, unsigned long long bad) {
  if (bad >= 2 * (unsigned long long)h->N) return LBM_OK;
  set_err("rho_init is not finite and positive on fluid node %zu", (size_t)(bad % h->N));
  return LBM_EINVAL;
}

bool fills_tiles(const lbm_throat *h) {
  const size_t lanes =
      (size_t)tile_columns(h->nx, h->ny) * (kTileTx * sc::tile_rows(kTileTy)) * (size_t)h->nz;
  return (double)h->n_live >= kTileFill * (double)lanes;
}

int tile_length(const std::vector<std::pair<long long, int>> &boxes) {
  int top = 1, length = 1;
  for (const auto &b : boxes) top = std::max(top, b.second);
  long long best = LLONG_MAX;
  for (int n = 1; n <= std::max(1, top / 16); ++n) {
    const int l = (top + n - 1) / n;
    long long groups = 0;
    for (const auto &b : boxes) {
      const int lz = std::min(l, b.second);
      groups += b.first * ((b.second + lz - 1) / lz);
    }
    const long long t = (groups + 255) / 256 * (l + 8);
    if (t < best) {
      best = t;
      length = l;
    }
  }
  return length;
}

sc::Sched batch_tiles(const std::vector<lbm_throat *> &boxes) {
  std::vector<std::pair<long long, int>> b;
  for (const lbm_throat *h : boxes) b.push_back({tile_columns(h->nx, h->ny), h->nz});
  const sc::Sched s{kTileTx, kTileTy, tile_length(b)};
  for (lbm_throat *h : boxes) h->sched = sc::Sched{s.tx, s.ty, std::min(s.lz, h->nz)};
  return s;
}

void fill_desc(lbm_throat *h) { ::fill_desc(h); }
sc::Dom dom(const lbm_throat *h) { return ::dom(h, nullptr, nullptr); }
}  // namespace lbmh


extern "C" {

const char *lbm_last_error(void) { return g_err.c_str(); }

int lbm_set_memory_budget(size_t bytes) {
  g_budget.store(bytes);
  return LBM_OK;
}

}  // extern "C"

namespace {

bool own_bricks(const lbm_throat *h) {
  return lbmh::fills_tiles(h) && lbmh::brick_slots(h) >= lbmh::kTileNodes;
}

bool alloc_device(void **q, size_t bytes) {
  if (hipMalloc(q, std::max<size_t>(bytes, 16)) == hipSuccess) return true;
  *q = nullptr;
  (void)hipGetLastError();
  set_err("hipMalloc of %zu bytes failed", bytes);
  return false;
}

// the number of the probe node, read from `map`, on the host and the device
bool set_probe(lbm_throat *h, const uint32_t *map) {
  long long probe = -1;
  if (h->probe_pos >= 0) {
    uint32_t number = 0;
    if (hipMemcpy(&number, map + h->probe_pos, sizeof number, hipMemcpyDeviceToHost) != hipSuccess)
      return false;
    probe = (long long)number;
  }
  const sc::RedInfo ri{probe, h->phib};
  if (hipMemcpy(h->redinfo_d, &ri, sizeof ri, hipMemcpyHostToDevice) != hipSuccess) return false;
  h->probe = probe;
  return true;
}

// The other numbering for a subdomain, its state and checkpoints carried over
// bit for bit.  Nothing of the handle is changed before all of it is there.
// Compact populations fit the buffers that held bricks: where no others can be
// had, they move into these, the state to the one that does not hold it and
// each checkpoint by way of the one that then no longer does.
int set_numbering(lbm_throat *h, bool bricks) {
  if (h->bricks == bricks) return LBM_OK;
  const size_t numbers = bricks ? lbmh::brick_numbers(h) : h->n_live;
  const size_t pop_bytes = sizeof(float) * sc::pop_elems(numbers);
  const size_t map_bytes = sizeof(uint32_t) * sc::map_elems(h->nx, h->ny, h->nz);
  const size_t side_bytes = bricks ? sizeof(uint32_t) * h->N : sizeof(float2) * numbers;
  const bool ghosts = bricks && (h->per & 4);
  const uint32_t n_live = (uint32_t)h->n_live;
  struct Storage {
    void *g[2] = {}, *save[2] = {}, *map = nullptr, *side = nullptr, *zper = nullptr;
    void drop() {
      for (void **p : {&g[0], &g[1], &save[0], &save[1], &map, &side, &zper}) {
        if (*p) (void)hipFree(*p);
        *p = nullptr;
      }
    }
    ~Storage() { drop(); }
  } f;
  TRY(lbmh::check_budget(
      lbmh::subdomain_bytes(h->nx, h->ny, h->nz, h->save[0] || h->save[1]), "lbm_set_schedule"));
  bool room = true;
  for (int i = 0; i < 2; ++i)
    room = room && alloc_device(&f.g[i], pop_bytes) &&
           (!h->save[i] || alloc_device(&f.save[i], pop_bytes));
  if (!room && bricks) return LBM_ENOMEM;
  if (!room) f.drop();
  if (!alloc_device(&f.map, map_bytes) || !alloc_device(&f.side, side_bytes) ||
      (ghosts && !alloc_device(&f.zper, sizeof(int))))
    return LBM_ENOMEM;
  const int zero = 0;
  if (ghosts) HIPCHK(hipMemcpyAsync(f.zper, &zero, sizeof zero, hipMemcpyHostToDevice, h->stream));
  sc::Dom d = dom(h, nullptr, nullptr);
  d.map = (uint32_t *)f.map;
  HIPCHK(sc::launch_renumber(d, h->types_d, h->pos_d, n_live, bricks, (uint32_t *)f.map,
                             h->stream));
  auto move = [&](const float *from, void *to) {
    return sc::launch_move(d, h->pos_d, n_live, bricks, from, (float *)to, h->stream);
  };
  if (room) {
    HIPCHK(move(h->g[h->cur], f.g[h->cur]));
    for (int i = 0; i < 2; ++i)
      if (h->save[i]) HIPCHK(move(h->save[i], f.save[i]));
  }
  if (bricks) HIPCHK(sc::launch_links(h->types_d, d, (uint32_t *)f.side, h->stream));
  HIPCHK(hipStreamSynchronize(h->stream));
  if (!set_probe(h, (uint32_t *)f.map)) {
    set_err("renumbering the probe failed");
    return LBM_EHIP;
  }
  // exchanged: what the handle had is released with f
  const auto take = [](auto *&mine, void *&fresh) {
    void *old = mine;
    mine = static_cast<std::remove_reference_t<decltype(mine)>>(fresh);
    fresh = old;
  };
  if (room) {
    for (int i = 0; i < 2; ++i) {
      take(h->g[i], f.g[i]);
      take(h->save[i], f.save[i]);
    }
  } else {
    float *idle = h->g[h->cur];
    h->cur = 1 - h->cur;
    HIPCHK(move(idle, h->g[h->cur]));
    for (float *save : h->save)
      if (save) {
        HIPCHK(move(save, idle));
        HIPCHK(hipMemcpyAsync(save, idle, pop_bytes, hipMemcpyDeviceToDevice, h->stream));
      }
    HIPCHK(hipStreamSynchronize(h->stream));
  }
  take(h->map_d, f.map);
  take(h->zper_d, f.zper);
  void *none = nullptr;
  if (bricks) {
    take(h->mask_d, f.side);
    take(h->rho_d, none);
  } else {
    take(h->rho_d, f.side);
    take(h->mask_d, none);
  }
  if (none) (void)hipFree(none);
  h->n_zper = ghosts ? 1 : 0;
  h->bricks = bricks;
  h->n_numbers = numbers;
  return LBM_OK;
}

// Launch shape s: the numbering it runs over, and its work items, which are the
// tiles that hold a non-solid node or the number of items of the two passes
// (one subdomain's need no list).  (The two passes over bricks touch four lines
// where tiles touch one: 4200 us a step at 256^3 against 1137, and 1523 over
// compact nodes.)  Without the memory for it the handle stays as it was.
int set_shape(lbm_throat *h, const sc::Sched &s) {
  const bool tiled = s.tx != sc::kListTx;
  std::vector<sc::TileRef> list;
  struct Fresh {
    void *d = nullptr;
    ~Fresh() {
      if (d) (void)hipFree(d);
    }
  } fresh;
  if (tiled) {
    if (h->brick_live.empty())
      sc::brick_map(h->types.data(), h->nx, h->ny, h->nz, h->brick_live);
    sc::list_tiles(h->brick_live.data(), h->nx, h->ny, h->nz, s.tx, sc::tile_rows(s.ty), s.lz, 0,
                   list);
    if (list.size() > h->tiles_cap && !alloc_device(&fresh.d, sizeof(sc::TileRef) * list.size()))
      return LBM_ENOMEM;
  }
  TRY(set_numbering(h, tiled));
  if (fresh.d) {
    HIPCHK(hipStreamSynchronize(h->stream));
    void *old = h->tiles_d;
    h->tiles_d = (sc::TileRef *)fresh.d;
    fresh.d = old;
    h->tiles_cap = list.size();
  }
  h->sched = s;
  h->ntiles = (int)(tiled ? list.size() : sc::list_count(h->n_live));
  if (!list.empty()) {
    HIPCHK(hipMemcpyAsync(h->tiles_d, list.data(), sizeof(sc::TileRef) * list.size(),
                          hipMemcpyHostToDevice, h->stream));
    HIPCHK(hipStreamSynchronize(h->stream));
  }
  return sync_desc(h);
}

int init_subdomain(const lbm_params *p, lbm_throat_t *out) {
  g_err.clear();
  if (!out) {
    set_err("out is NULL");
    return LBM_EINVAL;
  }
  TRY(validate(p));
  TRY(lbmh::check_budget(lbmh::subdomain_bytes(p->nx, p->ny, p->nz, false), "lbm_throat_init"));
  lbm_throat *h = new (std::nothrow) lbm_throat();
  if (!h) {
    set_err("host allocation failed");
    return LBM_ENOMEM;
  }
  fill_handle(p, h);

  auto fail = [&](int code) {
    release(h);
    return code;
  };
  if (p->stream) {
    h->stream = (hipStream_t)p->stream;
  } else {
    if (hipStreamCreate(&h->stream) != hipSuccess) {
      set_err("hipStreamCreate failed");
      return fail(LBM_EHIP);
    }
    h->own_stream = true;
  }
#define ALLOC(ptr, bytes)                                                      \
  do {                                                                         \
    if (hipMalloc((void **)&(ptr), (bytes)) != hipSuccess) {                   \
      set_err("hipMalloc of %zu bytes failed", (size_t)(bytes));               \
      return fail(LBM_ENOMEM);                                                 \
    }                                                                          \
  } while (0)
  ALLOC(h->types_d, h->N);
  ALLOC(h->map_d, sizeof(uint32_t) * sc::map_elems(h->nx, h->ny, h->nz));
  ALLOC(h->rres_d, 4 * sizeof(double));
  ALLOC(h->redinfo_d, sizeof(sc::RedInfo));
  ALLOC(h->desc_d, sizeof(sc::Throat));
  if (hipHostMalloc((void **)&h->red_h, 5 * sizeof(double), hipHostMallocDefault) != hipSuccess) {
    set_err("hipHostMalloc failed");
    return fail(LBM_ENOMEM);
  }
  for (int i = 0; i < 2; ++i)
    if (hipEventCreate(&h->ev[i]) != hipSuccess || hipEventCreate(&h->tev[i]) != hipSuccess) {
      set_err("hipEventCreate failed");
      return fail(LBM_EHIP);
    }

  // geometry on the device
  double *sph_d = nullptr, *rho_d = nullptr;
  const lbmh::Geometry geo(*p);
  const std::vector<double> &sph = geo.sph;
  const std::vector<int> &bin_start = geo.bin_start, &bin_ids = geo.bin_ids;
  int *bins_d = nullptr;
  ALLOC(sph_d, sizeof(double) * sph.size());
  if (hipMalloc((void **)&bins_d, sizeof(int) * (bin_start.size() + bin_ids.size())) !=
      hipSuccess) {
    (void)hipGetLastError();
    (void)hipFree(sph_d);
    set_err("hipMalloc of the sphere bins failed");
    return fail(LBM_ENOMEM);
  }
  std::vector<uint32_t> rows((size_t)h->ny * h->nz);
  uint32_t *rows_d = nullptr;
  if (hipMalloc((void **)&rows_d, sizeof(uint32_t) * rows.size()) != hipSuccess) {
    (void)hipGetLastError();
    (void)hipFree(sph_d);
    (void)hipFree(bins_d);
    set_err("hipMalloc of the row counts failed");
    return fail(LBM_ENOMEM);
  }
  int rc = LBM_OK;
  do {
    if (hipMemcpyAsync(sph_d, sph.data(), sizeof(double) * sph.size(), hipMemcpyHostToDevice,
                       h->stream) != hipSuccess ||
        hipMemcpyAsync(bins_d, bin_start.data(), sizeof(int) * bin_start.size(),
                       hipMemcpyHostToDevice, h->stream) != hipSuccess ||
        hipMemcpyAsync(bins_d + bin_start.size(), bin_ids.data(), sizeof(int) * bin_ids.size(),
                       hipMemcpyHostToDevice, h->stream) != hipSuccess) {
      rc = LBM_EHIP;
      break;
    }
    if (geo.voxelize(*p, sph_d, bins_d, bins_d + bin_start.size(), h->types_d, h->stream) !=
            hipSuccess ||
        sc::launch_row_counts(h->types_d, h->nx, h->ny, h->nz, rows_d, h->stream) !=
            hipSuccess) {
      rc = LBM_EHIP;
      break;
    }
    h->types.resize(h->N);
    if (hipMemcpyAsync(rows.data(), rows_d, sizeof(uint32_t) * rows.size(),
                       hipMemcpyDeviceToHost, h->stream) != hipSuccess ||
        hipMemcpyAsync(h->types.data(), h->types_d, h->N, hipMemcpyDeviceToHost, h->stream) !=
            hipSuccess ||
        hipStreamSynchronize(h->stream) != hipSuccess) {
      rc = LBM_EHIP;
      break;
    }
  } while (0);
  if (rc == LBM_OK && hipStreamSynchronize(h->stream) != hipSuccess) rc = LBM_EHIP;
  (void)hipFree(sph_d);
  (void)hipFree(bins_d);
  auto fail_rows = [&](int code) {
    (void)hipFree(rows_d);
    return fail(code);
  };
  if (rc != LBM_OK) {
    set_err("geometry setup failed");
    return fail_rows(rc);
  }
  // numbering, populations, work items
  h->n_live = sc::number_rows(rows.data(), h->ny, h->nz);
  const size_t plane = (size_t)h->nx * h->ny;
  h->n_fluid = (long long)h->n_live;
  if (p->bc[2] == LBM_BC_RESERVOIR)
    for (size_t n = 0; n < plane; ++n)
      h->n_fluid -= (h->types[n] != sc::kSolid) + (h->types[h->N - plane + n] != sc::kSolid);
  h->bricks = own_bricks(h);
  h->n_numbers = h->bricks ? lbmh::brick_numbers(h) : h->n_live;
  const size_t pop_bytes = sizeof(float) * sc::pop_elems(h->n_numbers);
  std::vector<sc::RedChunk> chunks;
  sc::red_chunks(h->n_live, 0, chunks);
  h->nchunks = (int)chunks.size();
  size_t free_b = 0, total_b = 0;
  if (hipMemGetInfo(&free_b, &total_b) != hipSuccess) {
    set_err("hipMemGetInfo failed");
    return fail_rows(LBM_EHIP);
  }
  const size_t need = 2 * pop_bytes + 4 * h->n_live +
                      (h->bricks ? 4 * h->N : 8 * h->n_numbers) + (64u << 20);
  if (need > free_b) {
    set_err("needs %zu bytes of device memory, %zu free", need, free_b);
    return fail_rows(LBM_ENOMEM);
  }
  auto alloc = [](auto **q, size_t bytes) { return alloc_device((void **)q, bytes); };
  if (!alloc(&h->g[0], pop_bytes) || !alloc(&h->g[1], pop_bytes) ||
      !alloc(&h->pos_d, sizeof(uint32_t) * h->n_live) ||
      (!h->bricks && !alloc(&h->rho_d, sizeof(float2) * h->n_numbers)) ||
      (h->bricks && !alloc(&h->mask_d, sizeof(uint32_t) * h->N)) ||
      !alloc(&h->chunks_d, sizeof(sc::RedChunk) * chunks.size()) ||
      !alloc(&h->partials, sizeof(double) * 3 * chunks.size()) ||
      !alloc(&h->red_first_d, sizeof(int)) || !alloc(&h->red_count_d, sizeof(int)))
    return fail_rows(LBM_ENOMEM);
  {
    const int zero = 0;
    bool ok = hipMemcpyAsync(rows_d, rows.data(), sizeof(uint32_t) * rows.size(),
                             hipMemcpyHostToDevice, h->stream) == hipSuccess &&
              sc::launch_number(h->types_d, h->nx, h->ny, h->nz, h->per, rows_d, h->bricks,
                                h->map_d, h->pos_d, h->stream) == hipSuccess;
    ok = ok && (chunks.empty() ||
                hipMemcpyAsync(h->chunks_d, chunks.data(), sizeof(sc::RedChunk) * chunks.size(),
                               hipMemcpyHostToDevice, h->stream) == hipSuccess);
    ok = ok &&
         hipMemcpyAsync(h->red_first_d, &zero, sizeof(int), hipMemcpyHostToDevice, h->stream) ==
             hipSuccess &&
         hipMemcpyAsync(h->red_count_d, &h->nchunks, sizeof(int), hipMemcpyHostToDevice,
                        h->stream) == hipSuccess;
    if (ok && h->bricks) {
      ok = sc::launch_links(h->types_d, dom(h, nullptr, nullptr), h->mask_d, h->stream) ==
           hipSuccess;
      if (ok && (h->per & 4)) {
        if (!alloc(&h->zper_d, sizeof(int))) return fail_rows(LBM_ENOMEM);
        ok = hipMemcpyAsync(h->zper_d, &zero, sizeof(int), hipMemcpyHostToDevice, h->stream) ==
             hipSuccess;
        h->n_zper = 1;
      }
    }
    if (hipStreamSynchronize(h->stream) != hipSuccess) ok = false;
    (void)hipFree(rows_d);
    if (!ok) {
      set_err("numbering of the nodes failed");
      return fail(LBM_EHIP);
    }
  }

  if (p->probe[0] >= 0) {
    if (p->probe[0] >= h->nx || p->probe[1] < 0 || p->probe[1] >= h->ny || p->probe[2] < 0 ||
        p->probe[2] >= h->nz) {
      set_err("probe node outside the box");
      return fail(LBM_EINVAL);
    }
    const size_t node = (size_t)p->probe[0] +
                        (size_t)h->nx * ((size_t)p->probe[1] + (size_t)h->ny * p->probe[2]);
    if (h->types[node] != sc::kFluid) {
      set_err("probe node is not a fluid node");
      return fail(LBM_EINVAL);
    }
    h->probe_pos =
        (long long)sc::map_pos(h->nx, h->ny, p->probe[0], p->probe[1], p->probe[2]);
  }
  if (!set_probe(h, h->map_d)) {
    set_err("upload of the reduction info failed");
    return fail(LBM_EHIP);
  }
  unsigned long long bad = ~0ull, *bad_d = nullptr;
  if (p->rho_init) {
    ALLOC(rho_d, sizeof(double) * (2 * h->N + 1));
    bad_d = (unsigned long long *)(rho_d + 2 * h->N);
    if (hipMemsetAsync(bad_d, 0xff, sizeof bad, h->stream) != hipSuccess ||
        hipMemcpyAsync(rho_d, p->rho_init, sizeof(double) * 2 * h->N, hipMemcpyHostToDevice,
                       h->stream) != hipSuccess) {
      (void)hipFree(rho_d);
      set_err("rho_init upload failed");
      return fail(LBM_EHIP);
    }
  }
  if (upload_rres(h) != LBM_OK) {
    if (rho_d) (void)hipFree(rho_d);
    return fail(LBM_EHIP);
  }
  const sc::Dom d = dom(h, nullptr, nullptr);
  hipError_t e = sc::launch_init(d, h->P, rho_d, h->rho_major, h->rho_minor, p->z_front, h->rres_d,
                                 h->g[0], bad_d, h->stream);
  if (e == hipSuccess && bad_d)
    e = hipMemcpyAsync(&bad, bad_d, sizeof bad, hipMemcpyDeviceToHost, h->stream);
  if (e == hipSuccess) e = hipMemsetAsync(h->g[1], 0, pop_bytes, h->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(h->stream);
  if (rho_d) (void)hipFree(rho_d);
  if (e != hipSuccess) {
    set_err("initial state failed: %s", hipGetErrorString(e));
    return fail(LBM_EHIP);
  }
  if (const int r = lbmh::check_rho_init(h, bad)) return fail(r);
  h->cur = 0;
  if (const int r = set_shape(h, h->bricks ? default_schedule(h->nx, h->ny, h->nz)
                                          : sc::Sched{sc::kListTx, 0, 0}))
    return fail(r);
  if (sc::launch_ghost(h->desc_d, h->zper_d, h->n_zper, 0, h->stream) != hipSuccess ||
      hipStreamSynchronize(h->stream) != hipSuccess) {
    set_err("initial ghost planes failed");
    return fail(LBM_EHIP);
  }
  *out = h;
  return LBM_OK;
#undef ALLOC
}

}  // namespace

extern "C" {

int lbm_throat_init(const lbm_params *p, lbm_throat_t *out) {
  return init_subdomain(p, out);
}

void lbm_throat_free(lbm_throat_t h) { release(h); }

int lbm_step(lbm_throat_t h, long long nsteps) {
  if (!h || nsteps < 0) {
    set_err("lbm_step: bad handle or negative step count");
    return LBM_EINVAL;
  }
  return run_steps(h, nsteps);
}

int lbm_sync(lbm_throat_t h) {
  if (!h) {
    set_err("NULL handle");
    return LBM_EINVAL;
  }
  HIPCHK(hipStreamSynchronize(h->stream));
  return LBM_OK;
}

int lbm_set_rho_in(lbm_throat_t h, double r) {
  if (!h || !finite_pos(r)) {
    set_err("lbm_set_rho_in: bad handle or density");
    return LBM_EINVAL;
  }
  return set_rho_in(h, r);
}

double lbm_rho_in_for_pc(lbm_throat_t h, double pc) {
  if (!h) return NAN;
  return h->rho_out + pc / (kCs2 * (1.0 + h->G * h->rho_minor));
}

long long lbm_nodes(lbm_throat_t h) { return h ? (long long)h->N : -1; }

int lbm_get_types(lbm_throat_t h, unsigned char *types) {
  if (!h || !types) {
    set_err("lbm_get_types: NULL argument");
    return LBM_EINVAL;
  }
  std::memcpy(types, h->types.data(), h->N);
  return LBM_OK;
}

int lbm_get_populations(lbm_throat_t h, double *f) {
  if (!h || !f) {
    set_err("lbm_get_populations: NULL argument");
    return LBM_EINVAL;
  }
  double *fd = nullptr;
  if (hipMalloc((void **)&fd, sizeof(double) * 38 * h->N) != hipSuccess) {
    set_err("hipMalloc for the export failed");
    return LBM_ENOMEM;
  }
  const sc::Dom d = dom(h, h->g[h->cur], nullptr);
  hipError_t e = sc::launch_export(d, h->P, h->rres_d, fd, h->stream);
  if (e == hipSuccess)
    e = hipMemcpyAsync(f, fd, sizeof(double) * 38 * h->N, hipMemcpyDeviceToHost, h->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(h->stream);
  (void)hipFree(fd);
  if (e != hipSuccess) {
    set_err("export failed: %s", hipGetErrorString(e));
    return LBM_EHIP;
  }
  return LBM_OK;
}

int lbm_get_density(lbm_throat_t h, double *rho) {
  if (!h || !rho) {
    set_err("lbm_get_density: NULL argument");
    return LBM_EINVAL;
  }
  double *rd = nullptr;
  if (hipMalloc((void **)&rd, sizeof(double) * 2 * h->N) != hipSuccess) {
    set_err("hipMalloc for the density read-back failed");
    return LBM_ENOMEM;
  }
  const sc::Dom d = dom(h, h->g[h->cur], nullptr);
  hipError_t e = sc::launch_density(d, h->P, h->rres_d, rd, h->stream);
  if (e == hipSuccess)
    e = hipMemcpyAsync(rho, rd, sizeof(double) * 2 * h->N, hipMemcpyDeviceToHost, h->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(h->stream);
  (void)hipFree(rd);
  if (e != hipSuccess) {
    set_err("density read-back failed: %s", hipGetErrorString(e));
    return LBM_EHIP;
  }
  return LBM_OK;
}

int lbm_get_density_noalloc(lbm_throat_t h, double *rho) {
  if (!h || !rho) {
    set_err("lbm_get_density_noalloc: NULL argument");
    return LBM_EINVAL;
  }
  if (h->N > sc::kScratchNodes) {
    set_err("lbm_get_density_noalloc: %zu nodes exceed the fixed staging array of %zu nodes",
            h->N, sc::kScratchNodes);
    return LBM_EINVAL;
  }
  double *stage = nullptr;
  hipError_t e = sc::scratch_address(&stage);
  if (e != hipSuccess) {
    set_err("lbm_get_density_noalloc: no address for the staging array: %s",
            hipGetErrorString(e));
    return LBM_EHIP;
  }
  // k_density writes all 2 N values, so nothing left by an earlier call is read
  const sc::Dom d = dom(h, h->g[h->cur], nullptr);
  e = sc::launch_density(d, h->P, h->rres_d, stage, h->stream);
  if (e == hipSuccess)
    e = hipMemcpyAsync(rho, stage, sizeof(double) * 2 * h->N, hipMemcpyDeviceToHost, h->stream);
  if (e == hipSuccess) e = hipStreamSynchronize(h->stream);
  if (e != hipSuccess) {
    set_err("lbm_get_density_noalloc: read-back failed: %s", hipGetErrorString(e));
    return LBM_EHIP;
  }
  return LBM_OK;
}

int lbm_reduce(lbm_throat_t h, double *mass2, double *S_w) {
  if (!h) {
    set_err("NULL handle");
    return LBM_EINVAL;
  }
  double r[5];
  TRY(reduce_now(h, r));
  if (mass2) {
    mass2[0] = r[0];
    mass2[1] = r[1];
  }
  if (S_w) *S_w = r[2];
  return LBM_OK;
}

int lbm_probe_invaded(lbm_throat_t h, int *invaded) {
  if (!h || !invaded) {
    set_err("NULL argument");
    return LBM_EINVAL;
  }
  if (h->probe < 0) {
    set_err("the handle has no probe node");
    return LBM_ESTATE;
  }
  double r[5];
  TRY(reduce_now(h, r));
  *invaded = r[4] > r[3] ? 1 : 0;
  return LBM_OK;
}

}  // extern "C"

namespace {

// ---- the drainage ramp of one subdomain as a resumable state machine -----
// Sec. 2.2.2: the capillary pressures are visited in increasing order, each
// held until the wetting saturation settles; the first invaded interval is
// bisected from the last stable state.  The machine advances in chunks of
// check_every steps, so a caller can stop it after any chunk, save the
// handle (lbm_save) and resume it in another handle (lbm_load); run to the
// end in one call it is lbm_drain_throat.

int check_drain_args(lbm_throat *h, const double *pc, int n_pc, const lbm_conv *c,
                     const char *who) {
  if (!h || !pc || n_pc < 1 || !c) {
    set_err("%s: NULL argument or n_pc < 1", who);
    return LBM_EINVAL;
  }
  if (!(c->tol > 0) || c->check_every < 1 || c->max_steps < c->check_every ||
      !(c->bisect_rel > 0)) {
    set_err("%s: invalid convergence settings", who);
    return LBM_EINVAL;
  }
  if (h->probe < 0) {
    set_err("%s needs a probe node", who);
    return LBM_ESTATE;
  }
  for (int i = 0; i < n_pc; ++i) {
    if (!std::isfinite(pc[i]) || !(pc[i] > 0) || !(lbm_rho_in_for_pc(h, pc[i]) > 0) ||
        (i > 0 && !(pc[i] > pc[i - 1]))) {
      set_err("%s: pc must be finite, positive, strictly increasing and give a positive inlet "
              "density", who);
      return LBM_EINVAL;
    }
  }
  return LBM_OK;
}

int ensure_checkpoints(lbm_throat *h, const char *who) {
  if (!h->save[0] || !h->save[1])
    TRY(lbmh::check_budget(lbmh::subdomain_bytes(h->nx, h->ny, h->nz, true), who));
  for (int i = 0; i < 2; ++i)
    if (!h->save[i] &&
        hipMalloc((void **)&h->save[i], sizeof(float) * sc::pop_elems(h->n_numbers)) !=
            hipSuccess) {
      set_err("hipMalloc of a ramp checkpoint failed");
      return LBM_ENOMEM;
    }
  return LBM_OK;
}

// a run to steady state starts: the saturation it is compared against
int run_start(lbm_throat *h) {
  double r[5];
  TRY(reduce_now(h, r));
  h->ramp.S_old = r[2];
  h->ramp.run_steps = 0;
  return LBM_OK;
}

// one chunk of check_every steps of the run in progress; *ended = 1 when the
// run has ended, with its status, saturation and invasion test
int run_chunk(lbm_throat *h, int *ended, int *st, double *S, int *inv) {
  HostRamp &R = h->ramp;
  double r[5];
  if (h->timing) HIPCHK(hipEventRecord(h->tev[0], h->stream));
  TRY(run_steps(h, R.c.check_every));
  if (h->timing) HIPCHK(hipEventRecord(h->tev[1], h->stream));
  R.run_steps += R.c.check_every;
  TRY(reduce_now(h, r));
  if (h->timing) {
    float ms = 0.f;
    HIPCHK(hipEventElapsedTime(&ms, h->tev[0], h->tev[1]));
    h->timed_ms += ms;
    h->timed_launches += R.c.check_every;
  }
  const double S_new = r[2];
  *ended = 1;
  if (!std::isfinite(S_new))
    *st = LBM_PT_NONFINITE;
  else if (std::fabs(S_new - R.S_old) < R.c.tol)
    *st = LBM_PT_CONVERGED;
  else if (R.run_steps >= R.c.max_steps)
    *st = LBM_PT_NOT_CONVERGED;
  else
    *ended = 0;
  *S = S_new;
  *inv = r[4] > r[3] ? 1 : 0;
  if (!*ended) R.S_old = S_new;
  return LBM_OK;
}

int ramp_next_point(lbm_throat *h) {
  HostRamp &R = h->ramp;
  R.point += 1;
  if (R.point >= (int)R.pc.size()) {
    R.phase = HostRamp::kDone;
    return LBM_OK;
  }
  R.phase = HostRamp::kRamp;
  TRY(set_rho_in(h, lbm_rho_in_for_pc(h, R.pc[R.point])));
  return run_start(h);
}

// the next bisection run from the last stable state, or the end of the
// bisection: back to the invaded ramp state and on to the next point
int ramp_bisect_or_resume(lbm_throat *h) {
  HostRamp &R = h->ramp;
  if ((R.hi - R.lo) / R.hi > R.c.bisect_rel) {
    if (R.runs < sc::kMaxBisect) {
      ++R.runs;
      R.mid = 0.5 * (R.lo + R.hi);
      R.phase = HostRamp::kBisect;
      TRY(copy_state(h, h->g[h->cur], h->save[0]));
      TRY(set_rho_in(h, lbm_rho_in_for_pc(h, R.mid)));
      return run_start(h);
    }
    R.warn = 1;  // bracket left wider than asked (a throat invaded at pc[0])
  }
  TRY(copy_state(h, h->g[h->cur], h->save[1]));
  TRY(set_rho_in(h, R.main_rho_in));
  return ramp_next_point(h);
}

int ramp_begin(lbm_throat *h, const double *pc, int n_pc, const lbm_conv *c) {
  TRY(ensure_checkpoints(h, "lbm_drain"));
  HostRamp R;
  R.pc.assign(pc, pc + n_pc);
  R.c = *c;
  R.S.assign(n_pc, 0.0);
  R.steps.assign(n_pc, 0);
  R.status.assign(n_pc, LBM_PT_NOT_RUN);
  R.phase = HostRamp::kRamp;
  R.point = 0;
  h->ramp = std::move(R);
  TRY(copy_state(h, h->save[0], h->g[h->cur]));
  TRY(set_rho_in(h, lbm_rho_in_for_pc(h, h->ramp.pc[0])));
  return run_start(h);
}

// advance by whole chunks until the ramp is done or max_steps lattice steps
// have run in this call
int ramp_advance(lbm_throat *h, long long max_steps) {
  HostRamp &R = h->ramp;
  long long ran = 0;
  while (R.phase == HostRamp::kRamp || R.phase == HostRamp::kBisect) {
    if (ran >= max_steps) break;
    int ended = 0, st = 0, inv = 0;
    double S = 0.0;
    TRY(run_chunk(h, &ended, &st, &S, &inv));
    ran += R.c.check_every;
    if (!ended) continue;
    if (st == LBM_PT_NONFINITE) {
      set_err("the state became non-finite %s", R.phase == HostRamp::kBisect
                                                    ? "while bisecting"
                                                    : "at a ramp point");
      R.failed = 1;
      R.phase = HostRamp::kDone;
      if (R.point < (int)R.status.size() && R.status[R.point] == LBM_PT_NOT_RUN)
        R.status[R.point] = LBM_PT_NONFINITE;
      for (size_t j = R.point + 1; j < R.status.size(); ++j) R.status[j] = LBM_PT_NONFINITE;
      return LBM_ENONFINITE;
    }
    if (R.phase == HostRamp::kRamp) {
      const int i = R.point;
      R.S[i] = S;
      R.steps[i] = R.run_steps;
      R.status[i] = st;
      R.total += R.run_steps;
      R.warn |= st == LBM_PT_NOT_CONVERGED;
      if (!inv) {
        TRY(copy_state(h, h->save[0], h->g[h->cur]));
        R.stable_pc = R.pc[i];
        TRY(ramp_next_point(h));
      } else if (R.inv_at >= 0) {
        TRY(ramp_next_point(h));
      } else {
        R.inv_at = i;
        R.lo = i == 0 ? 0.0 : R.stable_pc;
        R.hi = R.pc[i];
        R.main_rho_in = h->rho_in;
        R.runs = 0;
        TRY(copy_state(h, h->save[1], h->g[h->cur]));
        TRY(ramp_bisect_or_resume(h));
      }
    } else {  // a bisection run ended
      R.total += R.run_steps;
      ++R.n_bisect;
      if (inv) {
        R.hi = R.mid;
      } else {
        R.lo = R.mid;
        TRY(copy_state(h, h->save[0], h->g[h->cur]));
      }
      TRY(ramp_bisect_or_resume(h));
    }
  }
  return LBM_OK;
}

void ramp_result(const lbm_throat *h, lbm_drain_result *out) {
  const HostRamp &R = h->ramp;
  const int n = (int)R.pc.size();
  for (int i = 0; i < n; ++i) {
    out->S[i] = R.S[i];
    out->steps[i] = R.steps[i];
    out->status[i] = R.status[i];
  }
  out->invaded_at = R.inv_at;
  out->n_bisect = R.n_bisect;
  out->total_steps = R.total;
  out->failed = R.failed;
  if (R.failed) {
    out->pce_lo = out->pce = out->pce_hi = NAN;
  } else if (R.inv_at < 0) {
    out->pce_lo = n ? R.pc[n - 1] : NAN;
    out->pce = NAN;
    out->pce_hi = INFINITY;
  } else {
    out->pce_lo = R.lo;
    out->pce_hi = R.hi;
    out->pce = 0.5 * (R.lo + R.hi);
  }
}

}  // namespace

extern "C" {

int lbm_drain_throat(lbm_throat_t h, const double *pc, int n_pc, const lbm_conv *c,
                     lbm_drain_result *out) {
  if (!out || !out->S || !out->steps || !out->status) {
    set_err("lbm_drain_throat: NULL result arrays");
    return LBM_EINVAL;
  }
  TRY(check_drain_args(h, pc, n_pc, c, "lbm_drain_throat"));
  TRY(ramp_begin(h, pc, n_pc, c));
  TRY(ramp_advance(h, LLONG_MAX));
  HIPCHK(hipStreamSynchronize(h->stream));
  ramp_result(h, out);
  return h->ramp.warn ? LBM_WNOTCONV : LBM_OK;
}

int lbm_drain_begin(lbm_throat_t h, const double *pc, int n_pc, const lbm_conv *c) {
  TRY(check_drain_args(h, pc, n_pc, c, "lbm_drain_begin"));
  return ramp_begin(h, pc, n_pc, c);
}

int lbm_drain_advance(lbm_throat_t h, long long max_steps, int *done) {
  if (!h || max_steps < 0) {
    set_err("lbm_drain_advance: NULL handle or negative step budget");
    return LBM_EINVAL;
  }
  if (h->ramp.phase == HostRamp::kIdle) {
    set_err("lbm_drain_advance: no drainage ramp begun on this handle");
    return LBM_ESTATE;
  }
  TRY(ramp_advance(h, max_steps));
  HIPCHK(hipStreamSynchronize(h->stream));
  if (done) *done = h->ramp.phase == HostRamp::kDone ? 1 : 0;
  return LBM_OK;
}

int lbm_drain_get(lbm_throat_t h, int n_pc, lbm_drain_result *out, int *done) {
  if (!h || !out || !out->S || !out->steps || !out->status) {
    set_err("lbm_drain_get: NULL argument");
    return LBM_EINVAL;
  }
  if (h->ramp.phase == HostRamp::kIdle) {
    set_err("lbm_drain_get: no drainage ramp begun on this handle");
    return LBM_ESTATE;
  }
  if (n_pc != (int)h->ramp.pc.size()) {
    set_err("lbm_drain_get: the ramp has %d points, not %d", (int)h->ramp.pc.size(), n_pc);
    return LBM_EINVAL;
  }
  ramp_result(h, out);
  if (done) *done = h->ramp.phase == HostRamp::kDone ? 1 : 0;
  return h->ramp.warn ? LBM_WNOTCONV : LBM_OK;
}

}  // extern "C"

namespace {

// ---- checkpoint files (lbm_save / lbm_load) --------------------------------
constexpr char kMagic[8] = {'L', 'B', 'M', 'S', 'C', 'v', '1', '\0'};
constexpr size_t kIoChunk = (size_t)16 << 20;  // floats per host staging chunk

uint64_t types_hash(const std::vector<uint8_t> &t) {
  uint64_t x = 1469598103934665603ULL;  // FNV-1a, 64 bit
  for (uint8_t b : t) {
    x ^= b;
    x *= 1099511628211ULL;
  }
  return x;
}

struct File {
  FILE *f = nullptr;
  ~File() {
    if (f) fclose(f);
  }
  template <class T>
  bool put(const T &v) { return fwrite(&v, sizeof(T), 1, f) == 1; }
  template <class T>
  bool put_n(const T *v, size_t n) { return n == 0 || fwrite(v, sizeof(T), n, f) == n; }
  template <class T>
  bool get(T &v) { return fread(&v, sizeof(T), 1, f) == 1; }
  template <class T>
  bool get_n(T *v, size_t n) { return n == 0 || fread(v, sizeof(T), n, f) == n; }
};

// the fixed part of a subdomain that a saved state must match
struct Header {
  char magic[8];
  int32_t nx, ny, nz, per;
  uint64_t N, pop_elems, types;
  double tau[2], G, Gads[2], rho_major, rho_minor, rho_out;
};

Header header_of(const lbm_throat *h) {
  Header H;
  std::memset(&H, 0, sizeof H);
  std::memcpy(H.magic, kMagic, sizeof kMagic);
  H.nx = h->nx;
  H.ny = h->ny;
  H.nz = h->nz;
  H.per = h->per;
  H.N = h->N;
  H.pop_elems = sc::brick_elems(h->nx, h->ny, h->nz);
  H.types = types_hash(h->types);
  H.tau[0] = h->tau[0];
  H.tau[1] = h->tau[1];
  H.G = h->G;
  H.Gads[0] = h->Gads[0];
  H.Gads[1] = h->Gads[1];
  H.rho_major = h->rho_major;
  H.rho_minor = h->rho_minor;
  H.rho_out = h->rho_out;
  return H;
}

bool put_ramp(File &F, const HostRamp &R) {
  const int32_t n = (int32_t)R.pc.size();
  bool ok = F.put((int32_t)R.phase) && F.put((int32_t)R.point) && F.put(n) && F.put(R.c.tol) &&
            F.put((int32_t)R.c.check_every) && F.put((int64_t)R.c.max_steps) &&
            F.put(R.c.bisect_rel) && F.put((int64_t)R.run_steps) && F.put(R.S_old) &&
            F.put(R.stable_pc) && F.put(R.lo) && F.put(R.hi) && F.put(R.mid) &&
            F.put(R.main_rho_in) && F.put((int32_t)R.inv_at) && F.put((int32_t)R.n_bisect) &&
            F.put((int32_t)R.runs) && F.put((int32_t)R.warn) && F.put((int32_t)R.failed) &&
            F.put((int64_t)R.total);
  ok = ok && F.put_n(R.pc.data(), n) && F.put_n(R.S.data(), n);
  for (int i = 0; ok && i < n; ++i) ok = F.put((int64_t)R.steps[i]) && F.put((int32_t)R.status[i]);
  return ok;
}

bool get_ramp(File &F, HostRamp &R) {
  int32_t phase, point, n, every, inv_at, n_bis, runs, warn, failed;
  int64_t max_steps, run_steps, total;
  bool ok = F.get(phase) && F.get(point) && F.get(n) && F.get(R.c.tol) && F.get(every) &&
            F.get(max_steps) && F.get(R.c.bisect_rel) && F.get(run_steps) && F.get(R.S_old) &&
            F.get(R.stable_pc) && F.get(R.lo) && F.get(R.hi) && F.get(R.mid) &&
            F.get(R.main_rho_in) && F.get(inv_at) && F.get(n_bis) && F.get(runs) && F.get(warn) &&
            F.get(failed) && F.get(total);
  if (!ok || n < 0 || n > (1 << 24) || phase < HostRamp::kIdle || phase > HostRamp::kDone)
    return false;
  R.phase = phase;
  R.point = point;
  R.c.check_every = every;
  R.c.max_steps = max_steps;
  R.run_steps = run_steps;
  R.inv_at = inv_at;
  R.n_bisect = n_bis;
  R.runs = runs;
  R.warn = warn;
  R.failed = failed;
  R.total = total;
  R.pc.resize(n);
  R.S.resize(n);
  R.steps.resize(n);
  R.status.resize(n);
  ok = F.get_n(R.pc.data(), n) && F.get_n(R.S.data(), n);
  for (int i = 0; ok && i < n; ++i) {
    int64_t st64 = 0;
    int32_t st32 = 0;
    ok = F.get(st64) && F.get(st32);
    R.steps[i] = st64;
    R.status[i] = st32;
  }
  return ok && (R.phase == HostRamp::kIdle || (n >= 1 && point >= 0 && point <= n));
}

// Staging of the file layout, n floats a chunk: the population buffer that does
// not hold the state, so that saving and loading ask for no device memory.  One
// shorter than kMinStage (a few nodes in a large box, whose chunks would be
// launches of a few floats) gives way to kMinStage floats of memory where they
// can be had.
constexpr size_t kMinStage = (size_t)1 << 20;
struct Staging {
  float *d = nullptr, *mine = nullptr;
  size_t n = 0;
  Staging(const lbm_throat *h, size_t total) : n(std::min(total, kIoChunk)) {
    if (h->n_live == 0) return;
    const size_t idle = sc::pop_elems(h->n_numbers);
    if (idle < std::min(n, kMinStage)) {
      n = std::min(n, kMinStage);
      if (hipMalloc((void **)&mine, sizeof(float) * n) == hipSuccess) {
        d = mine;
        return;
      }
      mine = nullptr;
      (void)hipGetLastError();
    }
    n = std::min(n, idle);
    d = h->g[1 - h->cur];
  }
  Staging(const Staging &) = delete;
  Staging &operator=(const Staging &) = delete;
  ~Staging() {
    if (mine) (void)hipFree(mine);
  }
};

// One population buffer to or from the file (file_elems floats), in chunks.  The
// file gets zeros wherever there is no node: a buffer in bricks is in the file's
// order, but what it holds there is never written.
int buffer_out(lbm_throat *h, File &F, const Staging &S, const float *dev, size_t n) {
  std::vector<float> tmp(S.n);
  const sc::Dom d = dom(h, nullptr, nullptr);
  for (size_t o = 0; o < n; o += S.n) {
    const size_t k = std::min(S.n, n - o);
    if (S.d) HIPCHK(sc::launch_to_file(d, dev, o, k, S.d, h->stream));
    if (S.d) {
      HIPCHK(hipMemcpyAsync(tmp.data(), S.d, sizeof(float) * k, hipMemcpyDeviceToHost, h->stream));
      HIPCHK(hipStreamSynchronize(h->stream));
    }
    if (!F.put_n(tmp.data(), k)) {
      set_err("lbm_save: write failed");
      return LBM_EIO;
    }
  }
  return LBM_OK;
}

int buffer_in(lbm_throat *h, File &F, const Staging &S, float *dev, size_t n) {
  std::vector<float> tmp(S.n);
  const sc::Dom d = dom(h, nullptr, nullptr);
  for (size_t o = 0; o < n; o += S.n) {
    const size_t k = std::min(S.n, n - o);
    if (!F.get_n(tmp.data(), k)) {
      set_err("lbm_load: the file ends inside a population buffer");
      return LBM_EIO;
    }
    if (!S.d) continue;
    HIPCHK(hipMemcpyAsync(h->bricks ? dev + o : S.d, tmp.data(), sizeof(float) * k,
                          hipMemcpyHostToDevice, h->stream));
    if (!h->bricks) HIPCHK(sc::launch_from_file(d, S.d, o, k, dev, h->stream));
    HIPCHK(hipStreamSynchronize(h->stream));
  }
  return LBM_OK;
}

}  // namespace

extern "C" {

int lbm_save(lbm_throat_t h, const char *path) {
  if (!h || !path) {
    set_err("lbm_save: NULL argument");
    return LBM_EINVAL;
  }
  HIPCHK(hipStreamSynchronize(h->stream));
  const size_t n = sc::brick_elems(h->nx, h->ny, h->nz);
  const Staging stage(h, n);
  File F;
  F.f = fopen(path, "wb");
  if (!F.f) {
    set_err("lbm_save: cannot open %s for writing", path);
    return LBM_EIO;
  }
  const Header H = header_of(h);
  const bool with_ckpt = h->ramp.phase == HostRamp::kRamp || h->ramp.phase == HostRamp::kBisect;
  const int32_t nbuf = with_ckpt ? 3 : 1;
  if (!F.put(H) || !F.put(h->rho_in) || !F.put((int64_t)h->steps_done) || !put_ramp(F, h->ramp) ||
      !F.put(nbuf)) {
    set_err("lbm_save: write to %s failed", path);
    return LBM_EIO;
  }
  TRY(buffer_out(h, F, stage, h->g[h->cur], n));
  if (with_ckpt) {
    TRY(buffer_out(h, F, stage, h->save[0], n));
    TRY(buffer_out(h, F, stage, h->save[1], n));
  }
  if (fflush(F.f) != 0) {
    set_err("lbm_save: write to %s failed", path);
    return LBM_EIO;
  }
  return LBM_OK;
}

int lbm_load(lbm_throat_t h, const char *path) {
  if (!h || !path) {
    set_err("lbm_load: NULL argument");
    return LBM_EINVAL;
  }
  File F;
  F.f = fopen(path, "rb");
  if (!F.f) {
    set_err("lbm_load: cannot open %s", path);
    return LBM_EIO;
  }
  Header H{};
  double rho_in = 0.0;
  int64_t steps_done = 0;
  HostRamp R;
  int32_t nbuf = 0;
  if (!F.get(H) || std::memcmp(H.magic, kMagic, sizeof kMagic) != 0) {
    set_err("lbm_load: %s is not a saved subdomain state", path);
    return LBM_EINVAL;
  }
  const Header mine = header_of(h);
  if (std::memcmp(&H, &mine, sizeof H) != 0) {
    set_err("lbm_load: %s holds the state of another subdomain (size, node classes or "
            "parameters differ)", path);
    return LBM_EINVAL;
  }
  if (!F.get(rho_in) || !F.get(steps_done) || !get_ramp(F, R) || !F.get(nbuf) ||
      !(nbuf == 1 || nbuf == 3) || !finite_pos(rho_in)) {
    set_err("lbm_load: %s is truncated or corrupt", path);
    return LBM_EINVAL;
  }
  // a ramp in progress must carry settings lbm_drain_begin would accept
  if (R.phase != HostRamp::kIdle &&
      (check_drain_args(h, R.pc.data(), (int)R.pc.size(), &R.c, "lbm_load") != LBM_OK ||
       !(R.phase == HostRamp::kDone || R.point < (int)R.pc.size()))) {
    set_err("lbm_load: %s holds a drainage ramp with invalid settings (corrupt file)", path);
    return LBM_EINVAL;
  }
  if ((nbuf == 3) != (R.phase == HostRamp::kRamp || R.phase == HostRamp::kBisect)) {
    set_err("lbm_load: %s is truncated or corrupt", path);
    return LBM_EINVAL;
  }
  if (nbuf == 3) TRY(ensure_checkpoints(h, "lbm_load"));
  const size_t n = sc::brick_elems(h->nx, h->ny, h->nz);
  const Staging stage(h, n);
  // from here on the handle's state is overwritten
  TRY(buffer_in(h, F, stage, h->g[h->cur], n));
  if (nbuf == 3) {
    TRY(buffer_in(h, F, stage, h->save[0], n));
    TRY(buffer_in(h, F, stage, h->save[1], n));
  }
  TRY(set_rho_in(h, rho_in));
  h->steps_done = steps_done;
  h->ramp = std::move(R);
  HIPCHK(hipStreamSynchronize(h->stream));
  return LBM_OK;
}

int lbm_time_steps(lbm_throat_t h, long long nsteps, double *ms) {
  if (!h || nsteps < 0 || !ms) {
    set_err("lbm_time_steps: bad argument");
    return LBM_EINVAL;
  }
  HIPCHK(hipEventRecord(h->ev[0], h->stream));
  TRY(run_steps(h, nsteps));
  HIPCHK(hipEventRecord(h->ev[1], h->stream));
  HIPCHK(hipEventSynchronize(h->ev[1]));
  float t = 0.f;
  HIPCHK(hipEventElapsedTime(&t, h->ev[0], h->ev[1]));
  *ms = t;
  return LBM_OK;
}

int lbm_step_timer(lbm_throat_t h, int enable, double *total_ms, long long *launches) {
  if (!h) {
    set_err("NULL handle");
    return LBM_EINVAL;
  }
  if (total_ms) *total_ms = h->timed_ms;
  if (launches) *launches = h->timed_launches;
  if (enable >= 0) {
    h->timing = enable != 0;
    h->timed_ms = 0.0;
    h->timed_launches = 0;
  }
  return LBM_OK;
}

int lbm_set_schedule(lbm_throat_t h, int tx, int ty, int lz) {
  if (!h) {
    set_err("NULL handle");
    return LBM_EINVAL;
  }
  sc::Sched s = h->sched;
  if (tx == sc::kListTx) {
    s = sc::Sched{sc::kListTx, 0, 0};
  } else {
    if (s.tx == sc::kListTx) s = sc::Sched{64, 4, 16};  // kept values of a list schedule
    if (tx) s.tx = tx;
    if (ty) s.ty = ty;
    if (lz) s.lz = lz;
  }
  if (!sc::schedule_valid(s)) {
    set_err("schedule (%d, %d, %d) not supported", s.tx, s.ty, s.lz);
    return LBM_EINVAL;
  }
  return set_shape(h, s);
}

int lbm_autotune(lbm_throat_t h, int trial_steps, int *tx, int *ty, int *lz) {
  if (!h || trial_steps < 1) {
    set_err("lbm_autotune: bad handle or trial_steps < 1");
    return LBM_EINVAL;
  }
  if (!own_bricks(h)) {  // nothing to choose from
    TRY(set_shape(h, sc::Sched{sc::kListTx, 0, 0}));
    if (tx) *tx = h->sched.tx;
    if (ty) *ty = h->sched.ty;
    if (lz) *lz = h->sched.lz;
    return LBM_OK;
  }
  if (!h->bricks) TRY(set_shape(h, default_schedule(h->nx, h->ny, h->nz)));
  // Trials advance the state with alternating buffers, as the ramp does (a
  // trial that re-reads one unchanged buffer times some shapes faster than
  // they run), from a copy of g[cur] that is put back at the end, also on an
  // error path.  Every candidate runs an even number of steps, so the newest
  // state stays in g[cur].  The close candidates are timed a second time and
  // keep their faster time, so that a slow first pass (clocks, caches) does
  // not decide between shapes a few per cent apart.
  struct Keep {
    lbm_throat *h;
    float *d = nullptr;
    size_t bytes = 0;
    ~Keep() {
      if (!d) return;
      (void)hipMemcpyAsync(h->g[h->cur], d, bytes, hipMemcpyDeviceToDevice, h->stream);
      (void)hipStreamSynchronize(h->stream);
      (void)hipFree(d);
    }
  } keep{h};
  keep.bytes = sizeof(float) * sc::pop_elems(h->n_numbers);
  if (hipMalloc((void **)&keep.d, keep.bytes) != hipSuccess) {
    keep.d = nullptr;
    set_err("lbm_autotune: hipMalloc of %zu bytes for the state copy failed", keep.bytes);
    return LBM_ENOMEM;
  }
  HIPCHK(hipMemcpyAsync(keep.d, h->g[h->cur], keep.bytes, hipMemcpyDeviceToDevice, h->stream));
  static const int lzs[8] = {1, 2, 4, 8, 16, 32, 64, 128};
  std::vector<sc::Sched> cand;
  for (const auto &sh : sc::kShapes)
    for (int l : lzs)
      if (l <= h->nz) cand.push_back(sc::Sched{sh[0], sh[1], l});
  cand.push_back(default_schedule(h->nx, h->ny, h->nz));
  std::vector<double> t(cand.size(), INFINITY);
  auto trial = [&](size_t c) -> int {
    TRY(set_shape(h, cand[c]));
    int par = h->cur;
    auto one = [&]() {
      const hipError_t e = one_step(h, par);
      par ^= 1;
      return e;
    };
    for (int w = 0; w < 2; ++w) HIPCHK(one());
    HIPCHK(hipEventRecord(h->ev[0], h->stream));
    for (int i = 0; i < trial_steps; ++i) HIPCHK(one());
    HIPCHK(hipEventRecord(h->ev[1], h->stream));
    if (trial_steps & 1) HIPCHK(one());
    HIPCHK(hipEventSynchronize(h->ev[1]));
    float ms = 0.f;
    HIPCHK(hipEventElapsedTime(&ms, h->ev[0], h->ev[1]));
    t[c] = std::min(t[c], (double)ms);
    return LBM_OK;
  };
  // first round: per tile shape in increasing lz, stop once a segment length
  // is 1.5x slower than the shape's best (longer ones only lengthen the
  // serial z-march); second round: the candidates within 1.25x of the best
  for (size_t c = 0; c < cand.size();) {
    double shape_best = INFINITY;
    size_t e = c;
    while (e < cand.size() && cand[e].tx == cand[c].tx && cand[e].ty == cand[c].ty) ++e;
    for (size_t k = c; k < e; ++k) {
      TRY(trial(k));
      if (t[k] > 1.5 * shape_best) break;
      shape_best = std::min(shape_best, t[k]);
    }
    c = e;
  }
  const double first = *std::min_element(t.begin(), t.end());
  for (size_t c = 0; c < cand.size(); ++c)
    if (t[c] <= 1.25 * first) TRY(trial(c));
  size_t best = 0;
  for (size_t c = 1; c < cand.size(); ++c)
    if (t[c] < t[best]) best = c;
  TRY(set_shape(h, cand[best]));
  if (tx) *tx = h->sched.tx;
  if (ty) *ty = h->sched.ty;
  if (lz) *lz = h->sched.lz;
  return LBM_OK;
}

int lbm_place(lbm_throat_t h, int tries, int trial_steps, double *ms_first, double *ms_best) {
  if (!h || tries < 0 || tries > 8 || trial_steps < 1) {
    set_err("lbm_place: bad handle, tries outside 0..8 or trial_steps < 1");
    return LBM_EINVAL;
  }
  const size_t bytes = sizeof(float) * sc::pop_elems(h->n_numbers);
  TRY(lbmh::check_budget(sizeof(float) * sc::brick_elems(h->nx, h->ny, h->nz) *
                             (1 + 2 * (size_t)tries),
                         "lbm_place"));
  // The state is kept in a copy; each placement (the current pair, then
  // `tries` new pairs allocated while the earlier ones are still held, so
  // that they land elsewhere) runs 2 + trial_steps steps from that copy with
  // alternating buffers, timed with events; the fastest pair gets the copy
  // back and the others are freed, also on an error path.
  struct Pair {
    float *g[2] = {nullptr, nullptr};
  };
  struct Work {
    lbm_throat *h;
    float *keep = nullptr;
    size_t bytes = 0;
    Pair orig;
    std::vector<Pair> cand;
    int chosen = -1;  // -1: the original pair
    ~Work() {
      // the handle keeps the chosen pair; the copy goes back into it
      if (chosen >= 0) {
        h->g[0] = cand[chosen].g[0];
        h->g[1] = cand[chosen].g[1];
        h->cur = 0;
      } else {
        h->g[0] = orig.g[0];
        h->g[1] = orig.g[1];
      }
      if (keep)
        (void)hipMemcpyAsync(h->g[h->cur], keep, bytes, hipMemcpyDeviceToDevice, h->stream);
      (void)sync_desc(h);
      (void)hipStreamSynchronize(h->stream);
      for (int i = 0; i < (int)cand.size(); ++i)
        if (i != chosen)
          for (float *b : cand[i].g)
            if (b) (void)hipFree(b);
      if (chosen >= 0)
        for (float *b : orig.g) (void)hipFree(b);
      if (keep) (void)hipFree(keep);
    }
  } w{h};
  w.bytes = bytes;
  w.orig.g[0] = h->g[0];
  w.orig.g[1] = h->g[1];
  if (hipMalloc((void **)&w.keep, bytes) != hipSuccess) {
    w.keep = nullptr;
    set_err("lbm_place: hipMalloc of %zu bytes for the state copy failed", bytes);
    return LBM_ENOMEM;
  }
  HIPCHK(hipMemcpyAsync(w.keep, h->g[h->cur], bytes, hipMemcpyDeviceToDevice, h->stream));
  const int state0 = h->cur;
  auto timed = [&](const Pair &pr, int parity, double *ms) -> int {
    h->g[0] = pr.g[0];
    h->g[1] = pr.g[1];
    TRY(sync_desc(h));
    HIPCHK(hipMemcpyAsync(pr.g[parity], w.keep, bytes, hipMemcpyDeviceToDevice, h->stream));
    int par = parity;
    auto one = [&]() {
      const hipError_t e = one_step(h, par);
      par ^= 1;
      return e;
    };
    for (int i = 0; i < 2; ++i) HIPCHK(one());
    HIPCHK(hipEventRecord(h->ev[0], h->stream));
    for (int i = 0; i < trial_steps; ++i) HIPCHK(one());
    HIPCHK(hipEventRecord(h->ev[1], h->stream));
    HIPCHK(hipEventSynchronize(h->ev[1]));
    float t = 0.f;
    HIPCHK(hipEventElapsedTime(&t, h->ev[0], h->ev[1]));
    *ms = (double)t / trial_steps;
    return LBM_OK;
  };
  double best = 0.0;
  TRY(timed(w.orig, state0, &best));
  const double first = best;
  for (int k = 0; k < tries; ++k) {
    Pair pr;
    if (hipMalloc((void **)&pr.g[0], bytes) != hipSuccess ||
        hipMalloc((void **)&pr.g[1], bytes) != hipSuccess) {
      (void)hipGetLastError();
      if (pr.g[0]) (void)hipFree(pr.g[0]);
      break;  // no room for another placement: keep the best so far
    }
    w.cand.push_back(pr);
    double t = 0.0;
    TRY(timed(pr, 0, &t));
    if (t < best) {
      best = t;
      w.chosen = (int)w.cand.size() - 1;
    }
  }
  if (w.chosen < 0) h->cur = state0;
  if (ms_first) *ms_first = first;
  if (ms_best) *ms_best = best;
  return LBM_OK;
}

int lbm_get_schedule(lbm_throat_t h, int *tx, int *ty, int *lz) {
  if (!h) {
    set_err("NULL handle");
    return LBM_EINVAL;
  }
  if (tx) *tx = h->sched.tx;
  if (ty) *ty = h->sched.ty;
  if (lz) *lz = h->sched.lz;
  return LBM_OK;
}

int lbm_bw_probe(size_t bytes, int reps, double *gbps) {
  if (bytes < (1u << 20) || reps < 1 || !gbps) {
    set_err("lbm_bw_probe: bytes >= 1 MiB, reps >= 1 and an output are required");
    return LBM_EINVAL;
  }
  const size_t nf = bytes / 16 * 4;
  float *a = nullptr, *b = nullptr;
  hipEvent_t e0 = nullptr, e1 = nullptr;
  int rc = LBM_OK;
  if (hipMalloc((void **)&a, nf * sizeof(float)) != hipSuccess ||
      hipMalloc((void **)&b, nf * sizeof(float)) != hipSuccess) {
    set_err("lbm_bw_probe: hipMalloc of 2 x %zu bytes failed", nf * sizeof(float));
    rc = LBM_ENOMEM;
  }
  if (rc == LBM_OK && (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess ||
                       hipMemset(a, 0, nf * sizeof(float)) != hipSuccess)) {
    set_err("lbm_bw_probe: setup failed");
    rc = LBM_EHIP;
  }
  if (rc == LBM_OK) {
    hipError_t e = sc::launch_copy(a, b, nf, nullptr);  // warm-up
    if (e == hipSuccess) e = hipEventRecord(e0, nullptr);
    for (int i = 0; i < reps && e == hipSuccess; ++i) e = sc::launch_copy(a, b, nf, nullptr);
    if (e == hipSuccess) e = hipEventRecord(e1, nullptr);
    if (e == hipSuccess) e = hipEventSynchronize(e1);
    float ms = 0.f;
    if (e == hipSuccess) e = hipEventElapsedTime(&ms, e0, e1);
    if (e != hipSuccess) {
      set_err("lbm_bw_probe: %s", hipGetErrorString(e));
      rc = LBM_EHIP;
    } else {
      *gbps = 2.0 * (double)nf * sizeof(float) * reps / (ms * 1e-3) / 1e9;
    }
  }
  if (e0) (void)hipEventDestroy(e0);
  if (e1) (void)hipEventDestroy(e1);
  if (a) (void)hipFree(a);
  if (b) (void)hipFree(b);
  return rc;
}

}  // extern "C"
