// lbm_batch.cpp -- batched drainage of many pore-throat subdomains
// (Montella et al., Sec. 2.2.2: the pore throats are solved independently).
//
// Every subdomain keeps its own buffers and node classes; one step
// covers the nodes of all active subdomains, and the ramp /
// bisection decisions of every subdomain are taken on the device between
// chunks of `check_every` steps.  The chunk [steps, reduction, decisions,
// state copies] is captured once as a HIP graph and replayed until no
// subdomain is running; the host only reads one counter between replays.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <memory>
#include <new>
#include <vector>

#include "lbm_abi.h"
#include "lbm_handle.h"
#include "sc_internal.h"

using lbmh::set_err;

namespace {

constexpr double kCs2 = 1.0 / 3.0;

struct Batch {
  int n = 0;
  hipStream_t stream = nullptr;
  std::vector<std::unique_ptr<lbm_throat>> h;  // their buffers lie in geo_d and mem_d
  char *geo_d = nullptr, *mem_d = nullptr;     // all device memory of the batch,
  char *rho_d = nullptr;                       // besides given initial states
  char *geo_h = nullptr, *mem_h = nullptr;     // pinned images of their exchanged parts
  sc::Throat *th_d = nullptr;
  sc::TileRef *items_d = nullptr;   // work items of the subdomains in two passes
  int nitems = 0;
  sc::TileRef *tiles_d = nullptr;   // tiles of those in bricks, at one shape
  int ntiles = 0;
  sc::Sched tiles{sc::kListTx, 0, 0};
  int *zper_d = nullptr;            // those in bricks that are periodic in z
  int n_zper = 0;
  bool wide = false;
  sc::RedChunk *chunks_d = nullptr;  // reduction chunks of all subdomains
  int nchunks = 0;
  sc::Chunk *cchunks_d = nullptr;  // ranges of the checkpoint copies
  int ncchunks = 0;
  int *first_d = nullptr, *count_d = nullptr;
  sc::RedInfo *info_d = nullptr;
  double *partials = nullptr, *sums = nullptr, *probe = nullptr;
  sc::Ckpt *ck_d = nullptr;
  double *pc_d = nullptr;
  // results, contiguous on the device and in the pinned image
  size_t res_lo = 0, res_hi = 0;
  sc::RampDev *rd_d = nullptr, *rd = nullptr;
  double *S_d = nullptr, *S = nullptr;
  long long *steps_d = nullptr, *steps = nullptr;
  int *status_d = nullptr, *status = nullptr;
  int *nact_d = nullptr, *nact_h = nullptr;
  hipGraph_t graph = nullptr;
  hipGraphExec_t exec = nullptr;
  hipEvent_t wall[2] = {nullptr, nullptr};  // the whole drain, first to last kernel

  ~Batch() {
    // an error return can leave replays queued: let them finish before any
    // graph, buffer or handle they use is released
    if (stream) (void)hipStreamSynchronize(stream);
    if (exec) (void)hipGraphExecDestroy(exec);
    if (graph) (void)hipGraphDestroy(graph);
    for (char *p : {geo_d, mem_d, rho_d})
      if (p) (void)hipFree(p);
    for (char *p : {geo_h, mem_h})
      if (p) (void)hipHostFree(p);
    for (auto e : wall)
      if (e) (void)hipEventDestroy(e);
    if (stream) (void)hipStreamDestroy(stream);
  }
};

// places of arrays in one block of memory
struct Layout {
  size_t size = 0;
  size_t add(size_t bytes, size_t align = 256) {
    const size_t at = (size + align - 1) / align * align;
    size = at + bytes;
    return at;
  }
};

#define BCHK(call)                                                             \
  do {                                                                         \
    hipError_t e_ = (call);                                                    \
    if (e_ != hipSuccess) {                                                    \
      set_err("%s failed: %s", #call, hipGetErrorString(e_));                  \
      return LBM_EHIP;                                                         \
    }                                                                          \
  } while (0)

int block(char **d, size_t bytes) {
  if (hipMalloc((void **)d, bytes) == hipSuccess) return LBM_OK;
  *d = nullptr;
  (void)hipGetLastError();
  set_err("lbm_drain_batch: hipMalloc of %zu bytes failed", bytes);
  return LBM_ENOMEM;
}

int pinned(char **h, size_t bytes) {
  if (hipHostMalloc((void **)h, bytes, hipHostMallocDefault) == hipSuccess) return LBM_OK;
  *h = nullptr;
  (void)hipGetLastError();
  set_err("lbm_drain_batch: hipHostMalloc of %zu bytes failed", bytes);
  return LBM_ENOMEM;
}

// Geometry, numbering, initial state and ramp tables of all subdomains, in two
// rounds of one upload, the kernels and one wait each: the second block can be
// laid out only when the nodes are counted.  Set up one by one, with an
// allocation and a release per array and a wait per copy, 16 throats of 24 to
// 36 nodes a side took 34 ms for a batch of which 17 are kernels; now 19.8.
int setup(Batch &B, const lbm_params *p, const double *pc, int n_pc) {
  const int n = B.n;
  struct At {
    size_t sph, start, ids, rows, types, map;
  };
  std::vector<At> at(n);
  std::vector<lbmh::Geometry> geo;
  geo.reserve(n);
  B.h.resize(n);
  Layout G;
  for (int t = 0; t < n; ++t) {
    B.h[t].reset(new (std::nothrow) lbm_throat());
    if (!B.h[t]) {
      set_err("host allocation failed");
      return LBM_ENOMEM;
    }
    if (const int r = lbmh::describe(&p[t], B.h[t].get())) return r;
    B.h[t]->stream = B.stream;
    if (p[t].probe[0] >= p[t].nx || p[t].probe[1] < 0 || p[t].probe[1] >= p[t].ny ||
        p[t].probe[2] < 0 || p[t].probe[2] >= p[t].nz) {
      set_err("probe node outside the box");
      return LBM_EINVAL;
    }
    geo.emplace_back(p[t]);
    at[t].sph = G.add(sizeof(double) * geo[t].sph.size(), 16);
    at[t].start = G.add(sizeof(int) * geo[t].bin_start.size(), 16);
    at[t].ids = G.add(sizeof(int) * geo[t].bin_ids.size(), 16);
  }
  const size_t up = G.size, rows_lo = G.add(0);
  for (int t = 0; t < n; ++t)
    at[t].rows = G.add(sizeof(uint32_t) * (size_t)p[t].ny * p[t].nz, 16);
  const size_t rows_hi = G.size;
  for (int t = 0; t < n; ++t) {
    at[t].types = G.add(B.h[t]->N);
    at[t].map = G.add(sizeof(uint32_t) * sc::map_elems(p[t].nx, p[t].ny, p[t].nz));
  }
  if (const int r = block(&B.geo_d, G.size)) return r;
  if (const int r = pinned(&B.geo_h, rows_hi)) return r;
  for (int t = 0; t < n; ++t) {
    auto put = [&](size_t o, const auto &v) {
      std::memcpy(B.geo_h + o, v.data(), sizeof(v[0]) * v.size());
    };
    put(at[t].sph, geo[t].sph);
    put(at[t].start, geo[t].bin_start);
    put(at[t].ids, geo[t].bin_ids);
  }
  BCHK(hipMemcpyAsync(B.geo_d, B.geo_h, up, hipMemcpyHostToDevice, B.stream));
  for (int t = 0; t < n; ++t) {
    lbm_throat &h = *B.h[t];
    h.types_d = (uint8_t *)(B.geo_d + at[t].types);
    h.map_d = (uint32_t *)(B.geo_d + at[t].map);
    BCHK(geo[t].voxelize(p[t], (double *)(B.geo_d + at[t].sph), (int *)(B.geo_d + at[t].start),
                         (int *)(B.geo_d + at[t].ids), h.types_d, B.stream));
    BCHK(sc::launch_row_counts(h.types_d, h.nx, h.ny, h.nz, (uint32_t *)(B.geo_d + at[t].rows),
                               B.stream));
  }
  BCHK(hipMemcpyAsync(B.geo_h + rows_lo, B.geo_d + rows_lo, rows_hi - rows_lo,
                      hipMemcpyDeviceToHost, B.stream));
  BCHK(hipStreamSynchronize(B.stream));

  // Numbers and work items.  Open boxes go into bricks by the rule of a single
  // subdomain, their sizes taken together, as one launch of tiles steps them all.
  // us a step, checks included, tiles / two passes (tuned tiles over the whole
  // box, before the compact numbering): 256^3 1173 / 1518 (1357), three 192^3
  // 1589 / 1929 (1727), eight 128^3 1118 / 1506 (1281), sixty-four 64^3 1139 /
  // 1463 (1238); just at kTileNodes, eight 64^3 0.89, sixty-four 32^3 0.84 of the
  // two passes.
  std::vector<int> first(n), count(n), zper;
  std::vector<sc::TileRef> items, tiles;
  std::vector<lbm_throat *> open;
  std::vector<sc::RedChunk> chunks;
  std::vector<sc::Chunk> cchunks;
  for (int t = 0; t < n; ++t) {
    lbm_throat &h = *B.h[t];
    uint32_t *rows = (uint32_t *)(B.geo_h + at[t].rows);
    long long baths = 0;
    if (h.bc[2] == LBM_BC_RESERVOIR)
      for (int y = 0; y < h.ny; ++y)
        baths += (long long)rows[y] + rows[(size_t)(h.nz - 1) * h.ny + y];
    h.n_live = sc::number_rows(rows, h.ny, h.nz);
    h.n_fluid = (long long)h.n_live - baths;
    if (lbmh::fills_tiles(&h)) open.push_back(&h);
  }
  size_t slots = 0;
  for (const lbm_throat *h : open) slots += lbmh::brick_slots(h);
  if (slots < lbmh::kTileNodes) open.clear();
  for (lbm_throat *h : open) {
    h->bricks = true;
    h->types.resize(h->N);
    BCHK(hipMemcpyAsync(h->types.data(), h->types_d, h->N, hipMemcpyDeviceToHost, B.stream));
  }
  if (!open.empty()) {
    BCHK(hipStreamSynchronize(B.stream));
    B.tiles = lbmh::batch_tiles(open);
  }
  for (int t = 0; t < n; ++t) {
    lbm_throat &h = *B.h[t];
    h.n_numbers = h.bricks ? lbmh::brick_numbers(&h) : h.n_live;
    first[t] = (int)chunks.size();
    sc::red_chunks(h.n_live, t, chunks);
    count[t] = (int)chunks.size() - first[t];
    sc::copy_chunks(t, sc::pop_elems(h.n_numbers), cchunks);
    if (h.bricks) {
      sc::brick_map(h.types.data(), h.nx, h.ny, h.nz, h.brick_live);
      sc::list_tiles(h.brick_live.data(), h.nx, h.ny, h.nz, h.sched.tx, sc::tile_rows(h.sched.ty),
                     h.sched.lz, t, tiles);
      if (h.per & 4) zper.push_back(t);
    } else {
      sc::list_items(h.n_live, t, items);
      B.wide = B.wide || lbmh::wide(&h);
    }
  }
  if (items.size() + tiles.size() > (size_t)INT_MAX) {
    set_err("lbm_drain_batch: %zu work items exceed one launch", items.size() + tiles.size());
    return LBM_EINVAL;
  }
  B.nitems = (int)items.size();
  B.ntiles = (int)tiles.size();
  B.n_zper = (int)zper.size();
  B.nchunks = (int)chunks.size();
  B.ncchunks = (int)cchunks.size();
  const size_t points = (size_t)n * n_pc;
  Layout M;
  const size_t o_th = M.add(sizeof(sc::Throat) * n),
               o_items = M.add(sizeof(sc::TileRef) * items.size()),
               o_tiles = M.add(sizeof(sc::TileRef) * tiles.size()),
               o_zper = M.add(sizeof(int) * zper.size()),
               o_chunks = M.add(sizeof(sc::RedChunk) * chunks.size()),
               o_cchunks = M.add(sizeof(sc::Chunk) * cchunks.size()),
               o_first = M.add(sizeof(int) * n), o_count = M.add(sizeof(int) * n),
               o_info = M.add(sizeof(sc::RedInfo) * n), o_ck = M.add(sizeof(sc::Ckpt) * n),
               o_pc = M.add(sizeof(double) * points), o_rres = M.add(sizeof(double) * 4 * n),
               o_rd = M.add(sizeof(sc::RampDev) * n), o_S = M.add(sizeof(double) * points),
               o_steps = M.add(sizeof(long long) * points), o_status = M.add(sizeof(int) * points);
  B.res_lo = o_rd;
  B.res_hi = M.size;
  const size_t o_nact = M.add(sizeof(int)), o_bad = M.add(sizeof(unsigned long long) * n),
               image = M.size;
  const size_t o_partials = M.add(sizeof(double) * 3 * std::max<size_t>(chunks.size(), 1)),
               o_sums = M.add(sizeof(double) * 3 * n), o_probe = M.add(sizeof(double) * 2 * n);
  std::vector<size_t> o_pos(n), o_side(n), o_pop[4];
  for (int t = 0; t < n; ++t) {
    const lbm_throat &h = *B.h[t];
    o_pos[t] = M.add(sizeof(uint32_t) * h.n_live);
    o_side[t] = M.add(h.bricks ? sizeof(uint32_t) * h.N : sizeof(float2) * h.n_numbers);
  }
  size_t lo[4];  // first buffers, second buffers, the two sets of checkpoints
  for (int i = 0; i < 4; ++i) {
    lo[i] = M.add(0, 4096);
    for (int t = 0; t < n; ++t)
      o_pop[i].push_back(M.add(sizeof(float) * sc::pop_elems(B.h[t]->n_numbers), 4096));
  }
  size_t free_b = 0, total_b = 0;
  BCHK(hipMemGetInfo(&free_b, &total_b));
  if (M.size + (64u << 20) > free_b) {
    set_err("needs %zu bytes of device memory, %zu free", M.size + (64u << 20), free_b);
    return LBM_ENOMEM;
  }
  if (const int r = block(&B.mem_d, M.size)) return r;
  if (const int r = pinned(&B.mem_h, image)) return r;
  std::memset(B.mem_h, 0, image);
  auto put = [&](size_t o, const auto &v) {
    if (!v.empty()) std::memcpy(B.mem_h + o, v.data(), sizeof(v[0]) * v.size());
  };
  put(o_items, items);
  put(o_tiles, tiles);
  put(o_zper, zper);
  put(o_chunks, chunks);
  put(o_cchunks, cchunks);
  put(o_first, first);
  put(o_count, count);
  std::memcpy(B.mem_h + o_pc, pc, sizeof(double) * points);
  sc::RedInfo *info = (sc::RedInfo *)(B.mem_h + o_info);
  B.rd = (sc::RampDev *)(B.mem_h + o_rd);
  B.S = (double *)(B.mem_h + o_S);
  B.steps = (long long *)(B.mem_h + o_steps);
  B.status = (int *)(B.mem_h + o_status);
  B.nact_h = (int *)(B.mem_h + o_nact);
  unsigned long long *bad = (unsigned long long *)(B.mem_h + o_bad);
  std::fill(bad, bad + n, ~0ull);
  for (size_t i = 0; i < points; ++i) B.status[i] = LBM_PT_NOT_RUN;
  for (int t = 0; t < n; ++t) {
    lbm_throat &h = *B.h[t];
    for (int i = 0; i < 2; ++i) {
      h.g[i] = (float *)(B.mem_d + o_pop[i][t]);
      h.save[i] = (float *)(B.mem_d + o_pop[2 + i][t]);
    }
    h.pos_d = (uint32_t *)(B.mem_d + o_pos[t]);
    if (h.bricks)
      h.mask_d = (uint32_t *)(B.mem_d + o_side[t]);
    else
      h.rho_d = (float2 *)(B.mem_d + o_side[t]);
    h.rres_d = (double *)(B.mem_d + o_rres) + 4 * t;
    lbmh::fill_desc(&h);
    ((sc::Throat *)(B.mem_h + o_th))[t] = h.desc;
    ((sc::Ckpt *)(B.mem_h + o_ck))[t] = sc::Ckpt{h.save[0], h.save[1]};
    info[t] = sc::RedInfo{(long long)sc::map_pos(h.nx, h.ny, p[t].probe[0], p[t].probe[1],
                                                 p[t].probe[2]),
                          h.phib};
    const double rr[4] = {h.rho_minor, h.rho_in, h.rho_out, h.rho_minor};
    std::memcpy(B.mem_h + o_rres + 4 * t * sizeof(double), rr, sizeof rr);
    sc::RampDev R{};
    R.rho_out = h.rho_out;
    R.dpc_drho = kCs2 * (1.0 + h.G * h.rho_minor);
    R.rho_ref = h.rho_minor;
    R.n_fluid = (unsigned)h.n_fluid;
    R.phase = sc::kPhaseDone;
    B.rd[t] = R;
  }
  B.th_d = (sc::Throat *)(B.mem_d + o_th);
  B.items_d = (sc::TileRef *)(B.mem_d + o_items);
  B.tiles_d = (sc::TileRef *)(B.mem_d + o_tiles);
  B.zper_d = (int *)(B.mem_d + o_zper);
  B.chunks_d = (sc::RedChunk *)(B.mem_d + o_chunks);
  B.cchunks_d = (sc::Chunk *)(B.mem_d + o_cchunks);
  B.first_d = (int *)(B.mem_d + o_first);
  B.count_d = (int *)(B.mem_d + o_count);
  B.info_d = (sc::RedInfo *)(B.mem_d + o_info);
  B.ck_d = (sc::Ckpt *)(B.mem_d + o_ck);
  B.pc_d = (double *)(B.mem_d + o_pc);
  B.rd_d = (sc::RampDev *)(B.mem_d + o_rd);
  B.S_d = (double *)(B.mem_d + o_S);
  B.steps_d = (long long *)(B.mem_d + o_steps);
  B.status_d = (int *)(B.mem_d + o_status);
  B.nact_d = (int *)(B.mem_d + o_nact);
  B.partials = (double *)(B.mem_d + o_partials);
  B.sums = (double *)(B.mem_d + o_sums);
  B.probe = (double *)(B.mem_d + o_probe);
  BCHK(hipMemcpyAsync(B.geo_d + rows_lo, B.geo_h + rows_lo, rows_hi - rows_lo,
                      hipMemcpyHostToDevice, B.stream));
  BCHK(hipMemcpyAsync(B.mem_d, B.mem_h, image, hipMemcpyHostToDevice, B.stream));
  for (int t = 0; t < n; ++t) {
    const lbm_throat &h = *B.h[t];
    BCHK(sc::launch_number(h.types_d, h.nx, h.ny, h.nz, h.per, (uint32_t *)(B.geo_d + at[t].rows),
                           h.bricks, h.map_d, h.pos_d, B.stream));
    if (h.bricks) BCHK(sc::launch_links(h.types_d, lbmh::dom(&h), h.mask_d, B.stream));
  }
  BCHK(sc::launch_probe_numbers(B.th_d, n, B.info_d, B.stream));
  BCHK(hipMemcpyAsync(info, B.info_d, sizeof(sc::RedInfo) * n, hipMemcpyDeviceToHost, B.stream));
  BCHK(hipMemsetAsync(B.mem_d + lo[1], 0, lo[2] - lo[1], B.stream));
  // given initial states pass through one buffer, in stream order
  size_t given = 0;
  for (int t = 0; t < n; ++t)
    if (p[t].rho_init) given = std::max(given, sizeof(double) * 2 * B.h[t]->N);
  if (given)
    if (const int r = block(&B.rho_d, given)) return r;
  for (int t = 0; t < n; ++t) {
    const lbm_throat &h = *B.h[t];
    if (p[t].rho_init)
      BCHK(hipMemcpyAsync(B.rho_d, p[t].rho_init, sizeof(double) * 2 * h.N, hipMemcpyHostToDevice,
                          B.stream));
    BCHK(sc::launch_init(lbmh::dom(&h), h.P, p[t].rho_init ? (const double *)B.rho_d : nullptr,
                         h.rho_major, h.rho_minor, p[t].z_front, h.rres_d, h.g[0],
                         (unsigned long long *)(B.mem_d + o_bad) + t, B.stream));
  }
  BCHK(sc::launch_ghost(B.th_d, B.zper_d, B.n_zper, 0, B.stream));
  BCHK(hipMemcpyAsync(bad, B.mem_d + o_bad, sizeof(unsigned long long) * n, hipMemcpyDeviceToHost,
                      B.stream));
  BCHK(hipStreamSynchronize(B.stream));
  for (int t = 0; t < n; ++t) {
    const lbm_throat &h = *B.h[t];
    const int z = p[t].probe[2];
    if ((uint32_t)info[t].probe == sc::kNoNode ||
        (h.bc[2] == LBM_BC_RESERVOIR && (z == 0 || z == h.nz - 1))) {
      set_err("probe node is not a fluid node");
      return LBM_EINVAL;
    }
    if (const int r = lbmh::check_rho_init(&h, bad[t])) return r;
  }
  return LBM_OK;
}

// one step of every running subdomain
hipError_t enqueue_step(Batch &B, int parity) {
  hipError_t e = hipSuccess;
  if (B.nitems)
    e = sc::launch_step(B.th_d, B.items_d, B.nitems, sc::kListTx, 0, B.wide, parity, B.stream,
                        nullptr, 0);
  if (e == hipSuccess && B.ntiles)
    e = sc::launch_step(B.th_d, B.tiles_d, B.ntiles, B.tiles.tx, B.tiles.ty, false, parity,
                        B.stream, B.zper_d, B.n_zper);
  return e;
}

// the kernels of one chunk: check_every steps, the reductions, the ramp
// decisions and the checkpoint copies they request
hipError_t enqueue_chunk(Batch &B, const sc::RampCfg &cfg) {
  hipError_t e = hipSuccess;
  for (int i = 0; i < cfg.every && e == hipSuccess; ++i)
    e = enqueue_step(B, i & 1);
  if (e == hipSuccess)
    e = sc::launch_reduce_chunks(B.th_d, B.chunks_d, B.nchunks, B.info_d, 0, B.partials, B.probe,
                                 B.stream);
  if (e == hipSuccess)
    e = sc::launch_reduce_throats(B.first_d, B.count_d, B.n, B.partials, B.sums, B.stream);
  if (e == hipSuccess)
    e = sc::launch_ramp_advance(B.th_d, B.rd_d, B.pc_d, cfg, B.sums, B.probe, B.S_d, B.steps_d,
                                B.status_d, B.n, B.nact_d, B.stream);
  if (e == hipSuccess)
    e = sc::launch_copy_requests(B.th_d, B.rd_d, B.ck_d, B.cchunks_d, B.ncchunks, 0, B.stream);
  return e;
}

int capture_chunk(Batch &B, const sc::RampCfg &cfg) {
  BCHK(hipStreamBeginCapture(B.stream, hipStreamCaptureModeThreadLocal));
  hipError_t e = enqueue_chunk(B, cfg);
  hipGraph_t g = nullptr;
  const hipError_t e2 = hipStreamEndCapture(B.stream, &g);
  if (e != hipSuccess || e2 != hipSuccess) {
    if (g) (void)hipGraphDestroy(g);
    set_err("graph capture failed: %s", hipGetErrorString(e != hipSuccess ? e : e2));
    return LBM_EHIP;
  }
  B.graph = g;
  BCHK(hipGraphInstantiate(&B.exec, g, nullptr, nullptr, 0));
  return LBM_OK;
}

}  // namespace

extern "C" {

int lbm_drain_batch(int n, const lbm_params *p, const double *pc, int n_pc, const lbm_conv *c,
                    lbm_drain_result *out, lbm_batch_info *info) {
  if (n < 1 || !p || !pc || n_pc < 1 || !c || !out) {
    set_err("lbm_drain_batch: n >= 1, params, pc, conv and results are required");
    return LBM_EINVAL;
  }
  if (!(c->tol > 0) || c->check_every < 2 || (c->check_every & 1) ||
      c->max_steps < c->check_every || !(c->bisect_rel > 0)) {
    set_err("lbm_drain_batch: tol > 0, an even check_every >= 2, max_steps >= check_every and "
            "bisect_rel > 0 are required");
    return LBM_EINVAL;
  }
  for (int t = 0; t < n; ++t) {
    if (!out[t].S || !out[t].steps || !out[t].status) {
      set_err("lbm_drain_batch: result %d has no output arrays", t);
      return LBM_EINVAL;
    }
    if (p[t].probe[0] < 0) {
      set_err("lbm_drain_batch: subdomain %d has no probe node", t);
      return LBM_EINVAL;
    }
    for (int i = 0; i < n_pc; ++i) {
      const double v = pc[(size_t)t * n_pc + i];
      if (!std::isfinite(v) || !(v > 0) || (i > 0 && !(v > pc[(size_t)t * n_pc + i - 1])) ||
          !(p[t].rho_out_w + v / (kCs2 * (1.0 + p[t].G * p[t].rho_minor)) > 0)) {
        set_err("lbm_drain_batch: pc of subdomain %d must be finite, positive, strictly "
                "increasing and give a positive inlet density", t);
        return LBM_EINVAL;
      }
    }
  }
  {
    // the whole batch's device memory against the budget, before any allocation
    size_t need = 0;
    for (int t = 0; t < n; ++t) {
      if (p[t].nx < 3 || p[t].ny < 3 || p[t].nz < 3) {
        set_err("lbm_drain_batch: subdomain %d is smaller than 3 nodes on a side", t);
        return LBM_EINVAL;
      }
      need += lbmh::subdomain_bytes(p[t].nx, p[t].ny, p[t].nz, true);
    }
    if (int r = lbmh::check_budget(need, "lbm_drain_batch")) return r;
  }
  Batch B;
  B.n = n;
  BCHK(hipStreamCreate(&B.stream));
  BCHK(hipEventCreate(&B.wall[0]));
  BCHK(hipEventCreate(&B.wall[1]));
  if (const int r = setup(B, p, pc, n_pc)) return r;
  hipEvent_t w0 = B.wall[0], w1 = B.wall[1];
  BCHK(hipEventRecord(w0, B.stream));
  // the initial decisions
  sc::RampCfg cfg{c->tol, c->bisect_rel, c->max_steps, c->check_every, n_pc};
  BCHK(sc::launch_reduce_chunks(B.th_d, B.chunks_d, B.nchunks, B.info_d, 0, B.partials, B.probe,
                                B.stream));
  BCHK(sc::launch_reduce_throats(B.first_d, B.count_d, n, B.partials, B.sums, B.stream));
  BCHK(sc::launch_ramp_begin(B.th_d, B.rd_d, B.pc_d, cfg, B.sums, n, B.stream));
  BCHK(sc::launch_copy_requests(B.th_d, B.rd_d, B.ck_d, B.cchunks_d, B.ncchunks, 0, B.stream));
  // LBM_BATCH_NO_GRAPH=1 in the environment: the same chunk launched kernel
  // by kernel instead of replayed as a graph (for tracers that do not
  // follow graph launches); results are identical
  const char *ng = std::getenv("LBM_BATCH_NO_GRAPH");
  const bool use_graph = !(ng && ng[0] == '1');
  if (use_graph)
    if (int r = capture_chunk(B, cfg)) return r;
  // replay until every subdomain has finished its ramp; a bound on the
  // replays guards against a run that would never end
  const long long max_bisect = sc::kMaxBisect;
  const long long max_replays =
      (long long)(n_pc + max_bisect + 2) * ((c->max_steps + c->check_every - 1) / c->check_every) +
      16;
  long long replays = 0;
  const int poll = 4;
  for (;;) {
    for (int i = 0; i < poll; ++i) {
      if (use_graph)
        BCHK(hipGraphLaunch(B.exec, B.stream));
      else
        BCHK(enqueue_chunk(B, cfg));
    }
    replays += poll;
    BCHK(hipMemcpyAsync(B.nact_h, B.nact_d, sizeof(int), hipMemcpyDeviceToHost, B.stream));
    BCHK(hipStreamSynchronize(B.stream));
    if (*B.nact_h == 0) break;
    if (replays > max_replays) {
      set_err("lbm_drain_batch: ramp did not finish within %lld chunk replays", replays);
      return LBM_ESTATE;
    }
  }
  BCHK(hipEventRecord(w1, B.stream));
  BCHK(hipEventSynchronize(w1));
  float wall = 0.f;
  BCHK(hipEventElapsedTime(&wall, w0, w1));
  // results
  BCHK(hipMemcpyAsync(B.mem_h + B.res_lo, B.mem_d + B.res_lo, B.res_hi - B.res_lo,
                      hipMemcpyDeviceToHost, B.stream));
  BCHK(hipStreamSynchronize(B.stream));
  bool warn = false, failed = false;
  long long node_updates = 0, fluid_updates = 0, lattice_steps = 0;
  for (int t = 0; t < n; ++t) {
    const sc::RampDev &R = B.rd[t];
    for (int i = 0; i < n_pc; ++i) {
      out[t].S[i] = B.S[(size_t)t * n_pc + i];
      out[t].steps[i] = B.steps[(size_t)t * n_pc + i];
      out[t].status[i] = B.status[(size_t)t * n_pc + i];
    }
    out[t].invaded_at = R.invaded_at;
    out[t].n_bisect = R.n_bisect;
    out[t].total_steps = R.total_steps;
    out[t].failed = R.failed ? 1 : 0;
    if (R.failed) {  // no entry pressure from a state that became non-finite
      out[t].pce_lo = NAN;
      out[t].pce = NAN;
      out[t].pce_hi = NAN;
    } else if (R.invaded_at < 0) {
      out[t].pce_lo = pc[(size_t)t * n_pc + n_pc - 1];
      out[t].pce = NAN;
      out[t].pce_hi = INFINITY;
    } else {
      out[t].pce_lo = R.lo;
      out[t].pce_hi = R.hi;
      out[t].pce = 0.5 * (R.lo + R.hi);
    }
    warn |= R.warn != 0;
    failed |= R.failed != 0;
    node_updates += R.total_steps * (long long)B.h[t]->N;
    fluid_updates += R.total_steps * (long long)B.h[t]->n_fluid;
    lattice_steps = std::max(lattice_steps, R.total_steps);
  }
  if (info) {
    const sc::Sched shape = B.nitems ? sc::Sched{sc::kListTx, 0, 0} : B.tiles;
    info->tx = shape.tx;
    info->ty = shape.ty;
    info->lz = shape.lz;
    info->replays = replays;
    info->lattice_steps = replays * c->check_every;
    info->node_updates = node_updates;
    info->fluid_updates = fluid_updates;
    info->wall_ms = wall;
    info->n_tiles = B.nitems + B.ntiles;
  }
  if (failed) return LBM_WPARTIAL;
  return warn ? LBM_WNOTCONV : LBM_OK;
}

}  // extern "C"
