// lbm_handle.h -- the subdomain handle behind lbm_throat_t and the host
// helpers shared by the single-subdomain and the batched entry points
// (internal; the public interface is lbm_abi.h).
#pragma once

#include <hip/hip_runtime.h>

#include <string>
#include <utility>
#include <vector>

#include "lbm_abi.h"
#include "sc_internal.h"

// host-side drainage ramp of one subdomain (Sec. 2.2.2), advanced in chunks
// of check_every steps so that a caller can stop it, save it and resume it
struct HostRamp {
  enum : int { kIdle = 0, kRamp = 1, kBisect = 2, kDone = 3 };
  int phase = kIdle;
  std::vector<double> pc;
  lbm_conv c{};
  int point = 0;                // ramp point being run (kRamp) or bisected (kBisect)
  // the run in progress: steps so far and the saturation of the last check
  long long run_steps = 0;
  double S_old = 0.0;
  // bracket of the entry pressure and the states kept for the bisection
  double stable_pc = 0.0, lo = 0.0, hi = 0.0, mid = 0.0, main_rho_in = 0.0;
  int inv_at = -1, n_bisect = 0, runs = 0, warn = 0, failed = 0;
  long long total = 0;
  std::vector<double> S;
  std::vector<long long> steps;
  std::vector<int> status;
};

struct lbm_throat {
  int nx = 0, ny = 0, nz = 0, per = 0, bc[3] = {0, 0, 0};
  size_t N = 0;
  hipStream_t stream = nullptr;
  bool own_stream = false;
  float *g[2] = {nullptr, nullptr};  // A/B population buffers
  int cur = 0;                       // g[cur] holds the current state
  float *save[2] = {nullptr, nullptr};  // checkpoints used by the ramp
  bool bricks = false;               // brick numbering (else compact)
  size_t n_live = 0;                 // non-solid nodes
  size_t n_numbers = 0;              // numbers: n_live, or with padding and ghost planes
  uint32_t *map_d = nullptr;         // index map
  uint32_t *pos_d = nullptr;         // map positions of the non-solid nodes
  float2 *rho_d = nullptr;           // densities of the current step (two passes)
  uint32_t *mask_d = nullptr;        // mask words (bricks)
  uint8_t *types_d = nullptr;
  double *rres_d = nullptr;          // [in/out][component]
  // FP64 reduction: chunks of the node list, their partials, sums + probe
  sc::RedChunk *chunks_d = nullptr;
  int nchunks = 0;
  sc::RedInfo *redinfo_d = nullptr;
  int *red_first_d = nullptr;        // [1] = 0
  int *red_count_d = nullptr;        // [1] = nchunks
  double *partials = nullptr;        // [nchunks][3]
  // [5]: masses, saturation sum, probe densities; pinned, the kernels write it
  double *red_h = nullptr;
  hipEvent_t ev[2] = {nullptr, nullptr};
  std::vector<uint8_t> types;
  long long n_fluid = 0;
  long long probe_pos = -1;          // map position of the probe node
  long long probe = -1;              // its number
  double tau[2], G, Gads[2], rho_major, rho_minor, rho_in, rho_out;
  double phib = 1.0;
  sc::Phys P{};
  sc::Sched sched{sc::kListTx, 0, 0};
  std::vector<uint8_t> brick_live;   // brick liveness map (sc::brick_map)
  long long steps_done = 0;
  // device descriptor and work items of the step
  sc::Throat desc{};
  sc::Throat *desc_d = nullptr;
  sc::TileRef *tiles_d = nullptr;
  int ntiles = 0;
  size_t tiles_cap = 0;
  int *zper_d = nullptr;             // {0} with ghost planes to refresh
  int n_zper = 0;
  // event-timed step launches inside the drainage ramp
  hipEvent_t tev[2] = {nullptr, nullptr};
  bool timing = false;
  double timed_ms = 0.0;
  long long timed_launches = 0;
  HostRamp ramp;
};


namespace lbmh {

void set_err(const char *fmt, ...);
// check the parameters and take them into a fresh handle (no device call)
int describe(const lbm_params *p, lbm_throat *h);
// the descriptor h->desc from the handle's buffers and parameters
void fill_desc(lbm_throat *h);
sc::Dom dom(const lbm_throat *h);
// spheres of a subdomain and their bins, as the voxelisation reads them
struct Geometry {
  std::vector<double> sph;  // (cx, cy, cz, r); at least one
  std::vector<int> bin_start, bin_ids;
  int ncx = 0, ncy = 0, ncz = 0;
  explicit Geometry(const lbm_params &p);
  hipError_t voxelize(const lbm_params &p, const double *sph_d, const int *start_d,
                      const int *ids_d, uint8_t *types_d, hipStream_t st) const;
};
// refuse a given initial state that is not finite and positive at c N + n = bad
int check_rho_init(const lbm_throat *h, unsigned long long bad);
// whether the two passes need 64-bit addresses
inline bool wide(const lbm_throat *h) {
  return sizeof(float) * sc::pop_elems(h->n_numbers) > sc::kNarrowBytes ||
         sizeof(uint32_t) * sc::map_elems(h->nx, h->ny, h->nz) > sc::kNarrowBytes;
}
// bricks: the box's nodes in whole bricks, and with the ghost planes; whether
// enough lanes of its default tiles have a node, and from how many slots on the
// tiles pay (one box's, or all such boxes' of a batch)
inline size_t brick_slots(const lbm_throat *h) {
  return (size_t)sc::pad_x(h->nx) * sc::pad_y(h->ny) * (size_t)h->nz;
}
inline size_t brick_numbers(const lbm_throat *h) {
  return (size_t)sc::pad_x(h->nx) * sc::pad_y(h->ny) * ((size_t)h->nz + 2);
}
bool fills_tiles(const lbm_throat *h);
constexpr size_t kTileNodes = (size_t)1 << 21;
// z-segments of boxes (tile columns, planes) stepped in one launch
int tile_length(const std::vector<std::pair<long long, int>> &boxes);
// the schedules of boxes in bricks that are stepped in one launch, and its shape
sc::Sched batch_tiles(const std::vector<lbm_throat *> &boxes);
// device memory of one subdomain (with or without the two ramp checkpoints)
// and the refusal of a call whose need exceeds the memory budget
size_t subdomain_bytes(int nx, int ny, int nz, bool checkpoints);
int check_budget(size_t need, const char *what);

}  // namespace lbmh
