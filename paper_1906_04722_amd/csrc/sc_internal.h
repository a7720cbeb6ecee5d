// sc_internal.h -- device-side data structures and kernel launchers of the
// Shan-Chen throat library (internal; the public interface is lbm_abi.h).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <vector>

namespace sc {

// node classes
enum : uint32_t { kFluid = 0, kSolid = 1, kResIn = 2, kResOut = 3 };

// Population storage of one buffer: shifted FP32 populations g = f - w_k
// rho_ref, q = 19 c + k for component c and direction k, of numbered nodes; 32
// consecutive numbers hold their 38 populations one after another, each a run
// of 32 floats (one 128-byte line): element (q, i) is at (i / 32) 38 * 32 +
// 32 q + i % 32.  Two numberings:
//
//  - compact: the non-solid nodes only, whole rows along x, in groups of
//    kGroupY rows that are marched through z.  No solid node takes space or
//    part of a line, and the 64 lanes of a wavefront pull runs of a few
//    neighbouring lines.  The step goes over it in two passes.
//  - bricks: every node of the box padded to whole bricks of 8 x 4 nodes per
//    z-plane, brick by brick, with a ghost plane at each end (brick_number).
//    Numbers follow from coordinates, so the tiled step needs no index map; it
//    reads each population once.  For nearly all-fluid boxes (kTileFill).
constexpr int kQ = 38;
constexpr int kLine = 32;
__host__ __device__ inline size_t pop_elems(size_t numbers) {
  return (numbers + kLine - 1) / kLine * (size_t)(kQ * kLine);
}
constexpr int kGroupY = 32;

// Index map of one subdomain: the number of the node at (x, y, z), or kNoNode
// where it is solid or beyond a wall, for -2 <= x < nx + 2 (likewise y, z); on
// periodic axes the two layers beyond the box repeat the nodes they wrap to.
// A pull or a density stencil reads its neighbours' numbers here, so no
// kernel handles walls, wraps or solid neighbours apart from kNoNode.
constexpr uint32_t kNoNode = 0xFFFFFFFFu;
constexpr int kPad = 2;
__host__ __device__ inline size_t map_elems(int nx, int ny, int nz) {
  return (size_t)(nx + 2 * kPad) * (size_t)(ny + 2 * kPad) * (size_t)(nz + 2 * kPad);
}
__host__ __device__ inline size_t map_pos(int nx, int ny, int x, int y, int z) {
  return ((size_t)(z + kPad) * (size_t)(ny + 2 * kPad) + (size_t)(y + kPad)) *
             (size_t)(nx + 2 * kPad) +
         (size_t)(x + kPad);
}

// Bricks of 8 x 4 nodes (x, y; the plane padded to multiples of 8 and 4):
// element (q, x, y, z) is at (z + 1) Pp + ((y / 4) (nxp / 8) + x / 8) 38 * 32 +
// 32 q + 8 (y mod 4) + x mod 8, Pp = 38 nxp nyp.  A line holds a compact 8 x 4
// patch of one population.  Planes z = -1 and z = nz are ghost copies of
// planes nz - 1 and 0 on z-periodic subdomains (unused otherwise), so that
// the pulls of a node on plane z read planes z - 1 .. z + 1 only: one base
// address and 32-bit offsets.  Checkpoint files hold every subdomain in this
// layout, solid nodes as zeros, whatever its numbering.
constexpr int kBX = 8, kBY = 4, kBN = kBX * kBY;
static_assert(kBN == kLine, "a brick is one line per population");
__host__ __device__ inline int pad_x(int nx) { return (nx + kBX - 1) / kBX * kBX; }
__host__ __device__ inline int pad_y(int ny) { return (ny + kBY - 1) / kBY * kBY; }
__host__ __device__ inline size_t brick_plane(int nx, int ny) {
  return (size_t)kQ * pad_x(nx) * pad_y(ny);
}
__host__ __device__ inline size_t brick_elems(int nx, int ny, int nz) {
  return brick_plane(nx, ny) * (size_t)(nz + 2);
}
// offset of population 0 of node (x, y) within its plane (0 <= x < nx,
// 0 <= y < ny); population q is 32 q further
__host__ __device__ inline uint32_t brick_x(int x) {
  return (uint32_t)(x / kBX) * (uint32_t)(kQ * kBN) + (uint32_t)(x % kBX);
}
__host__ __device__ inline uint32_t brick_y(int y, int nx) {
  return (uint32_t)(y / kBY) * (uint32_t)(pad_x(nx) / kBX) * (uint32_t)(kQ * kBN) +
         (uint32_t)(y % kBY) * (uint32_t)kBX;
}
// number of node (x, y, z) in the brick numbering
__host__ __device__ inline uint32_t brick_number(int nx, int ny, int x, int y, int z) {
  const uint32_t bricks = (uint32_t)(pad_x(nx) / kBX) * (uint32_t)(pad_y(ny) / kBY);
  return ((uint32_t)(z + 1) * bricks + (uint32_t)(y / kBY) * (uint32_t)(pad_x(nx) / kBX) +
          (uint32_t)(x / kBX)) * (uint32_t)kBN + (uint32_t)(y % kBY) * kBX + (uint32_t)(x % kBX);
}
// largest padded nx * ny whose three-plane pull offsets fit 32 bits of bytes
constexpr long long kMaxPlaneNodes = (1LL << 32) / (3LL * kQ * 4) - 1;

// mask word of a node (tiled step): bits 1..18 flag the directions k whose
// pull source x - e_k is solid or beyond a wall, bits 24..25 its class
constexpr int kTypeShift = 24;
constexpr uint32_t kLinkBits = 0x7FFFEu;

// one subdomain as the per-node kernels see it
struct Dom {
  const float *src;      // post-collision state of the previous step
  float *dst;            // post-collision state written by this step
  const uint32_t *map;   // index map
  const uint32_t *mask;  // [N] mask words (brick numbering only)
  size_t N;              // box nodes = nx * ny * nz
  int nx, ny, nz;
  int per;               // bit 0/1/2: x/y/z periodic
  int res;               // 1: z = 0 and z = nz - 1 are density baths
};

// physical parameters in the precision the step computes in
struct Phys {
  float tau[2], itau[2];
  float G, Gads[2];
  float rho_ref;         // shift of the stored populations
  float rres[2][2];      // bath densities [in/out][component]
  float gres[2][2];      // rres - rho_ref
};

// launch shape of the step: tiles of tx x ty columns marching lz planes in
// one fused pass (brick numbering), or (tx = kListTx) two passes over the
// non-solid nodes
struct Sched {
  int tx, ty, lz;
};
constexpr int kListTx = -1;

// tile shapes (tx, ty) the fused step is built for; lz is free (>= 1)
constexpr int kNumShapes = 6;
constexpr int kShapes[kNumShapes][2] = {{32, 4}, {32, 8}, {64, 4}, {16, 4}, {16, 8}, {8, 8}};
// rows of a workgroup's tile: two of the schedule's tiles in y
constexpr int tile_rows(int ty) { return 2 * ty; }

// one subdomain as the step sees it (a launch covers one or many of these)
struct Throat {
  float *g[2];           // A/B buffers; the state is in g[parity]
  const uint32_t *map;
  const uint32_t *pos;   // map position of each non-solid node, in number order
  float2 *rho;           // two passes: densities of the current step, by number
  uint32_t n_live;
  int nx, ny, nz, res;
  int active;            // 0: the launch skips this subdomain
  Phys P;
  const uint32_t *mask;  // tiled step: mask words, box size, tile grid
  uint32_t N;
  int per, ntx, nty, lz;
};

// a work item of the two passes: kListNodes consecutive nodes of a subdomain
constexpr int kListNodes = 64;
inline size_t list_count(size_t n_live) { return (n_live + kListNodes - 1) / kListNodes; }
// one item of work: subdomain and its packed tile coordinate
// tix + ntx * (tiy + nty * tiz), or its index among the subdomain's items
struct TileRef {
  int throat;
  int tile;
};

// spheres binned into cubic cells of kVoxCell nodes (CSR lists, device)
constexpr int kVoxCell = 16;
struct VoxBins {
  const int *start;  // [ncells + 1]
  const int *ids;    // sphere indices, increasing within a cell
  int ncx, ncy, ncz;
};
// host side of the binning: every sphere goes to each cell that its bounding
// box, widened by one node, meets
void bin_spheres(const double *sph, int ns, int nx, int ny, int nz, std::vector<int> &start,
                 std::vector<int> &ids, int &ncx, int &ncy, int &ncz);

// kernel launchers (all asynchronous on `st`)
hipError_t launch_voxelize(const double *spheres, const VoxBins &bins, int prism,
                           const int *prism_ids, int nx, int ny, int nz, int bc_z_reservoir,
                           uint8_t *types, hipStream_t st);
// non-solid nodes of each row (y, z), counts[z * ny + y]
hipError_t launch_row_counts(const uint8_t *types, int nx, int ny, int nz, uint32_t *counts,
                             hipStream_t st);
// host: first number of each row in the compact numbering, from its count, in
// place; returns the number of nodes
size_t number_rows(uint32_t *rows, int ny, int nz);
// index map and positions: compact from the rows' first numbers, or (rows
// null) bricks, whose live nodes are listed row by row in the same order
hipError_t launch_number(const uint8_t *types, int nx, int ny, int nz, int per,
                         const uint32_t *rows, bool bricks, uint32_t *map, uint32_t *pos,
                         hipStream_t st);
// The other numbering of a subdomain with positions pos: launch_renumber writes
// the index map of bricks or of the compact numbering, launch_move takes a
// population buffer to it from the other one (ghost planes of bricks included).
hipError_t launch_renumber(const Dom &d, const uint8_t *types, const uint32_t *pos, uint32_t n_live,
                           bool bricks, uint32_t *map, hipStream_t st);
hipError_t launch_move(const Dom &d, const uint32_t *pos, uint32_t n_live, bool bricks,
                       const float *src, float *dst, hipStream_t st);
hipError_t launch_links(const uint8_t *types, const Dom &d, uint32_t *mask, hipStream_t st);
// initial state; with a given one (rho_init [2][N]), *bad falls to the first
// c N + n at which it is not finite and positive on a fluid node
hipError_t launch_init(const Dom &d, const Phys &P, const double *rho_init, double rho_major,
                       double rho_minor, int z_front, const double *rres_d, float *g,
                       unsigned long long *bad, hipStream_t st);
// one time step of every active subdomain in `throats` over the listed items
// (device arrays) at launch shape tx, ty.  wide: some buffer or index map
// exceeds kNarrowBytes (two passes).  zper_ids (device, n_zper entries): the
// z-periodic subdomains in bricks, whose ghost planes are refreshed after the
// step.
constexpr size_t kNarrowBytes = ((size_t)1 << 32) - 16384;
hipError_t launch_step(const Throat *throats, const TileRef *tiles, int ntiles, int tx, int ty,
                       bool wide, int parity, hipStream_t st, const int *zper_ids, int n_zper);
// refresh the ghost planes of buffer g[which] of the listed subdomains
hipError_t launch_ghost(const Throat *throats, const int *zper_ids, int n_zper, int which,
                        hipStream_t st);
// host: per plane, which 8 x 4 bricks hold a non-solid node ([nz][nyp / 4]
// [nxp / 8] bytes); computed once per subdomain in bricks
void brick_map(const uint8_t *types, int nx, int ny, int nz, std::vector<uint8_t> &live);
// host: append the tiles of subdomain `throat` that hold at least one
// non-solid node (solid-only tiles need no update), from its brick map; every
// tile shape is a whole number of bricks
void list_tiles(const uint8_t *live, int nx, int ny, int nz, int tx, int ty, int lz, int throat,
                std::vector<TileRef> &out);
// host: append the two passes' items of subdomain `throat`
void list_items(size_t n_live, int throat, std::vector<TileRef> &out);
// populations of the flat range [first, first + count) of the checkpoint-file
// layout, gathered from or scattered into a population buffer
hipError_t launch_to_file(const Dom &d, const float *g, size_t first, size_t count, float *out,
                          hipStream_t st);
hipError_t launch_from_file(const Dom &d, const float *in, size_t first, size_t count, float *g,
                            hipStream_t st);
hipError_t launch_export(const Dom &d, const Phys &P, const double *rres_d, double *f,
                         hipStream_t st);
hipError_t launch_density(const Dom &d, const Phys &P, const double *rres_d, double *rho,
                          hipStream_t st);
// fixed device staging array of the allocation-free density read-back:
// kScratchDoubles doubles (32 MiB), enough for 2 densities of 2^21 nodes (a
// 128^3 box).  scratch_address gives the device address of the current
// device's copy (looked up once per device, then cached).
constexpr size_t kScratchNodes = (size_t)1 << 21;
constexpr size_t kScratchDoubles = 2 * kScratchNodes;
hipError_t scratch_address(double **out);
// FP64 reduction over subdomains: the sums of rho_w, rho_nw and the
// saturation term over the fluid nodes among a chunk of consecutive non-solid
// nodes, then per subdomain the sum of these, both in a fixed order.
struct RedInfo {
  long long probe;  // number of the probe node or -1
  double phib;      // bulk order parameter of the saturation map
};
// replace the map position that info[t].probe holds by the number found there
hipError_t launch_probe_numbers(const Throat *throats, int n, RedInfo *info, hipStream_t st);
struct RedChunk {
  int throat;
  uint32_t first, end;  // indices of its nodes
};
void red_chunks(size_t n_live, int throat, std::vector<RedChunk> &out);
// partials[c][3]; probe_out[t][2] = densities at subdomain t's probe node
hipError_t launch_reduce_chunks(const Throat *th, const RedChunk *chunks, int nchunks,
                                const RedInfo *info, int parity, double *partials,
                                double *probe_out, hipStream_t st);
// sums[t][3] over chunks first[t] .. first[t]+count[t]-1
hipError_t launch_reduce_throats(const int *first, const int *count, int n, const double *partials,
                                 double *sums, hipStream_t st);
// a range of a subdomain's population buffer (the batch's checkpoint copies):
// `count` 16-byte elements from `start`, both in units of 4 floats
struct Chunk {
  int throat;
  uint32_t count;
  unsigned long long start;
};
constexpr uint32_t kCopyChunk = 32768;
void copy_chunks(int throat, size_t elems, std::vector<Chunk> &out);
// plain copy of n_floats (a multiple of 4) floats, 16-byte aligned buffers
hipError_t launch_copy(const float *a, float *b, size_t n_floats, hipStream_t st);

bool schedule_valid(const Sched &s);

// ---- device-side drainage ramp of a batch of subdomains -------------------
enum : int { kPhaseRamp = 0, kPhaseBisect = 1, kPhaseDone = 2 };
// copy requests executed after each ramp decision, saves before restores
enum : int { kSaveStable = 1, kSaveMain = 2, kRestoreStable = 4, kRestoreMain = 8 };

// bisection runs of one drain at most: a throat already invaded at the first
// ramp point has 0 as its lower bracket, where halving alone need not reach
// the relative width; the drain then ends with its bracket and a warning
constexpr int kMaxBisect = 40;

struct RampCfg {
  double tol;        // |S(t) - S(t - every)| < tol ends a ramp point
  double rel;        // bisection stops at (hi - lo) / hi <= rel
  long long cap;     // steps per ramp point or bisection run
  int every;         // steps between checks (even)
  int n_pc;
};

struct RampDev {
  double rho_out, dpc_drho, rho_ref;   // rho_in = rho_out + pc / dpc_drho
  double S_old, S_stable, S_main, lo, hi, mid, stable_pc, rho_in_main;
  long long steps_pt, total_steps;
  unsigned int n_fluid;
  int phase, point, invaded_at, n_bisect, req, warn, failed;
};

struct Ckpt {
  float *stable, *main;
};

// first decision: record the initial saturation, save it as the stable
// state, set the first inlet density
hipError_t launch_ramp_begin(Throat *th, RampDev *rd, const double *pc, const RampCfg &cfg,
                             const double *sums, int n, hipStream_t st);
// one decision per subdomain after `every` steps; n_active_out[0] = number of
// subdomains still running
hipError_t launch_ramp_advance(Throat *th, RampDev *rd, const double *pc, const RampCfg &cfg,
                               const double *sums, const double *probe, double *S_out,
                               long long *steps_out, int *status_out, int n, int *n_active_out,
                               hipStream_t st);
// perform the copy requests of every subdomain, over its copy chunks
hipError_t launch_copy_requests(const Throat *th, const RampDev *rd, const Ckpt *ck,
                                const Chunk *chunks, int nchunks, int parity, hipStream_t st);

}  // namespace sc
