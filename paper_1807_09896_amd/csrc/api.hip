// C ABI of the DPD step library (declared in include/dpd.h): context set-up,
// validation, buffer management, the per-step launch sequence, getters,
// HIP-graph capture of the step and the launch-shape autotuner.
//
// A context holds R >= 1 independent boxes ("replicas") in concatenated
// arrays; a single box is a batch of one.  Every step kernel covers all
// boxes: integrate and pair-force read their box's descriptor per block, the
// cell-list kernels work on one global cell index space.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstddef>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <fstream>
#include <sstream>
#include <string>
#include <vector>

#include "dpd.h"
#include "device.h"
#include "kernels.h"

using dpd::Box;
using dpd::KGeom;
using dpd::KParams;
using dpd::Status;
using dpd::StatusBlock;
using dpd::Tile;

namespace {

thread_local std::string g_create_error = "no error";

enum Kernel { K_INTEGRATE = 0, K_SCAN_REDUCE, K_PERSIST, K_SCAN_DOWN, K_SCATTER, K_SORT,
              K_FORCE, K_OTHER, K_CODES };
// "step_persistent": the one launch of a persistent step (dpd_use_persistent),
// which does the work of all the others.
const char *kKernelNames[DPD_NUM_KERNELS] = {"integrate_reflect_bin", "scan_reduce",
                                             "step_persistent", "scan_down", "scatter",
                                             "sort_cells", "pair_force", "other", "pair_codes"};

struct TimedLaunch {
  int kernel;
  hipEvent_t a, b;
};

// Host view of one box.
struct Replica {
  int64_t n = 0, nf = 0, nw = 0;
  int64_t fo = 0, wo = 0, co = 0, ncell = 0, go = 0, bo = 0, nwords = 0;
  int nc[3] = {0, 0, 0}, ng[3] = {0, 0, 0};
  double L[3] = {0, 0, 0}, h[3] = {0, 0, 0};
  double rc = 0;
  bool moving = false;   // some wall particle has a nonzero velocity
  bool brick = false;    // pair forces by the LDS-staged brick kernel
  KGeom G{};
  KParams P{};
  int64_t flagged_cubes = 0;
};

// Buffers and bookkeeping of a recorded window (adjoint form).
struct Window {
  bool valid = false;
  int steps = 0, ckpt = 0, nck = 0, axis = 2, nbins = 0;
  float scale = 0.f;
  uint64_t k0 = 0, gen = 0;
  int64_t nf = 0;
  // the whole window kept (store), where it fits kWindowStore: per step its
  // start state, drifted positions, predicted velocities and cell list, so that
  // the sweep recomputes nothing
  bool full = false;
  char *store = nullptr;
  size_t store_cap = 0;
  float4 *ck = nullptr;    // nck checkpoints of 3 x NF (pos, vel, frc)
  float4 *seg = nullptr;   // ckpt states of one segment, 3 x NF each
  float4 *save = nullptr;  // the context state during a backward sweep
  float4 *wpos = nullptr;  // positions of the sweep, NF + NW + 1
  float4 *adj = nullptr;   // 11 x NF adjoint arrays
  double *sums = nullptr, *acc = nullptr, *part_f = nullptr, *part_g = nullptr;
  unsigned long long *counts = nullptr, *dk0 = nullptr;
  float *lw = nullptr;
  Status *status_save = nullptr;
  int cap_nck = 0, cap_ckpt = 0, cap_nbins = 0, cap_f = 0, cap_g = 0;
};

}  // namespace

struct dpd_ctx {
  int device = 0;
  hipStream_t stream = nullptr;
  dpd_allocator al{};
  bool has_al = false;
  std::string err = "no error";
  std::vector<void *> owned;

  int R = 0;
  std::vector<Replica> rep;
  int64_t NF = 0, NW = 0, NCELL = 0, NGRID = 0, NWORDS = 0;
  int grid_f64 = 0;
  int use_mask = 1;

  Box *boxes = nullptr;
  int ppt = 2, fblock = 256;            // launch shapes (autotuned)
  bool wide = false;      // pair forces with 16 lanes per particle (use_wide)
  int box_list = 0;       // blocks per box of the one-launch cell list, 0: not used (box_parts)
  bool box_codes = false; // its blocks write the runs' coarse codes as well
  Tile *itiles = nullptr, *ftiles = nullptr;
  int n_itiles = 0, n_ftiles = 0;
  int itiles_cap = 0, ftiles_cap = 0;
  // pair forces: bricks of the boxes that take the LDS-staged kernel, and
  // tiles of fluid slots of the others (the per-particle kernel)
  dpd::Brick *bricks = nullptr;
  int nbricks = 0;
  Tile *otiles = nullptr;
  int n_otiles = 0, otiles_cap = 0;

  float4 *pos[2] = {nullptr, nullptr}, *vel[2] = {nullptr, nullptr}, *frc[2] = {nullptr, nullptr};
  float4 *vt = nullptr;
  int cur = 0;
  int32_t *cell_of = nullptr, *rank_of = nullptr, *count = nullptr, *cstart = nullptr,
          *idx = nullptr, *bsum = nullptr;
  int nscan = 0;
  int32_t *wcstart = nullptr;   // exclusive scan of wall counts per cell (static)
  int32_t *wcell = nullptr;     // global cell of each cell-sorted wall (rebuilt by the wall pass)
  int32_t *idx_all = nullptr;   // merged per-cell runs: walls (NF + w), then fluid
  uint32_t *cq = nullptr;       // coarse position codes of the merged runs
  // moving walls: re-sorted by cell every step (moved copy, velocities,
  // cells, ranks, per-cell counts)
  bool moving = false;
  bool reflect = false;   // some box has moving walls or specular reflection
  bool sph = false;       // some box uses the attractive-repulsive conservative force
  float4 *wtmp = nullptr, *wvtmp = nullptr;
  int32_t *wcell_tmp = nullptr, *wrank = nullptr, *wcount = nullptr, *widx = nullptr,
          *wsum = nullptr;
  int32_t *start_all = nullptr; // start of each cell's merged run
  int32_t *fluid_off = nullptr; // start of each cell's fluid part in the merged run
  void *grid = nullptr;
  void *quad = nullptr;         // the grids in the face layout (4 values a node)
  uint32_t *bits = nullptr;     // near-interface grid cubes, one bit each
  Status *status = nullptr; // head of a StatusBlock
  Status *note = nullptr;   // pinned host memory the kernels of a getter leave the status in
  unsigned long long *dk = nullptr;  // force evaluation index on the device
  unsigned long long *pair_counter = nullptr;

  uint64_t k = 0;
  int64_t steps = 0;

  bool timing = false;
  std::vector<TimedLaunch> pending;
  std::vector<hipEvent_t> free_events;
  double kernel_ms[DPD_NUM_KERNELS] = {0};
  int64_t kernel_launches[DPD_NUM_KERNELS] = {0};

  bool use_graph = false;
  hipStream_t cap_stream = nullptr;
  hipGraphExec_t graph[2] = {nullptr, nullptr};
  // steps in a row (step_run): second prediction and cell counts, in turn with vt and
  // count (null: not used)
  float4 *vt2 = nullptr;
  int32_t *count2 = nullptr;
  bool captured = false;   // a caller's own graph may hold them

  // persistent step (dpd_use_persistent): work items, per-(box, phase) item
  // counts and arrivals, the queue counter, per-box scan chunk sums, 256-particle
  // force tiles, and the launch arguments for either buffer set
  bool persistent = false;
  dpd::PItem *pitems = nullptr;
  int n_pitems = 0;
  int32_t *pneed = nullptr, *parrive = nullptr, *phead = nullptr, *pbsum = nullptr;
  Tile *ptiles = nullptr;
  int n_ptiles = 0, ptiles_cap = 0;
  dpd::PArgs *pargs[2] = {nullptr, nullptr};
  int pblocks = 0;

  Window win;
  uint64_t gen = 0;  // bumped when parameters, phi or the state are replaced
};

namespace {

int fail(dpd_ctx *c, int code, const std::string &msg) {
  if (c)
    c->err = msg;
  else
    g_create_error = msg;
  return code;
}

int hip_fail(dpd_ctx *c, hipError_t e, const char *where) {
  std::string m = std::string(where) + ": " + hipGetErrorString(e);
  return fail(c, e == hipErrorOutOfMemory ? DPD_E_NOMEM : DPD_E_DEVICE, m);
}

#define HIP_TRY(ctx, expr)                                      \
  do {                                                          \
    hipError_t e_ = (expr);                                     \
    if (e_ != hipSuccess) return hip_fail((ctx), e_, #expr);    \
  } while (0)

bool give_back(dpd_ctx *c);

// spare: memory that the caller can do without.  For any other, what the context holds
// of such memory makes room where there is none.
void *dalloc(dpd_ctx *c, size_t bytes, bool spare = false) {
  bytes = (bytes + 255) & ~(size_t)255;
  if (bytes == 0) bytes = 256;
  void *p = nullptr;
  do {
    if (c->has_al) {
      p = c->al.alloc(bytes, (void *)c->stream, c->al.user);
    } else if (hipMalloc(&p, bytes) != hipSuccess) {
      p = nullptr;
      (void)hipGetLastError();   // reported by the caller, or done without
    }
  } while (!p && !spare && give_back(c));
  if (p) c->owned.push_back(p);
  return p;
}

void dfree(dpd_ctx *c, void *p) {
  for (size_t q = 0; q < c->owned.size(); ++q) {
    if (c->owned[q] != p) continue;
    if (c->has_al)
      c->al.free(p, (void *)c->stream, c->al.user);
    else
      (void)hipFree(p);
    c->owned.erase(c->owned.begin() + (std::ptrdiff_t)q);
    return;
  }
}

void drop_graphs(dpd_ctx *c) {
  for (int g = 0; g < 2; ++g)
    if (c->graph[g]) {
      (void)hipGraphExecDestroy(c->graph[g]);
      c->graph[g] = nullptr;
    }
}

hipError_t write_persistent_args(dpd_ctx *c);

void free_store(Window &W, dpd_ctx *c) {
  if (W.store) dfree(c, W.store);
  W.store = nullptr;
  W.store_cap = 0;
}

// Memory that only saves time, back to the allocator: the store of a window that can
// no longer be swept, and the second prediction and counts of steps in a row (both
// counts are clear between calls, and the walls' part of both predictions is the same).
// False where the context holds none.
bool give_back(dpd_ctx *c) {
  Window &W = c->win;
  const bool store = W.store && !(W.valid && W.gen == c->gen), row = c->vt2 && !c->captured;
  if (!store && !row) return false;
  (void)hipStreamSynchronize(c->stream);
  if (store) {
    free_store(W, c);
    W.full = false;
  }
  if (row) {
    drop_graphs(c);   // a captured step holds one of each pair
    dfree(c, c->vt2);
    if (c->count2) dfree(c, c->count2);
    c->vt2 = nullptr;
    c->count2 = nullptr;
    if (c->persistent) (void)write_persistent_args(c);
  }
  return true;
}

void release_all(dpd_ctx *c) {
  drop_graphs(c);
  if (c->cap_stream) {
    (void)hipStreamDestroy(c->cap_stream);
    c->cap_stream = nullptr;
  }
  for (void *p : c->owned) {
    if (c->has_al)
      c->al.free(p, (void *)c->stream, c->al.user);
    else
      (void)hipFree(p);
  }
  c->owned.clear();
  if (c->note) (void)hipHostFree(c->note);
  c->note = nullptr;
  for (auto &t : c->pending) {
    (void)hipEventDestroy(t.a);
    (void)hipEventDestroy(t.b);
  }
  c->pending.clear();
  for (auto e : c->free_events) (void)hipEventDestroy(e);
  c->free_events.clear();
}

hipEvent_t get_event(dpd_ctx *c) {
  if (!c->free_events.empty()) {
    hipEvent_t e = c->free_events.back();
    c->free_events.pop_back();
    return e;
  }
  hipEvent_t e = nullptr;
  (void)hipEventCreate(&e);
  return e;
}

// Collect finished timings (the stream must have been synchronised).
void harvest_timings(dpd_ctx *c) {
  for (auto &t : c->pending) {
    float ms = 0.f;
    if (hipEventElapsedTime(&ms, t.a, t.b) == hipSuccess) {
      c->kernel_ms[t.kernel] += ms;
      c->kernel_launches[t.kernel] += 1;
    }
    c->free_events.push_back(t.a);
    c->free_events.push_back(t.b);
  }
  c->pending.clear();
}

// Launch helper: brackets a launch with events when timing is on.
template <typename F>
hipError_t timed(dpd_ctx *c, hipStream_t s, int kernel, F &&launch) {
  if (!c->timing || s != c->stream) return launch();
  if (c->pending.size() > 4096) {
    hipError_t e = hipStreamSynchronize(c->stream);
    if (e != hipSuccess) return e;
    harvest_timings(c);
  }
  TimedLaunch t{kernel, get_event(c), get_event(c)};
  (void)hipEventRecord(t.a, c->stream);
  hipError_t e = launch();
  (void)hipEventRecord(t.b, c->stream);
  c->pending.push_back(t);
  return e;
}

int read_status(dpd_ctx *c, Status &st) {
  HIP_TRY(c, dpd::launch_note_status(c->stream, c->status, c->note));
  HIP_TRY(c, hipStreamSynchronize(c->stream));
  st = *c->note;
  return DPD_OK;
}

// A status read earlier back to the device (st lives until the stream has come to it).
int write_status(dpd_ctx *c, const Status &st) {
  HIP_TRY(c, dpd::launch_fill_zero(c->stream, c->status, sizeof(StatusBlock)));
  HIP_TRY(c, hipMemcpyAsync(c->status, &st, sizeof(Status), hipMemcpyHostToDevice, c->stream));
  return DPD_OK;
}

// The error that a status holds.
int status_error(dpd_ctx *c, const Status &st) {
  if (st.nonfinite)
    return fail(c, DPD_E_UNSTABLE, "non-finite positions or forces (" +
                                       std::to_string(st.nonfinite) + " events)");
  if (st.unstable)
    return fail(c, DPD_E_UNSTABLE, "a particle moved more than half a cell in one step (" +
                                       std::to_string(st.unstable) + " events)");
  if (st.stalled)
    return fail(c, DPD_E_DEVICE, "a persistent step's wait reached its bound (" +
                                     std::to_string(st.stalled) +
                                     " waits); the state after it is not valid");
  return DPD_OK;
}

int latched_error(dpd_ctx *c) {
  Status st;
  int rc = read_status(c, st);
  return rc ? rc : status_error(c, st);
}

// Rows of box r by gid and, once the stream has come to it, the status.
hipError_t export_box(dpd_ctx *c, int32_t r, float *pos, float *vel, float *frc, int32_t *events,
                      int32_t *cell_of) {
  const Replica &p = c->rep[r];
  const int a = c->cur;
  return dpd::launch_export(c->stream, p.G, p.nf, p.nw, c->pos[a] + p.fo, c->vel[a] + p.fo,
                            c->frc[a] + p.fo, c->pos[a] + c->NF + p.wo, c->vt + c->NF + p.wo, pos,
                            vel, frc, events, cell_of, c->status, c->note);
}

// Release a half-built context, keeping its message as the create error.
int abandon_create(dpd_ctx *c, int code) {
  (void)hipStreamSynchronize(c->stream);
  release_all(c);
  g_create_error = c->err;
  delete c;
  return code;
}

bool finite3(const float *p) {
  return std::isfinite(p[0]) && std::isfinite(p[1]) && std::isfinite(p[2]);
}

// Pair-kernel tiles of a single-box context in y-bands of this many cell
// rows (see band_order).
constexpr int64_t kForceBandRows = 56;

// Order of a single box's pair-kernel tiles.  The kernel gives each XCD one
// contiguous eighth of the tile list (a z-slab of the cell-sorted box), and
// an XCD's resident blocks take its tiles in list order, so the neighbour
// records they gather at any one time come from the rows around the tiles
// in flight.  In plain cell order those are about three whole z-planes, more
// than a 4 MB L2 holds; taken in y-bands of kForceBandRows rows (band, then
// z, then y), the tiles in flight cover a shorter, deeper region whose
// neighbourhood is smaller.  A tile's place is estimated from its first
// slot as if the fluid filled the cells evenly, which is enough for
// locality: the order decides nothing else, each tile's forces are the same
// whichever block takes it.  Measured on the 168^3 porous box (168 rows):
// the kernel fetched 0.98 GB per launch instead of 1.17 with 56-row bands,
// at equal or slightly shorter time; 34 and 42 rows fetched 1.12 and 1.05
// GB, 84 rows 0.96 GB, and bands of 12 or 24 rows took longer.
void band_order(const Replica &p, std::vector<Tile> &t) {
  const int T = (int)t.size(), per = (T + 7) / 8;
  const int64_t nx = p.nc[0], ny = p.nc[1];
  if (ny <= kForceBandRows || T < 8) return;
  std::vector<Tile> u(t.size());
  std::vector<std::pair<int64_t, int>> key;
  for (int k = 0; k < 8; ++k) {
    const int a = k * per, b = std::min(T, (k + 1) * per);
    key.clear();
    for (int i = a; i < b; ++i) {
      const double frac = (double)(t[i].first - p.fo) / (double)p.nf;
      const int64_t cell = std::min<int64_t>((int64_t)(frac * (double)p.ncell), p.ncell - 1);
      const int64_t z = cell / (nx * ny), y = (cell / nx) % ny;
      key.push_back({(((y / kForceBandRows) * p.nc[2] + z) * ny + y) * (int64_t)T + i, i});
    }
    std::sort(key.begin(), key.end());
    for (size_t j = 0; j < key.size(); ++j) u[a + j] = t[key[j].second];
  }
  t.swap(u);
}

// Tile tables: runs of consecutive particles of one box, `size` per tile
// (without_bricks: only the boxes whose pair forces take the per-particle
// kernel; banded: a single box's tiles in the order of band_order).
int build_tiles(dpd_ctx *c, int size, Tile **dst, int *n, int *cap, bool without_bricks = false,
                bool banded = false) {
  std::vector<Tile> t;
  for (int r = 0; r < c->R; ++r) {
    const Replica &p = c->rep[r];
    if (without_bricks && p.brick) continue;
    for (int64_t f = 0; f < p.nf; f += size) {
      Tile x;
      x.box = r;
      x.first = (int32_t)(p.fo + f);
      x.count = (int32_t)std::min<int64_t>(size, p.nf - f);
      x.pad = 0;
      t.push_back(x);
    }
  }
  if (banded && c->R == 1 && !t.empty()) band_order(c->rep[0], t);
  if ((int)t.size() > *cap) {
    if (*dst) dfree(c, *dst);
    *dst = (Tile *)dalloc(c, sizeof(Tile) * std::max<size_t>(t.size(), 1));
    if (!*dst) return fail(c, DPD_E_NOMEM, "tile table allocation failed");
    *cap = (int)t.size();
  }
  *n = (int)t.size();
  if (!t.empty())
    HIP_TRY(c, hipMemcpyAsync(*dst, t.data(), sizeof(Tile) * t.size(), hipMemcpyHostToDevice,
                              c->stream));
  HIP_TRY(c, hipStreamSynchronize(c->stream));
  return DPD_OK;
}

int build_persistent(dpd_ctx *c);

// The context's wider integrate shape: 4 particles per thread
// (80 VGPRs, six wavefronts per SIMD, four particles' loads in flight per
// lane) for contexts of at least 2^20 fluid particles whose boxes all use
// the plain instance; 2 otherwise.  The instance with moving walls and
// specular reflection needs 112 VGPRs at 4 and took longer (Couette channel:
// integrate 0.051 -> 0.073 ms).
int wide_ppt(const dpd_ctx *c) { return !c->reflect && c->NF >= ((int64_t)1 << 20) ? 4 : 2; }

// The shape a context starts with: 1 particle per thread below 2^20, where a
// step waits for one thread's chain of loads rather than for the chip (whole step,
// us, 1 against 2: 22.1 / 23.6 at 2,000 particles, 37.9 / 40.1 at 16,000, 71.6 /
// 73.8 at 177,000, 89.4 / 91.4 at 330,000, 221 / 222 at 746,000 with moving
// walls), the wider one above (4 against 1: 1.199 / 1.217 ms at 6.3 million) and for
// batches from 2^18 on, whose boxes end in part-filled tiles (127.4 against 128.7
// at 64 uneven boxes of 350,000).
int default_ppt(const dpd_ctx *c) {
  return c->NF < ((int64_t)1 << (c->R > 1 ? 18 : 20)) ? 1 : wide_ppt(c);
}

// Pair forces with 16 lanes per particle (k_force_wide) up to this many fluid
// particles in the context.  It spends about 0.43 ns per particle where the
// one-lane kernel spends 0.14 to 0.17, but the latter takes 27 (density 3) to 33
// us (density 4) however few there are.  Measured (graph-replayed step, us, 16
// lanes against one): 31 / 50 at 2,000 particles, 40 / 57 at 16,000, 46 / 57
// at 29,000, 54 / 58 at 56,000 (density 4: 65 / 69 at 75,000), and 68 / 62 at
// 97,000 (86 / 74 at 129,000).  The bits are the same either way.
constexpr int64_t kWideMax = 65536;
bool use_wide(const dpd_ctx *c) { return c->NF <= kWideMax; }

// Steps in a row (step_run) where the pair kernel has 16 lanes per particle: up to this
// many blocks, of 16 particles, which are all on the chip at once (five on each of
// 256 CUs); where they are not, one lane of 16 drifting costs as much as the launch it
// saves.  Step, us, without / with: 19.6 / 16.2 at 2,400 particles, 20.5 / 17.2 at
// 7,400, 24.1 / 21.9 at 16,500, 25.4 / 24.4 at 20,000; 32.8 / 33.1 at 27,000, 37.9 /
// 40.4 at 61,000.  With one lane per particle it pays at every size (force_tile).
constexpr int kRunTiles = 1280;

// Blocks per box of the one-launch cell list (k_cells_box); 0 where some box does
// not fit its LDS, where the brick kernel needs the separate launches' arrays, and
// where walls move (list_both lists them with the fluid).
// 256 CUs hold one such block each, so the boxes share 256, up to 16 a box (a box of
// at most 1,024 particles is one round of one block's threads).  Whole step, us,
// four launches / 1 / 4 / 16 blocks per box: 29.0 / 24.4 / 22.9 / 22.9 at 2,000
// particles, 36.1 / 31.1 / 26.9 / 24.9 at 8,400, 38.3 / 39.9 / 31.1 / 27.9 at 16,000,
// 41.3 / 48.1 / 35.9 / 32.2 at 22,000; 64 boxes: 127 / 126 / 115 / 131.
// More boxes than CUs take turns, each block's chain of phases after another's.  From
// the third turn on that costs more than the launches save, unless the boxes are large
// enough for the blocks to work through them about as fast as the launches do (step of
// steps in a row, us, four launches / one: 300 particles a box 57.7 / 54.1 at 512
// boxes, 63.5 / 63.9 at 576, 88 / 93 at 1,024, 150 / 174 at 2,048; 1,000 a box 107 /
// 103 at 512, 116 / 118 at 576, 179 / 184 at 1,024, 325 / 345 at 2,048; 1,500 a box
// 176 / 174 at 768, 223 / 225 at 1,024, 423 / 431 at 2,048; 2,200 a box 247 / 244 at
// 768, 318 / 317 at 1,024, 617 / 622 at 2,048; 8,200 a box 1,124 / 1,100 at 1,024,
// 2,240 / 2,200 at 2,048).
constexpr int kBoxTurns = 2 * 256, kBoxLarge = 1536;
int box_parts(const dpd_ctx *c) {
  if (c->nbricks > 0 || c->moving) return 0;
  if (c->R > kBoxTurns && c->NF < (int64_t)kBoxLarge * c->R) return 0;
  int64_t most = 0;
  for (const Replica &p : c->rep) {
    if (p.ncell > dpd::kBoxCells || p.nf > dpd::kBoxFluid) return 0;
    most = std::max(most, p.nf);
  }
  return most <= 1024 ? 1 : std::max(1, std::min(16, 256 / c->R));
}

// Launch shapes: particles per thread of integrate (1, 2 or 4; at most 2
// under the persistent step, whose kernel holds every phase at six
// wavefronts per SIMD) and the pair kernel's work-group size.
int set_shapes(dpd_ctx *c, int ppt, int fblock) {
  if (c->persistent && ppt > 2) ppt = 2;
  c->ppt = ppt;
  c->fblock = fblock;
  drop_graphs(c);
  int rc = build_tiles(c, 256 * ppt, &c->itiles, &c->n_itiles, &c->itiles_cap);
  if (!rc)
    rc = build_tiles(c, c->wide ? dpd::kWideParts : fblock, &c->ftiles, &c->n_ftiles,
                     &c->ftiles_cap);
  if (!rc)
    rc = build_tiles(c, c->wide ? dpd::kWideParts : fblock, &c->otiles, &c->n_otiles,
                     &c->otiles_cap, true, true);
  if (!rc && c->persistent) rc = build_persistent(c);
  return rc;
}

// Work items of the persistent step, in queue order: every box's integrate
// tiles (grouped, see add_tiles), then per box its scan chunks (reduce, then
// down), its scatter ranges (fluid slots, then walls), its per-cell sort
// ranges, and its force tiles (grouped); each
// phase's items of all boxes before the next phase's, so that no item waits
// on one after it.  need[box][phase] counts them.
constexpr int kScatterItem = 4096;   // particles per scatter item
constexpr int kSortItem = 2048;      // cells per sort item
constexpr int kTilesPerItem = 16;    // at most, integrate or force tiles per item

int build_persistent(dpd_ctx *c) {
  using dpd::PItem;
  const int R = c->R, NP = dpd::kPhases;
  int ncu = 0;
  HIP_TRY(c, hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, c->device));
  const int per = dpd::persistent_blocks_per_cu(c->ppt, c->grid_f64, c->reflect ? 1 : 0,
                                                c->sph ? 1 : 0);
  if (per <= 0) return fail(c, DPD_E_DEVICE, "persistent step: no resident blocks");
  c->pblocks = per * ncu;
  int rc = build_tiles(c, 256, &c->ptiles, &c->n_ptiles, &c->ptiles_cap, true);
  if (rc) return rc;
  std::vector<Tile> it((size_t)c->n_itiles), ft((size_t)c->n_ptiles);
  if (c->n_itiles)
    HIP_TRY(c, hipMemcpy(it.data(), c->itiles, sizeof(Tile) * it.size(), hipMemcpyDeviceToHost));
  if (c->n_ptiles)
    HIP_TRY(c, hipMemcpy(ft.data(), c->ptiles, sizeof(Tile) * ft.size(), hipMemcpyDeviceToHost));
  std::vector<PItem> items;
  std::vector<int32_t> need((size_t)R * NP, 0);
  auto add = [&](int phase, int box, int64_t a, int64_t b) {
    items.push_back(PItem{phase, box, (int32_t)a, (int32_t)b});
    need[(size_t)box * NP + phase] += 1;
  };
  // integrate and force items: consecutive tiles of one box, about twice
  // as many per item as the phase has tiles per resident block, at most
  // kTilesPerItem (every item ends with a device-scope release, the costly
  // part, but small boxes need the items to spread over the blocks)
  auto add_tiles = [&](int phase, const std::vector<Tile> &tl) {
    const size_t per_item = std::max<size_t>(
        1, std::min<size_t>(kTilesPerItem, 2 * tl.size() / (size_t)c->pblocks));
    for (size_t t = 0; t < tl.size();) {
      size_t e = t + 1;
      while (e < tl.size() && e - t < per_item && tl[e].box == tl[t].box) ++e;
      add(phase, tl[t].box, (int64_t)t, (int64_t)e);
      t = e;
    }
  };
  add_tiles(dpd::kPhIntegrate, it);
  std::vector<int> chunk0((size_t)R);
  int nch_all = 0;
  for (int r = 0; r < R; ++r) {
    chunk0[r] = nch_all;
    nch_all += (int)((c->rep[r].ncell + dpd::kScanChunk - 1) / dpd::kScanChunk);
  }
  for (int ph : {(int)dpd::kPhReduce, (int)dpd::kPhDown})
    for (int r = 0; r < R; ++r) {
      const int n = (int)((c->rep[r].ncell + dpd::kScanChunk - 1) / dpd::kScanChunk);
      for (int j = 0; j < n; ++j) add(ph, r, j, chunk0[r]);
    }
  for (int r = 0; r < R; ++r) {
    const Replica &p = c->rep[r];
    for (int64_t a = p.fo; a < p.fo + p.nf; a += kScatterItem)
      add(dpd::kPhScatter, r, a, std::min(a + kScatterItem, p.fo + p.nf));
    const int64_t w0 = c->NF + p.wo, w1 = w0 + p.nw;
    for (int64_t a = w0; a < w1; a += kScatterItem)
      add(dpd::kPhScatter, r, a, std::min(a + kScatterItem, w1));
  }
  for (int r = 0; r < R; ++r) {
    const Replica &p = c->rep[r];
    // an empty box has nothing to sort; its sort items would find no scatter item to wait
    // for, and read run starts that the scan may not have written yet (where the context's
    // lists come from k_cells_box, nothing else has)
    if (p.n == 0) continue;
    for (int64_t a = p.co; a < p.co + p.ncell; a += kSortItem)
      add(dpd::kPhSort, r, a, std::min(a + kSortItem, p.co + p.ncell));
  }
  add_tiles(dpd::kPhForce, ft);
  if (c->NF + c->NW + (int64_t)nch_all >= ((int64_t)1 << 31))
    return fail(c, DPD_E_INVAL, "the batch is too large for the persistent step");

  for (void *q : {(void *)c->pitems, (void *)c->pneed, (void *)c->parrive, (void *)c->phead,
                  (void *)c->pbsum, (void *)c->pargs[0], (void *)c->pargs[1]})
    if (q) dfree(c, q);
  c->pargs[0] = c->pargs[1] = nullptr;
  c->pitems = (PItem *)dalloc(c, sizeof(PItem) * std::max<size_t>(items.size(), 1));
  c->pneed = (int32_t *)dalloc(c, 4 * need.size());
  c->parrive = (int32_t *)dalloc(c, 4 * need.size());
  c->phead = (int32_t *)dalloc(c, 4);
  c->pbsum = (int32_t *)dalloc(c, 4 * (size_t)std::max(nch_all, 1));
  c->pargs[0] = (dpd::PArgs *)dalloc(c, sizeof(dpd::PArgs));
  c->pargs[1] = (dpd::PArgs *)dalloc(c, sizeof(dpd::PArgs));
  if (!c->pitems || !c->pneed || !c->parrive || !c->phead || !c->pbsum || !c->pargs[0] ||
      !c->pargs[1])
    return fail(c, DPD_E_NOMEM, "persistent-step allocation failed");
  c->n_pitems = (int)items.size();
  if (!items.empty())
    HIP_TRY(c, hipMemcpy(c->pitems, items.data(), sizeof(PItem) * items.size(),
                         hipMemcpyHostToDevice));
  HIP_TRY(c, hipMemcpy(c->pneed, need.data(), 4 * need.size(), hipMemcpyHostToDevice));
  HIP_TRY(c, write_persistent_args(c));
  return DPD_OK;
}

// The persistent step's arguments for either buffer set, with the context's buffers of now.
hipError_t write_persistent_args(dpd_ctx *c) {
  for (int a = 0; a < 2 && c->pargs[1]; ++a) {
    const int b = 1 - a;
    dpd::PArgs A{};
    A.boxes = c->boxes;
    A.items = c->pitems;
    A.nitems = c->n_pitems;
    A.spin_limit = 1 << 16;
    A.need = c->pneed;
    A.arrive = c->parrive;
    A.head = c->phead;
    A.itiles = c->itiles;
    A.ftiles = c->ptiles;
    A.pos4 = c->pos[a];
    A.vel4 = c->vel[a];
    A.frc4 = c->frc[a];
    A.vt4 = c->vt;
    A.cell_of = c->cell_of;
    A.rank_of = c->rank_of;
    A.count = c->count;
    A.bits = c->bits;
    A.use_mask = c->use_mask;
    A.quad = c->quad;
    A.st = c->status;
    A.NF = c->NF;
    A.NW = c->NW;
    A.wcstart = c->wcstart;
    A.wcell = c->wcell;
    A.cstart = c->cstart;
    A.bsum = c->pbsum;
    A.start_all = c->start_all;
    A.fluid_off = c->fluid_off;
    A.idx = c->idx;
    A.idx_all = c->idx_all;
    A.cq = c->cq;
    A.pad = (int32_t)(c->NF + c->NW);
    A.ncell_all = (int32_t)c->NCELL;
    A.pos_out = c->pos[b];
    A.vel_out = c->vel[b];
    A.frc_out = c->frc[b];
    A.dk = c->dk;
    const hipError_t e = hipMemcpy(c->pargs[a], &A, sizeof(A), hipMemcpyHostToDevice);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// Cuts of one axis of n cells into bricks of at most B cells.  The brick at
// the high edge holds at most (n - 3) / 2 cells, so that every column its
// halo stages without wrapping lies at x >= L/2 and moves by -L exactly
// (Sterbenz); every axis needs at least two bricks.  Empty when the axis is
// too short (n < 5): such boxes take the per-particle kernel.
std::vector<std::pair<int, int>> axis_bricks(int n, int B) {
  std::vector<std::pair<int, int>> v;
  const int last = std::min(B, (n - 3) / 2);
  if (n < 5 || last < 1) return v;
  const int rest = n - last;
  for (int x = 0; x < rest; x += B) v.push_back({x, std::min(B, rest - x)});
  v.push_back({rest, last});
  return v;
}

// Brick table of every box that can be cut (x fastest, then y, then z, so
// that consecutive blocks work on neighbouring bricks), and the flag of the
// boxes that cannot.  The per-particle kernel is the default;
// DPD_PAIR_KERNEL=bricks in the environment at create selects the brick
// kernel for every box that can be cut.
int build_bricks(dpd_ctx *c) {
  const char *env = std::getenv("DPD_PAIR_KERNEL");
  const bool cells_only = !(env && std::strcmp(env, "bricks") == 0);
  std::vector<dpd::Brick> t;
  for (int r = 0; r < c->R; ++r) {
    Replica &p = c->rep[r];
    p.brick = false;
    if (cells_only || p.nf == 0) continue;
    const auto bx = axis_bricks(p.nc[0], dpd::kBrickX), by = axis_bricks(p.nc[1], dpd::kBrickY),
               bz = axis_bricks(p.nc[2], dpd::kBrickZ);
    if (bx.empty() || by.empty() || bz.empty()) continue;
    p.brick = true;
    for (const auto &z : bz)
      for (const auto &y : by)
        for (const auto &x : bx) {
          dpd::Brick b;
          b.box = r;
          b.x0 = x.first;
          b.sx = x.second;
          b.y0 = y.first;
          b.sy = y.second;
          b.z0 = z.first;
          b.sz = z.second;
          b.pad = 0;
          t.push_back(b);
        }
  }
  if (c->bricks) dfree(c, c->bricks);
  c->bricks = nullptr;
  c->nbricks = (int)t.size();
  if (t.empty()) return DPD_OK;
  c->bricks = (dpd::Brick *)dalloc(c, sizeof(dpd::Brick) * t.size());
  if (!c->bricks) return fail(c, DPD_E_NOMEM, "brick table allocation failed");
  HIP_TRY(c, hipMemcpyAsync(c->bricks, t.data(), sizeof(dpd::Brick) * t.size(),
                            hipMemcpyHostToDevice, c->stream));
  HIP_TRY(c, hipStreamSynchronize(c->stream));
  return DPD_OK;
}

// Bin the current fluid positions of every box (counting-sort pass 1).
int bin_all(dpd_ctx *c, hipStream_t s) {
  for (int r = 0; r < c->R; ++r) {
    const Replica &p = c->rep[r];
    HIP_TRY(c, timed(c, s, K_OTHER, [&] {
              return dpd::launch_bin(s, p.G, p.co, p.nf, c->pos[c->cur] + p.fo,
                                     c->cell_of + p.fo, c->rank_of + p.fo, c->count);
            }));
  }
  return DPD_OK;
}

// Cell list of the fluid at its current positions and the merged per-cell
// runs, with the runs' coarse position codes.  key4: sort each cell by gid (a
// state loaded from outside) instead of by storage index; bump: the force
// evaluation index advances in the same launches; codes = false: positions
// elsewhere than pos[cur] (the adjoint window's), whose pair walk does not
// read the codes; force_next: force_pass follows on the stream, which clears the
// cell counts where the list's own launch cannot.
int scan_scatter_sort(dpd_ctx *c, hipStream_t s, const float4 *key4 = nullptr,
                      unsigned long long *bump = nullptr, bool codes = true,
                      bool force_next = false) {
  if (c->box_list && !key4) {
    HIP_TRY(c, timed(c, s, K_SORT, [&] {
              return dpd::launch_cells_box(s, c->boxes, c->R, c->box_list, c->NF, c->cell_of, c->rank_of,
                                           c->count, c->wcstart, c->start_all, c->idx,
                                           c->idx_all, c->wcell, c->pos[c->cur],
                                           codes && !c->wide && c->box_codes ? c->cq : nullptr,
                                           bump);
            }));
    if (c->box_list > 1 && !force_next)
      HIP_TRY(c, dpd::launch_fill_zero(s, c->count, 4 * (size_t)c->NCELL));
  } else {
    HIP_TRY(c, timed(c, s, K_SCAN_REDUCE, [&] {
              return dpd::launch_scan_reduce(s, c->NCELL, c->count, c->bsum);
            }));
    HIP_TRY(c, timed(c, s, K_SCAN_DOWN, [&] {
              return dpd::launch_scan_down(s, c->NCELL, c->count, c->cstart, c->bsum, c->wcstart,
                                           c->start_all, c->fluid_off);
            }));
    HIP_TRY(c, timed(c, s, K_SCATTER, [&] {
              return dpd::launch_scatter(s, c->NF, c->cell_of, c->rank_of, c->cstart, c->idx,
                                         c->NW, c->wcell, c->wcstart, c->start_all, c->idx_all,
                                         bump);
            }));
    HIP_TRY(c, timed(c, s, K_SORT, [&] {
              return dpd::launch_sort_cells(s, c->NCELL, c->cstart, c->idx, key4, c->fluid_off,
                                            c->idx_all);
            }));
  }
  // the pair kernel with 16 lanes per particle reads no codes
  if (codes && !c->wide && (key4 || !c->box_codes))
    HIP_TRY(c, timed(c, s, K_CODES, [&] {
              return dpd::launch_quant_runs(s, c->NF + c->NW, c->idx_all, c->pos[c->cur], c->cq);
            }));
  return DPD_OK;
}

// The next drift in the pair kernel's launch, to pos and vt, binned into count2.
dpd::NextStep next_step(dpd_ctx *c, float4 *pos, float4 *vt) {
  return {c->bits,    c->use_mask, c->grid_f64, c->quad,
          pos,        vt,          c->cell_of,  c->rank_of,
          c->count2 ? c->count2 : c->count,
          c->reflect ? 1 : 0, c->wcstart};
}

// Forces at the current state in sorted order; init = 1 keeps velocities.
int force_pass(dpd_ctx *c, hipStream_t s, int init, const dpd::NextStep *next = nullptr) {
  const int a = c->cur, b = 1 - c->cur;
  int32_t *const clear = c->box_list > 1 ? c->count : nullptr;
  if (c->n_otiles > 0)
    HIP_TRY(c, timed(c, s, K_FORCE, [&] {
              if (c->wide)
                return dpd::launch_force_wide(s, c->boxes, c->otiles, c->n_otiles, c->NF, init,
                                              c->pos[a], c->vt, c->vel[a], c->frc[a], c->idx,
                                              c->idx_all, c->start_all, c->pos[b], c->vel[b],
                                              c->frc[b], c->dk, c->status, c->sph ? 1 : 0,
                                              clear, (int32_t)c->NCELL, next);
              return dpd::launch_force(s, c->fblock, c->boxes, c->otiles, c->n_otiles, c->NF,
                                       (int32_t)(c->NF + c->NW), (int32_t)c->NCELL, init,
                                       c->pos[a], c->vt, c->vel[a], c->frc[a], c->idx,
                                       c->idx_all, c->start_all, c->cq, c->pos[b], c->vel[b],
                                       c->frc[b], c->dk, c->status, c->sph ? 1 : 0, clear, next);
            }));
  if (c->nbricks > 0)
    HIP_TRY(c, timed(c, s, K_FORCE, [&] {
              return dpd::launch_force_brick(s, c->boxes, c->bricks, c->nbricks, c->NF,
                                             (int32_t)(c->NF + c->NW), init, c->pos[a], c->vt,
                                             c->vel[a], c->frc[a], c->idx_all, c->start_all,
                                             c->fluid_off, c->cstart, c->pos[b], c->vel[b],
                                             c->frc[b], c->dk, c->status, c->sph ? 1 : 0);
            }));
  c->cur = b;
  return DPD_OK;
}

// The walls of every box binned at their positions into wcell_tmp, wrank and wcount, with
// copies in wtmp and wvtmp; with move, those of every box whose solid moves first
// advance by dt v.
int bin_walls(dpd_ctx *c, hipStream_t s, int move) {
  float4 *wp = c->pos[c->cur] + c->NF, *wv = c->vt + c->NF;
  for (int r = 0; r < c->R; ++r) {
    const Replica &p = c->rep[r];
    if (p.nw == 0) continue;
    HIP_TRY(c, timed(c, s, K_OTHER, [&] {
              return dpd::launch_wall_move_bin(s, p.G, p.P.hdt, p.P.dt, move && p.moving ? 1 : 0,
                                               p.co, p.nw, wp + p.wo, wv + p.wo, c->wtmp + p.wo,
                                               c->wvtmp + p.wo, c->wcell_tmp + p.wo,
                                               c->wrank + p.wo, c->wcount);
            }));
  }
  return DPD_OK;
}

// The binned walls in the order idx, into both position buffers and both predictions.
int order_walls(dpd_ctx *c, hipStream_t s, const int32_t *idx) {
  const int a = c->cur, b = 1 - a;
  HIP_TRY(c, timed(c, s, K_OTHER, [&] {
            return dpd::launch_permute(s, c->NW, idx, c->wtmp, c->pos[a] + c->NF, c->wvtmp,
                                       c->vt + c->NF, c->wtmp, c->pos[b] + c->NF,
                                       c->vt2 ? c->wvtmp : nullptr,
                                       c->vt2 ? c->vt2 + c->NF : nullptr);
          }));
  return DPD_OK;
}

// A step's cell list where walls move: as scan_scatter_sort with the walls
// advanced by dt v and put back in cell order on the way.
int list_both(dpd_ctx *c, hipStream_t s) {
  int rc = bin_walls(c, s, 1);
  if (rc) return rc;
  const dpd::BothLists L = {c->NCELL, c->NF, c->NW, c->count, c->cstart, c->bsum, c->wcount,
                            c->wcstart, c->wsum, c->start_all, c->fluid_off, c->cell_of,
                            c->rank_of, c->wcell_tmp, c->wrank, c->idx, c->widx, c->idx_all,
                            c->wcell, c->dk};
  HIP_TRY(c, timed(c, s, K_SCAN_REDUCE, [&] {
            return dpd::launch_scan_reduce(s, c->NCELL, c->count, c->bsum, c->wcount, c->wsum);
          }));
  HIP_TRY(c, timed(c, s, K_SCAN_DOWN, [&] { return dpd::launch_scan_both(s, L); }));
  HIP_TRY(c, timed(c, s, K_SCATTER, [&] { return dpd::launch_scatter_both(s, L); }));
  HIP_TRY(c, timed(c, s, K_SORT, [&] { return dpd::launch_sort_both(s, L); }));
  rc = order_walls(c, s, c->widx);
  if (rc) return rc;
  if (!c->wide)
    HIP_TRY(c, timed(c, s, K_CODES, [&] {
              return dpd::launch_quant_runs(s, c->NF + c->NW, c->idx_all, c->pos[c->cur], c->cq);
            }));
  return DPD_OK;
}

// Walls re-sorted by cell after their positions changed outside a step.  Reads the
// walls at pos[cur] + NF (velocities at vt + NF), writes them back in cell
// order (within a cell by storage index) to both position buffers and vt,
// and rebuilds wcell and wcstart.
int wall_pass(dpd_ctx *c, hipStream_t s) {
  if (c->NW == 0) return DPD_OK;
  const int rc = bin_walls(c, s, 0);
  if (rc) return rc;
  HIP_TRY(c, timed(c, s, K_SCAN_REDUCE, [&] {
            return dpd::launch_scan_reduce(s, c->NCELL, c->wcount, c->bsum);
          }));
  HIP_TRY(c, timed(c, s, K_SCAN_DOWN, [&] {
            return dpd::launch_scan_down(s, c->NCELL, c->wcount, c->wcstart, c->bsum, nullptr,
                                         nullptr, nullptr);
          }));
  HIP_TRY(c, timed(c, s, K_SCATTER, [&] {
            return dpd::launch_scatter(s, c->NW, c->wcell_tmp, c->wrank, c->wcstart, c->idx);
          }));
  // per-cell sort, rebuilding wcell (the cell of each sorted wall) on the way
  HIP_TRY(c, timed(c, s, K_SORT, [&] {
            return dpd::launch_sort_wall_cells(s, c->NCELL, c->wcstart, c->idx, c->wcell);
          }));
  return order_walls(c, s, c->idx);
}

int drift(dpd_ctx *c, hipStream_t s) {
  const int a = c->cur;
  HIP_TRY(c, timed(c, s, K_INTEGRATE, [&] {
            return dpd::launch_integrate(s, c->ppt, c->boxes, c->itiles, c->n_itiles, c->pos[a],
                                         c->pos[a], c->vel[a], c->frc[a], c->vt, c->cell_of, c->rank_of,
                                         c->count, c->bits, c->use_mask, c->quad, c->grid_f64,
                                         c->status, c->NF, c->wcstart, c->reflect ? 1 : 0);
          }));
  return DPD_OK;
}

// The launches of one step on stream s (swaps cur).
int enqueue_step(dpd_ctx *c, hipStream_t s) {
  const int a = c->cur;
  if (c->persistent) {
    HIP_TRY(c, timed(c, s, K_PERSIST, [&] {
              return dpd::launch_step_persistent(
                  s, c->pargs[a], c->n_pitems, c->pblocks, c->parrive, dpd::kPhases * c->R,
                  c->phead, c->dk, c->grid_f64, c->ppt, c->reflect ? 1 : 0, c->sph ? 1 : 0);
            }));
    c->cur = 1 - a;
    return DPD_OK;
  }
  int rc = drift(c, s);
  if (rc) return rc;
  rc = c->moving ? list_both(c, s) : scan_scatter_sort(c, s, nullptr, c->dk, true, true);
  if (rc) return rc;
  return force_pass(c, s, 0);
}

// Capture the step from buffer set `from` into an executable graph.
int capture_step(dpd_ctx *c, int from) {
  if (!c->cap_stream) HIP_TRY(c, hipStreamCreateWithFlags(&c->cap_stream, hipStreamNonBlocking));
  const int saved = c->cur;
  c->cur = from;
  hipGraph_t g = nullptr;
  HIP_TRY(c, hipStreamBeginCapture(c->cap_stream, hipStreamCaptureModeThreadLocal));
  int rc = enqueue_step(c, c->cap_stream);
  hipError_t e = hipStreamEndCapture(c->cap_stream, &g);
  c->cur = saved;
  if (rc) {
    if (g) (void)hipGraphDestroy(g);
    return rc;
  }
  if (e != hipSuccess) return hip_fail(c, e, "hipStreamEndCapture");
  e = hipGraphInstantiate(&c->graph[from], g, nullptr, nullptr, 0);
  (void)hipGraphDestroy(g);
  if (e != hipSuccess) return hip_fail(c, e, "hipGraphInstantiate");
  return DPD_OK;
}

int one_step(dpd_ctx *c) {
  if (c->use_graph && !c->timing) {
    const int a = c->cur;
    if (!c->graph[a]) {
      int rc = capture_step(c, a);
      if (rc) return rc;
    }
    HIP_TRY(c, hipGraphLaunch(c->graph[a], c->stream));
    c->cur = 1 - a;
  } else {
    int rc = enqueue_step(c, c->stream);
    if (rc) return rc;
  }
  c->k += 1;
  c->steps += 1;
  return DPD_OK;
}

// n >= 2 steps in a row: the pair kernel goes on to the next step's drift, so only the
// first step has a launch for it.  The results are those of n steps one by one, and the
// launches are direct with use_graph too: they keep the GPU busier than a replay a
// step (16.2 against 20.5 us at 2,400 particles, 21.8 against 26.2 at 16,500).
int step_run(dpd_ctx *c, int64_t n) {
  int rc = drift(c, c->stream);
  for (int64_t s = 0; s < n && !rc; ++s) {
    const bool last = s + 1 == n;
    rc = c->moving ? list_both(c, c->stream)
                   : scan_scatter_sort(c, c->stream, nullptr, c->dk, true, true);
    if (rc) break;
    const dpd::NextStep next = next_step(c, c->pos[1 - c->cur], c->vt2);
    rc = force_pass(c, c->stream, 0, last ? nullptr : &next);
    if (!last) {
      std::swap(c->vt, c->vt2);
      if (c->count2) std::swap(c->count, c->count2);
    }
    c->k += 1;
    c->steps += 1;
  }
  return rc;
}

// n steps as a call of dpd_step takes them.
int run_steps(dpd_ctx *c, int64_t n) {
  if (n > 1 && c->vt2 && !c->persistent && !c->timing) return step_run(c, n);
  int rc = DPD_OK;
  for (int64_t s = 0; s < n && !rc; ++s) rc = one_step(c);
  return rc;
}

// Re-sort the fluid state into cell order after positions changed outside a
// step (set_state): bin, scan, scatter, sort, permute into the other buffers.
// Within a cell particles are ordered by gid, so the stored order (and with
// it every later summation order) depends only on the state, not on how the
// context stored its particles before.
int resort(dpd_ctx *c) {
  int rc = c->moving ? wall_pass(c, c->stream) : DPD_OK;
  if (!rc) rc = bin_all(c, c->stream);
  if (!rc) rc = scan_scatter_sort(c, c->stream, c->pos[c->cur]);
  if (rc) return rc;
  const int a = c->cur, b = 1 - a;
  HIP_TRY(c, dpd::launch_permute(c->stream, c->NF, c->idx, c->pos[a], c->pos[b], c->vel[a],
                                 c->vel[b], c->frc[a], c->frc[b]));
  c->cur = b;
  return DPD_OK;
}

// Host-side checks and splitting of one box's inputs.
struct HostBox {
  std::vector<float> pos, vel;
  std::vector<int32_t> type;
  std::vector<uint32_t> gid;
  std::vector<int64_t> rows_f, rows_w;
};

// Kernel parameters of a box from validated dpd_params (cells of R set).
void make_kparams(const dpd_params &P, const Replica &R, KParams &K) {
  K.a_ff = (float)P.a[0];
  K.a_fw = (float)P.a[1];
  K.gamma = (float)P.gamma;
  K.sigma_rdt = (float)(std::sqrt(2.0 * P.gamma * P.kBT) / std::sqrt(P.dt));
  K.rc2 = (float)(P.rc * P.rc);
  K.inv_rc = (float)(1.0 / P.rc);
  K.dt = (float)P.dt;
  K.hdt = (float)(0.5 * P.dt);
  K.lamdt = (float)(P.lambda * P.dt);
  for (int a = 0; a < 3; ++a) K.g[a] = (float)P.g[a];
  double wmin = R.L[0] / R.nc[0];
  for (int a = 1; a < 3; ++a) wmin = std::fmin(wmin, R.L[a] / R.nc[a]);
  K.max_disp2 = (float)(0.25 * wmin * wmin);
  {
    const double sigma = std::sqrt(2.0 * P.gamma * P.kBT);
    K.dsig_rdt = sigma > 0.0 ? (float)(P.kBT / (sigma * std::sqrt(P.dt))) : 0.0f;
  }
  K.key0 = (uint32_t)P.seed;
  K.key1 = (uint32_t)(P.seed >> 32);
  K.replica = P.replica;
  K.reflect = (R.moving ? dpd::kReflectMoving : 0u) |
              ((P.flags & DPD_FLAG_SPECULAR) ? dpd::kReflectSpecular : 0u);
  // Eq. 22-24: F_c = -cr P'(r / h_r) + ca P'(r / h_a), with c = S / (pi h^4)
  // and P' the derivative of Eq. 23's polynomial in v = r / h
  K.sph = (P.flags & DPD_FLAG_SPH) ? 1u : 0u;
  K.cr_ff = K.cr_fw = K.ca_ff = K.ca_fw = 0.f;
  K.inv_hr = K.inv_ha = 0.f;
  if (K.sph) {
    const double pi = 3.14159265358979323846;
    const double hr = 0.5 * P.r0r, ha = 0.5 * P.r0a;
    const double qr = 1.0 / (pi * hr * hr * hr * hr), qa = 1.0 / (pi * ha * ha * ha * ha);
    K.cr_ff = (float)(P.sr[0] * qr);
    K.cr_fw = (float)(P.sr[1] * qr);
    K.ca_ff = (float)(P.sa[0] * qa);
    K.ca_fw = (float)(P.sa[1] * qa);
    K.inv_hr = (float)(1.0 / hr);
    K.inv_ha = (float)(1.0 / ha);
  }
}

// Checks of dpd_params that need no particles.
std::string check_params(const dpd_params &P) {
  if (!(std::isfinite(P.rc) && P.rc > 0)) return "rc must be > 0";
  if (!(std::isfinite(P.dt) && P.dt > 0)) return "dt must be > 0";
  if (!(std::isfinite(P.gamma) && P.gamma >= 0) || !(std::isfinite(P.kBT) && P.kBT >= 0))
    return "gamma and kBT must be finite and >= 0";
  if (!std::isfinite(P.lambda)) return "lambda must be finite";
  for (int a = 0; a < 4; ++a)
    if (!std::isfinite(P.a[a])) return "a_ij must be finite";
  if (P.a[1] != P.a[2]) return "a_ij must be symmetric";
  for (int a = 0; a < 3; ++a)
    if (!std::isfinite(P.g[a])) return "g must be finite";
  if (P.replica >= 65536u) return "replica must be < 65536";
  if (P.flags & DPD_FLAG_SPH) {
    for (int a = 0; a < 4; ++a)
      if (!std::isfinite(P.sr[a]) || !std::isfinite(P.sa[a])) return "sr, sa must be finite";
    if (P.sr[1] != P.sr[2] || P.sa[1] != P.sa[2]) return "sr, sa must be symmetric";
    if (!(P.r0r > 0 && P.r0r <= P.rc && P.r0a > 0 && P.r0a <= P.rc))
      return "r0r and r0a must lie in (0, rc]";
  }
  return "";
}

int check_box(int r, const dpd_box *box, const dpd_particles *pp, const dpd_params *prm,
              const dpd_phi_grid *phi, Replica &R, HostBox &H) {
  const std::string pre = "box " + std::to_string(r) + ": ";
  if (!box || !pp || !prm || !phi) return fail(nullptr, DPD_E_INVAL, pre + "NULL argument");
  const dpd_params &P = *prm;
  for (int a = 0; a < 3; ++a)
    if (!(std::isfinite(box->L[a]) && box->L[a] > 0))
      return fail(nullptr, DPD_E_INVAL, pre + "box edges must be finite and positive");
  {
    const std::string e = check_params(P);
    if (!e.empty()) return fail(nullptr, DPD_E_INVAL, pre + e);
  }
  for (int a = 0; a < 3; ++a) {
    R.nc[a] = (int)std::floor(box->L[a] / P.rc);
    if (R.nc[a] < 3)
      return fail(nullptr, DPD_E_INVAL, pre + "box must hold at least 3 cells per axis");
  }
  R.ncell = (int64_t)R.nc[0] * R.nc[1] * R.nc[2];
  if (R.ncell > (int64_t)1 << 30) return fail(nullptr, DPD_E_INVAL, pre + "too many cells");
  if (!(phi->dtype == 4 || phi->dtype == 8))
    return fail(nullptr, DPD_E_INVAL, pre + "phi dtype must be 4 or 8");
  if (!phi->data) return fail(nullptr, DPD_E_INVAL, pre + "phi data is NULL");
  for (int a = 0; a < 3; ++a) {
    if (phi->n[a] < 2 || !(phi->h[a] > 0))
      return fail(nullptr, DPD_E_INVAL, pre + "phi grid needs >= 2 nodes and h > 0 per axis");
    if (std::fabs(phi->n[a] * phi->h[a] - box->L[a]) > 1e-9 * box->L[a])
      return fail(nullptr, DPD_E_INVAL, pre + "phi grid n*h must equal the box edge");
  }
  const int64_t n = pp->n;
  if (n < 0 || n >= ((int64_t)1 << 31))
    return fail(nullptr, DPD_E_INVAL, pre + "particle count out of range");
  if (n > 0 && (!pp->pos || !pp->vel || !pp->type))
    return fail(nullptr, DPD_E_INVAL, pre + "particle arrays are NULL");
  H.pos.resize(3 * (size_t)n);
  H.vel.resize(3 * (size_t)n);
  H.type.resize((size_t)n);
  H.gid.resize((size_t)n);
  if (n > 0) {
    if (pp->on_device) {
      if (hipMemcpy(H.pos.data(), pp->pos, 12 * (size_t)n, hipMemcpyDeviceToHost) != hipSuccess ||
          hipMemcpy(H.vel.data(), pp->vel, 12 * (size_t)n, hipMemcpyDeviceToHost) != hipSuccess ||
          hipMemcpy(H.type.data(), pp->type, 4 * (size_t)n, hipMemcpyDeviceToHost) != hipSuccess ||
          (pp->gid && hipMemcpy(H.gid.data(), pp->gid, 4 * (size_t)n, hipMemcpyDeviceToHost) !=
                          hipSuccess))
        return fail(nullptr, DPD_E_DEVICE, pre + "copying particle arrays failed");
    } else {
      std::memcpy(H.pos.data(), pp->pos, 12 * (size_t)n);
      std::memcpy(H.vel.data(), pp->vel, 12 * (size_t)n);
      std::memcpy(H.type.data(), pp->type, 4 * (size_t)n);
      if (pp->gid) std::memcpy(H.gid.data(), pp->gid, 4 * (size_t)n);
    }
  }
  if (!pp->gid)
    for (int64_t i = 0; i < n; ++i) H.gid[i] = (uint32_t)i;
  {
    std::vector<uint8_t> seen((size_t)n, 0);
    for (int64_t i = 0; i < n; ++i) {
      if (H.gid[i] >= (uint64_t)n || seen[H.gid[i]])
        return fail(nullptr, DPD_E_INVAL, pre + "gid must be a permutation of 0..n-1");
      seen[H.gid[i]] = 1;
    }
  }
  for (int64_t i = 0; i < n; ++i) {
    if (H.type[i] != DPD_TYPE_FLUID && H.type[i] != DPD_TYPE_WALL)
      return fail(nullptr, DPD_E_INVAL, pre + "type must be 0 (fluid) or 1 (wall)");
    if (!finite3(&H.pos[3 * i]) || !finite3(&H.vel[3 * i]))
      return fail(nullptr, DPD_E_INVAL, pre + "non-finite particle position or velocity");
    for (int a = 0; a < 3; ++a)
      if (!(H.pos[3 * i + a] >= 0.0f && H.pos[3 * i + a] < (float)box->L[a]))
        return fail(nullptr, DPD_E_INVAL, pre + "particle position outside [0, L)");
    (H.type[i] == DPD_TYPE_FLUID ? H.rows_f : H.rows_w).push_back(i);
  }
  R.n = n;
  R.nf = (int64_t)H.rows_f.size();
  R.nw = (int64_t)H.rows_w.size();
  // a wall particle's velocity is the velocity of its solid; nonzero ones
  // translate the walls, by less than half a cell per step
  for (int64_t i : H.rows_w) {
    const float *v = &H.vel[3 * i];
    if (v[0] != 0.0f || v[1] != 0.0f || v[2] != 0.0f) R.moving = true;
    for (int a = 0; a < 3; ++a)
      if (std::fabs((double)v[a]) * P.dt > 0.5 * box->L[a] / R.nc[a])
        return fail(nullptr, DPD_E_INVAL, pre + "a wall moves more than half a cell per step");
  }
  for (int a = 0; a < 3; ++a) {
    R.ng[a] = phi->n[a];
    R.L[a] = box->L[a];
    R.h[a] = phi->h[a];
    R.G.L[a] = (float)box->L[a];
    R.G.invw[a] = (float)((double)R.nc[a] / box->L[a]);
    R.G.nc[a] = R.nc[a];
    R.G.ng[a] = phi->n[a];
    R.G.inv_h[a] = (float)(1.0 / phi->h[a]);
    R.G.inv_h64[a] = 1.0 / phi->h[a];
    R.G.h[a] = (float)phi->h[a];
  }
  R.rc = P.rc;
  make_kparams(P, R, R.P);
  return DPD_OK;
}

int create_impl(int32_t nbox, const dpd_box *boxes, const dpd_particles *parts,
                const dpd_params *params, const dpd_phi_grid *grids,
                const dpd_allocator *alloc, void *hip_stream, dpd_ctx **out) {
  if (!out) return fail(nullptr, DPD_E_INVAL, "out is NULL");
  *out = nullptr;
  if (nbox < 1) return fail(nullptr, DPD_E_INVAL, "need at least one box");
  if (!boxes || !parts || !params || !grids) return fail(nullptr, DPD_E_INVAL, "NULL argument");

  // ---- host-side checks, which need no device ----
  std::vector<Replica> rep((size_t)nbox);
  std::vector<HostBox> host((size_t)nbox);
  for (int r = 0; r < nbox; ++r) {
    int rc = check_box(r, &boxes[r], &parts[r], &params[r], &grids[r], rep[r], host[r]);
    if (rc) return rc;
    if (grids[r].dtype != grids[0].dtype)
      return fail(nullptr, DPD_E_INVAL, "all phi grids of a batch must have the same dtype");
    if ((params[r].flags & DPD_FLAG_NO_MASK) != (params[0].flags & DPD_FLAG_NO_MASK))
      return fail(nullptr, DPD_E_INVAL, "all boxes of a batch must use the same flags");
  }
  int64_t NF = 0, NW = 0, NCELL = 0, NGRID = 0, NWORDS = 0;
  for (int r = 0; r < nbox; ++r) {
    Replica &p = rep[r];
    p.fo = NF;
    p.wo = NW;
    p.co = NCELL;
    p.go = NGRID;
    p.bo = NWORDS;
    const int64_t nodes = (int64_t)p.ng[0] * p.ng[1] * p.ng[2];
    p.nwords = (nodes + 31) / 32;
    NF += p.nf;
    NW += p.nw;
    NCELL += p.ncell;
    NGRID += nodes;
    NWORDS += p.nwords;
  }
  if (NF + NW + 1 >= ((int64_t)1 << 31) || NCELL >= ((int64_t)1 << 31))
    return fail(nullptr, DPD_E_INVAL, "too many particles or cells in total");

  // ---- device (after the host-side checks) ----
  int ndev = 0;
  if (hipGetDeviceCount(&ndev) != hipSuccess || ndev <= 0)
    return fail(nullptr, DPD_E_DEVICE, "no HIP device");
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return fail(nullptr, DPD_E_DEVICE, "hipGetDevice failed");
  {
    hipDeviceProp_t prop;
    if (hipGetDeviceProperties(&prop, dev) != hipSuccess)
      return fail(nullptr, DPD_E_DEVICE, "hipGetDeviceProperties failed");
    if (std::strncmp(prop.gcnArchName, "gfx950", 6) != 0)
      return fail(nullptr, DPD_E_DEVICE,
                  std::string("library built for gfx950, device is ") + prop.gcnArchName);
  }

  // ---- context ----
  dpd_ctx *c = new (std::nothrow) dpd_ctx();
  if (!c) return fail(nullptr, DPD_E_NOMEM, "host allocation failed");
  c->device = dev;
  c->stream = (hipStream_t)hip_stream;
  if (alloc && alloc->alloc && alloc->free) {
    c->al = *alloc;
    c->has_al = true;
  }
  c->R = nbox;
  c->rep = rep;
  c->NF = NF;
  c->NW = NW;
  c->NCELL = NCELL;
  c->NGRID = NGRID;
  c->NWORDS = NWORDS;
  c->grid_f64 = grids[0].dtype == 8;
  c->use_mask = (params[0].flags & DPD_FLAG_NO_MASK) ? 0 : 1;
  auto bail = [c](int code) { return abandon_create(c, code); };

  // ---- device buffers ----
  const size_t nf = (size_t)NF, nw = (size_t)NW, ncell = (size_t)NCELL;
  for (int b = 0; b < 2; ++b) {
    c->pos[b] = (float4 *)dalloc(c, 16 * (nf + nw + 1));
    c->vel[b] = (float4 *)dalloc(c, 16 * nf);
    c->frc[b] = (float4 *)dalloc(c, 16 * nf);
  }
  c->vt = (float4 *)dalloc(c, 16 * (nf + nw + 1));
  c->cell_of = (int32_t *)dalloc(c, 4 * std::max(nf, nw));
  c->rank_of = (int32_t *)dalloc(c, 4 * std::max(nf, nw));
  c->idx = (int32_t *)dalloc(c, 4 * std::max(nf, nw));
  c->count = (int32_t *)dalloc(c, 4 * ncell);
  c->cstart = (int32_t *)dalloc(c, 4 * (ncell + 1));
  c->nscan = dpd::scan_blocks(NCELL);
  c->bsum = (int32_t *)dalloc(c, 4 * (size_t)c->nscan);
  c->wcstart = (int32_t *)dalloc(c, 4 * (ncell + 1));
  c->wcell = (int32_t *)dalloc(c, 4 * nw);
  c->idx_all = (int32_t *)dalloc(c, 4 * (nf + nw + dpd::kIdxSlack));
  c->cq = (uint32_t *)dalloc(c, 4 * (nf + nw + dpd::kIdxSlack));
  for (const Replica &p : c->rep) {
    c->moving = c->moving || p.moving;
    c->reflect = c->reflect || p.P.reflect != 0;
    c->sph = c->sph || p.P.sph != 0;
  }
  if (c->moving) {
    c->wtmp = (float4 *)dalloc(c, 16 * nw);
    c->wvtmp = (float4 *)dalloc(c, 16 * nw);
    c->wcell_tmp = (int32_t *)dalloc(c, 4 * nw);
    c->wrank = (int32_t *)dalloc(c, 4 * nw);
    c->wcount = (int32_t *)dalloc(c, 4 * ncell);
    c->widx = (int32_t *)dalloc(c, 4 * std::max<size_t>((size_t)NW, 1));
    c->wsum = (int32_t *)dalloc(c, 4 * (size_t)c->nscan);
    if (!c->wtmp || !c->wvtmp || !c->wcell_tmp || !c->wrank || !c->wcount || !c->widx || !c->wsum)
      return bail(fail(c, DPD_E_NOMEM, "device allocation failed"));
  }
  c->start_all = (int32_t *)dalloc(c, 4 * (ncell + 1 + dpd::kStartSlack));
  c->fluid_off = (int32_t *)dalloc(c, 4 * ncell);
  c->grid = dalloc(c, (size_t)NGRID * (size_t)grids[0].dtype);
  c->quad = dalloc(c, 4 * (size_t)NGRID * (size_t)grids[0].dtype);
  c->bits = (uint32_t *)dalloc(c, 4 * (size_t)NWORDS);
  c->boxes = (Box *)dalloc(c, sizeof(Box) * (size_t)nbox);
  c->status = (Status *)dalloc(c, sizeof(StatusBlock));
  if (hipHostMalloc((void **)&c->note, sizeof(Status), hipHostMallocDefault) != hipSuccess)
    c->note = nullptr;
  c->dk = (unsigned long long *)dalloc(c, 8);
  c->pair_counter = (unsigned long long *)dalloc(c, 8);
  for (int b = 0; b < 2; ++b)
    if (!c->pos[b] || !c->vel[b] || !c->frc[b])
      return bail(fail(c, DPD_E_NOMEM, "device allocation failed"));
  if (!c->vt || !c->cell_of || !c->rank_of || !c->idx || !c->count || !c->cstart || !c->bsum ||
      !c->wcstart || !c->wcell || !c->idx_all || !c->cq || !c->start_all || !c->fluid_off ||
      !c->grid || !c->quad ||
      !c->bits || !c->boxes || !c->status || !c->note || !c->dk || !c->pair_counter)
    return bail(fail(c, DPD_E_NOMEM, "device allocation failed"));

  int rc = DPD_OK;
  auto chk = [&](hipError_t e, const char *w) {
    if (e != hipSuccess && rc == DPD_OK) rc = hip_fail(c, e, w);
  };
  chk(dpd::launch_fill_zero(c->stream, c->status, sizeof(StatusBlock)), "zero status");
  chk(dpd::launch_fill_zero(c->stream, c->count, 4 * ncell), "zero counts");
  chk(dpd::launch_fill_zero(c->stream, c->pair_counter, 8), "zero counter");
  chk(dpd::launch_fill_zero(c->stream, c->dk, 8), "zero k");
  for (int r = 0; r < nbox; ++r) {
    const Replica &p = c->rep[r];
    const size_t gb = (size_t)p.ng[0] * p.ng[1] * p.ng[2] * (size_t)grids[0].dtype;
    chk(hipMemcpyAsync((char *)c->grid + (size_t)p.go * grids[0].dtype, grids[r].data, gb,
                       grids[r].on_device ? hipMemcpyDeviceToDevice : hipMemcpyHostToDevice,
                       c->stream),
        "upload phi");
  }
  if (rc) return bail(rc);

  // ---- particles: fluid into its slots, walls sorted by cell (once) ----
  {
    float4 *wtmp = (float4 *)dalloc(c, 16 * std::max<size_t>(nw, 1));
    float4 *wvel = (float4 *)dalloc(c, 16 * std::max<size_t>(nw, 1));
    if (!wtmp || !wvel) return bail(fail(c, DPD_E_NOMEM, "staging allocation failed"));
    for (int r = 0; r < nbox && !rc; ++r) {
      const Replica &p = c->rep[r];
      const HostBox &H = host[r];
      const size_t nn = (size_t)std::max<int64_t>(p.n, 1);
      float *dpos = (float *)dalloc(c, 12 * nn);
      float *dvel = (float *)dalloc(c, 12 * nn);
      uint32_t *dgid = (uint32_t *)dalloc(c, 4 * nn);
      int64_t *drows = (int64_t *)dalloc(c, 8 * nn);
      if (!dpos || !dvel || !dgid || !drows)
        return bail(fail(c, DPD_E_NOMEM, "staging allocation failed"));
      if (p.n > 0) {
        chk(hipMemcpyAsync(dpos, H.pos.data(), 12 * (size_t)p.n, hipMemcpyHostToDevice, c->stream), "upload pos");
        chk(hipMemcpyAsync(dvel, H.vel.data(), 12 * (size_t)p.n, hipMemcpyHostToDevice, c->stream), "upload vel");
        chk(hipMemcpyAsync(dgid, H.gid.data(), 4 * (size_t)p.n, hipMemcpyHostToDevice, c->stream), "upload gid");
      }
      if (p.nf > 0) {
        chk(hipMemcpyAsync(drows, H.rows_f.data(), 8 * (size_t)p.nf, hipMemcpyHostToDevice, c->stream), "rows");
        chk(dpd::launch_pack(c->stream, p.nf, dpos, dvel, dgid, drows, c->pos[0] + p.fo,
                             c->vel[0] + p.fo, c->vt + p.fo, c->frc[0] + p.fo),
            "pack fluid");
      }
      if (p.nw > 0) {
        chk(hipStreamSynchronize(c->stream), "sync");
        chk(hipMemcpyAsync(drows, H.rows_w.data(), 8 * (size_t)p.nw, hipMemcpyHostToDevice, c->stream), "rows");
        chk(dpd::launch_pack(c->stream, p.nw, dpos, dvel, dgid, drows, wtmp + p.wo,
                             wvel + p.wo, nullptr, nullptr),
            "pack walls");
        chk(dpd::launch_bin(c->stream, p.G, p.co, p.nw, wtmp + p.wo, c->cell_of + p.wo,
                            c->rank_of + p.wo, c->count),
            "bin walls");
      }
      chk(hipStreamSynchronize(c->stream), "sync");
      for (void *q : {(void *)dpos, (void *)dvel, (void *)dgid, (void *)drows}) dfree(c, q);
    }
    chk(dpd::launch_scan_reduce(c->stream, NCELL, c->count, c->bsum), "scan");
    chk(dpd::launch_scan_down(c->stream, NCELL, c->count, c->wcstart, c->bsum, nullptr, nullptr,
                              nullptr),
        "scan");
    if (nw > 0) {
      // walls sorted by global cell (so each box's walls stay contiguous)
      // into the tail of both position buffers, with their solid's velocity
      // as predicted velocity
      chk(dpd::launch_scatter(c->stream, NW, c->cell_of, c->rank_of, c->wcstart, c->idx),
          "scatter walls");
      chk(dpd::launch_sort_cells(c->stream, NCELL, c->wcstart, c->idx, nullptr, nullptr, nullptr),
          "sort walls");
      chk(dpd::launch_permute(c->stream, NW, c->idx, wtmp, c->pos[0] + nf, wvel, c->vt + nf,
                              nullptr, nullptr),
          "permute walls");
      chk(hipMemcpyAsync(c->pos[1] + nf, c->pos[0] + nf, 16 * nw, hipMemcpyDeviceToDevice,
                         c->stream),
          "copy walls");
      for (int r = 0; r < nbox; ++r) {
        const Replica &p = c->rep[r];
        chk(dpd::launch_cells(c->stream, p.G, p.co, p.nw, c->pos[0] + nf + p.wo, c->wcell + p.wo),
            "wall cells");
      }
    }
    // the wall counts start at zero (each wall pass leaves them zero again)
    if (c->moving) chk(dpd::launch_fill_zero(c->stream, c->wcount, 4 * ncell), "zero wall counts");
    chk(dpd::launch_set_pad(c->stream, c->pos[0] + nf + nw, c->vt + nf + nw, c->idx_all + nf + nw,
                            (int32_t)(nf + nw)), "pad");
    chk(dpd::launch_set_pad(c->stream, c->pos[1] + nf + nw, nullptr, nullptr, 0), "pad");
    chk(hipStreamSynchronize(c->stream), "sync");
    dfree(c, wtmp);
    dfree(c, wvel);
    if (rc) return bail(rc);
  }

  // ---- phase field: cube masks and create-time checks ----
  for (int r = 0; r < nbox; ++r) {
    const Replica &p = c->rep[r];
    const size_t es = (size_t)grids[0].dtype;
    const void *g = (const char *)c->grid + (size_t)p.go * es;
    chk(dpd::launch_cube_mask(c->stream, p.G, g, c->grid_f64, p.nwords, c->bits + p.bo), "mask");
    chk(dpd::launch_build_quad(c->stream, p.G, g, c->grid_f64,
                               (char *)c->quad + 4 * (size_t)p.go * es),
        "phase-field layout");
    chk(dpd::launch_check_grid(c->stream, g, c->grid_f64, (int64_t)p.ng[0] * p.ng[1] * p.ng[2],
                               c->status),
        "check grid");
    chk(dpd::launch_check_phi(c->stream, p.G, g, c->grid_f64, p.nf, c->pos[0] + p.fo, c->status),
        "check phi");
  }
  if (rc) return bail(rc);
  {
    Status st;
    int r2 = read_status(c, st);
    if (r2) return bail(r2);
    if (st.bad_grid)
      return bail(fail(c, DPD_E_INVAL, std::to_string(st.bad_grid) + " non-finite phi values"));
    if (st.bad_phi)
      return bail(fail(c, DPD_E_INVAL,
                       std::to_string(st.bad_phi) + " fluid particles start at phi < 0"));
    std::vector<uint32_t> hb((size_t)NWORDS);
    chk(hipMemcpy(hb.data(), c->bits, 4 * (size_t)NWORDS, hipMemcpyDeviceToHost), "mask readback");
    if (rc) return bail(rc);
    for (int r = 0; r < nbox; ++r) {
      int64_t m = 0;
      for (int64_t w = 0; w < c->rep[r].nwords; ++w) m += __builtin_popcount(hb[c->rep[r].bo + w]);
      c->rep[r].flagged_cubes = m;
    }
  }

  // ---- descriptors, tiles, initial cell list and forces f(0) with k = 0 ----
  {
    std::vector<Box> hb((size_t)nbox);
    for (int r = 0; r < nbox; ++r) {
      const Replica &p = c->rep[r];
      hb[r].G = p.G;
      hb[r].P = p.P;
      hb[r].fo = p.fo;
      hb[r].nf = p.nf;
      hb[r].wo = p.wo;
      hb[r].nw = p.nw;
      hb[r].co = p.co;
      hb[r].ncell = p.ncell;
      hb[r].go = p.go;
      hb[r].bo = p.bo;
    }
    chk(hipMemcpy(c->boxes, hb.data(), sizeof(Box) * (size_t)nbox, hipMemcpyHostToDevice),
        "upload boxes");
    if (rc) return bail(rc);
  }
  rc = build_bricks(c);
  c->wide = use_wide(c);
  c->box_list = box_parts(c);
  // a box's 16 blocks write the codes too, a launch less (16 cylinder cells: 63.1 to
  // 61.6 us a step); fewer blocks of large boxes take longer than the launch (64
  // uneven boxes, 4 each: 110.9 to 112.1)
  c->box_codes = c->box_list == 16;
  if (!rc) rc = set_shapes(c, default_ppt(c), 256);
  // steps in a row (step_run), where the buffers can be had
  if (!rc && c->nbricks == 0 && (!c->wide || c->n_otiles <= kRunTiles)) {
    const size_t vt_bytes = 16 * (size_t)(c->NF + c->NW + 1), count_bytes = 4 * (size_t)c->NCELL;
    c->vt2 = (float4 *)dalloc(c, vt_bytes, true);
    if (c->vt2 && c->box_list) c->count2 = (int32_t *)dalloc(c, count_bytes, true);
    if (c->vt2 && (c->count2 || !c->box_list)) {
      chk(hipMemcpyAsync(c->vt2, c->vt, vt_bytes, hipMemcpyDeviceToDevice, c->stream),
          "copy predictions");   // the walls' velocities
      if (c->count2) chk(dpd::launch_fill_zero(c->stream, c->count2, count_bytes), "zero counts");
    } else {
      if (c->vt2) dfree(c, c->vt2);
      c->vt2 = nullptr;
    }
  }
  if (rc) return bail(rc);
  c->cur = 0;
  c->k = 0;
  rc = bin_all(c, c->stream);
  if (!rc) rc = scan_scatter_sort(c, c->stream, nullptr, nullptr, true, true);
  if (!rc) rc = force_pass(c, c->stream, 1);
  if (!rc) {
    hipError_t e = hipStreamSynchronize(c->stream);
    if (e != hipSuccess) rc = hip_fail(c, e, "initial forces");
  }
  if (!rc) rc = latched_error(c);
  if (rc) return bail(rc);
  *out = c;
  return DPD_OK;
}

int check_replica(dpd_ctx *c, int32_t r) {
  if (r < 0 || r >= c->R) return fail(c, DPD_E_INVAL, "replica index out of range");
  return DPD_OK;
}

// Time a call of `steps` steps with the current shapes from the saved state; returns ms.
int trial(dpd_ctx *c, int steps, float *ms) {
  hipEvent_t a = get_event(c), b = get_event(c);
  // warm-up, and where steps are replayed the capture from either buffer set
  int rc = run_steps(c, steps > 1 ? 2 : 1);
  if (!rc && steps == 1) rc = run_steps(c, 1);
  if (!rc) (void)hipEventRecord(a, c->stream);
  if (!rc) rc = run_steps(c, steps);
  if (!rc) (void)hipEventRecord(b, c->stream);
  if (!rc) {
    hipError_t e = hipEventSynchronize(b);
    if (e != hipSuccess)
      rc = hip_fail(c, e, "autotune");
    else if (hipEventElapsedTime(ms, a, b) != hipSuccess)
      rc = fail(c, DPD_E_DEVICE, "timing");
  }
  c->free_events.push_back(a);
  c->free_events.push_back(b);
  return rc;
}

std::string tune_signature(dpd_ctx *c) {
  hipDeviceProp_t prop;
  std::string dev = "unknown";
  if (hipGetDeviceProperties(&prop, c->device) == hipSuccess) dev = prop.gcnArchName;
  for (auto &ch : dev)
    if (ch == ' ') ch = '_';
  std::ostringstream s;
  s << dev << ":R" << c->R << ":F" << c->NF << ":W" << c->NW << ":C" << c->NCELL << ":g"
    << (c->use_graph ? 1 : 0);
  return s.str();
}


// ---- adjoint form: window forward and backward sweep ----

// Copy the fluid state (pos, vel, frc of the current buffers) to/from a
// 3 x NF block.
int save_state(dpd_ctx *c, float4 *dst) {
  const size_t b = 16 * (size_t)c->NF;
  if (!b) return DPD_OK;
  HIP_TRY(c, hipMemcpyAsync(dst, c->pos[c->cur], b, hipMemcpyDeviceToDevice, c->stream));
  HIP_TRY(c, hipMemcpyAsync(dst + c->NF, c->vel[c->cur], b, hipMemcpyDeviceToDevice, c->stream));
  HIP_TRY(c, hipMemcpyAsync(dst + 2 * c->NF, c->frc[c->cur], b, hipMemcpyDeviceToDevice,
                            c->stream));
  return DPD_OK;
}

int load_state(dpd_ctx *c, const float4 *src) {
  const size_t b = 16 * (size_t)c->NF;
  if (!b) return DPD_OK;
  HIP_TRY(c, hipMemcpyAsync(c->pos[c->cur], src, b, hipMemcpyDeviceToDevice, c->stream));
  HIP_TRY(c, hipMemcpyAsync(c->vel[c->cur], src + c->NF, b, hipMemcpyDeviceToDevice, c->stream));
  HIP_TRY(c, hipMemcpyAsync(c->frc[c->cur], src + 2 * c->NF, b, hipMemcpyDeviceToDevice,
                            c->stream));
  return DPD_OK;
}

// Carried force recomputed at the current (r, v) with the current
// parameters and k: f = F(r, vt = v) + g (as at create).
int refresh_forces(dpd_ctx *c) {
  int rc = bin_all(c, c->stream);
  if (!rc) rc = scan_scatter_sort(c, c->stream, nullptr, nullptr, true, true);
  if (rc) return rc;
  HIP_TRY(c, dpd::launch_vt_from_v(c->stream, c->NF, c->vel[c->cur], c->vt));
  return force_pass(c, c->stream, 1);
}

template <typename P>
int grow(dpd_ctx *c, P **ptr, size_t count, int *cap, int want) {
  if (*ptr && *cap >= want) return DPD_OK;
  if (*ptr) dfree(c, *ptr);
  *ptr = (P *)dalloc(c, sizeof(P) * std::max<size_t>(count, 1));
  if (!*ptr) return fail(c, DPD_E_NOMEM, "window buffer allocation failed");
  *cap = want;
  return DPD_OK;
}

// One step of a stored window: X (3 x NF: the state it starts from), the drifted
// positions D and predicted velocities V (NF + NW + 1 records, walls and pad at
// the end) and its cell list.  Steps are `stride` bytes apart, a multiple of 256.
struct StoredStep {
  float4 *X, *D, *V;
  int32_t *idx, *idx_all, *start_all;
};

struct StoreLayout {
  size_t d, v, idx, idx_all, start_all, stride;   // byte offsets within a step
  explicit StoreLayout(const dpd_ctx *c) {
    const size_t nf = (size_t)c->NF, nrec = nf + (size_t)c->NW + 1;
    auto up = [](size_t b) { return (b + 255) & ~(size_t)255; };
    d = up(48 * nf);
    v = d + up(16 * nrec);
    idx = v + up(16 * nrec);
    idx_all = idx + up(4 * nf);
    start_all = idx_all + up(4 * (nrec - 1 + dpd::kIdxSlack));
    stride = start_all + up(4 * ((size_t)c->NCELL + 1 + dpd::kStartSlack));
  }
};

StoredStep stored_step(const dpd_ctx *c, int t) {
  const StoreLayout l(c);
  char *p = c->win.store + (size_t)t * l.stride;
  return {(float4 *)p,           (float4 *)(p + l.d),         (float4 *)(p + l.v),
          (int32_t *)(p + l.idx), (int32_t *)(p + l.idx_all), (int32_t *)(p + l.start_all)};
}

// Windows of up to this many bytes are kept whole, whatever their ckpt.  A step of the
// 20^3 slit (19,700 particles) takes 1.9 MB; keeping its 24-step window, the sweep
// launches two kernels per step, and one before the first, instead of recomputing the
// segment and then each step's drift and cell list.  Larger windows keep a state every
// ckpt steps, as do those whose store cannot be allocated.  The store stays for the
// windows to come, until one does not use it (window_alloc) or its memory is
// needed (give_back).
constexpr size_t kWindowStore = (size_t)2 << 30;

// The state a segment starts from.
const float4 *segment_start(const dpd_ctx *c, int seg) {
  const Window &W = c->win;
  return W.full ? stored_step(c, seg * W.ckpt).X : W.ck + (size_t)seg * 3 * c->NF;
}

// Per-block partial sums of the backward sweep's kernels.
int window_partials(dpd_ctx *c) {
  Window &W = c->win;
  const int nb_f = dpd::force_vjp_blocks(c->n_ftiles), nb_g = dpd::adj_prep_blocks(c->NF);
  const int rc = grow(c, &W.part_f, 3 * (size_t)std::max(nb_f, 1), &W.cap_f, nb_f);
  return rc ? rc : grow(c, &W.part_g, 3 * (size_t)std::max(nb_g, 1), &W.cap_g, nb_g);
}

int window_alloc(dpd_ctx *c, int steps, int ckpt, int nbins) {
  Window &W = c->win;
  const size_t nf = (size_t)std::max<int64_t>(c->NF, 1);
  const int nck = (steps + ckpt - 1) / ckpt;
  if (W.nf != c->NF) {
    // sizes depend on NF: start over
    for (void *q : {(void *)W.ck, (void *)W.seg, (void *)W.save, (void *)W.wpos, (void *)W.adj})
      if (q) dfree(c, q);
    W.ck = W.seg = W.save = W.wpos = W.adj = nullptr;
    W.cap_nck = W.cap_ckpt = 0;
    W.nf = c->NF;
  }
  int dummy = 0;
  int rc = DPD_OK;
  if (!W.save) rc = grow(c, &W.save, 3 * nf, &dummy, 1);
  if (!rc && !W.wpos) rc = grow(c, &W.wpos, (size_t)(c->NF + c->NW + 1), &dummy, 1);
  if (!rc && !W.adj) rc = grow(c, &W.adj, 11 * nf, &dummy, 1);
  if (!rc && W.cap_nbins < nbins) {
    for (void *q : {(void *)W.sums, (void *)W.counts, (void *)W.lw})
      if (q) dfree(c, q);
    W.sums = nullptr;
    W.counts = nullptr;
    W.lw = nullptr;
    W.sums = (double *)dalloc(c, 8 * (size_t)nbins);
    W.counts = (unsigned long long *)dalloc(c, 8 * (size_t)nbins);
    W.lw = (float *)dalloc(c, 4 * (size_t)nbins);
    if (!W.sums || !W.counts || !W.lw) return fail(c, DPD_E_NOMEM, "window buffer allocation failed");
    W.cap_nbins = nbins;
  }
  if (!rc && !W.acc) {
    W.acc = (double *)dalloc(c, 8 * 8);
    W.dk0 = (unsigned long long *)dalloc(c, 8);
    W.status_save = (Status *)dalloc(c, sizeof(StatusBlock));
    if (!W.acc || !W.dk0 || !W.status_save)
      return fail(c, DPD_E_NOMEM, "window buffer allocation failed");
  }
  if (!rc) rc = window_partials(c);
  // the store last, so that it takes nothing that a window has to have; one that does not
  // serve this window goes back
  const size_t want = StoreLayout(c).stride * (size_t)steps;
  const bool fits = c->NF > 0 && c->nbricks == 0 && want <= kWindowStore;
  if (!fits || W.store_cap < want) free_store(W, c);
  if (!rc && fits && !W.store) {
    W.store = (char *)dalloc(c, want, true);
    W.store_cap = W.store ? want : 0;
  }
  W.full = W.store != nullptr;
  if (!rc && !W.full) rc = grow(c, &W.ck, 3 * nf * (size_t)nck, &W.cap_nck, nck);
  if (!rc && !W.full) rc = grow(c, &W.seg, 3 * nf * (size_t)ckpt, &W.cap_ckpt, ckpt);
  return rc;
}

// Step t of a window that is kept whole: its launches read and write the
// store's arrays in place of the context's (the last step's new state goes to
// the context), so nothing is copied.
int stored_window_step(dpd_ctx *c, int t, bool last) {
  const StoredStep st = stored_step(c, t);
  const int64_t NF = c->NF;
  const int a = c->cur, b = 1 - a;
  float4 *const next = last ? nullptr : stored_step(c, t + 1).X;
  const bool row = c->vt2 && !c->timing;   // as step_run: the drifts in the pair kernel
  struct Saved {
    float4 *pos[2], *vel[2], *frc[2], *vt;
    int32_t *idx, *idx_all, *start_all;
  } keep = {{c->pos[0], c->pos[1]}, {c->vel[0], c->vel[1]}, {c->frc[0], c->frc[1]}, c->vt,
            c->idx, c->idx_all, c->start_all};
  c->pos[a] = st.D;
  c->vel[a] = st.X + NF;
  c->frc[a] = st.X + 2 * NF;
  c->vt = st.V;
  c->idx = st.idx;
  c->idx_all = st.idx_all;
  c->start_all = st.start_all;
  if (next) {
    c->pos[b] = next;
    c->vel[b] = next + NF;
    c->frc[b] = next + 2 * NF;
  }
  auto launches = [&]() -> int {
    if (t == 0 || !row)
      HIP_TRY(c, timed(c, c->stream, K_INTEGRATE, [&] {
              return dpd::launch_integrate(c->stream, c->ppt, c->boxes, c->itiles, c->n_itiles,
                                           st.X, st.D, st.X + NF, st.X + 2 * NF, st.V, c->cell_of,
                                           c->rank_of, c->count, c->bits, c->use_mask, c->quad,
                                           c->grid_f64, c->status, NF, c->wcstart, 0);
            }));
    int rc = scan_scatter_sort(c, c->stream, nullptr, c->dk, true, true);
    if (rc || !row || last) return rc ? rc : force_pass(c, c->stream, 0);
    const dpd::NextStep drifted = next_step(c, stored_step(c, t + 1).D, stored_step(c, t + 1).V);
    rc = force_pass(c, c->stream, 0, &drifted);
    if (c->count2) std::swap(c->count, c->count2);
    return rc;
  };
  const int rc = launches();
  for (int q = 0; q < 2; ++q) {
    c->pos[q] = keep.pos[q];
    c->vel[q] = keep.vel[q];
    c->frc[q] = keep.frc[q];
  }
  c->vt = keep.vt;
  c->idx = keep.idx;
  c->idx_all = keep.idx_all;
  c->start_all = keep.start_all;
  c->cur = rc || !last ? a : b;
  if (rc) return rc;
  c->k += 1;
  c->steps += 1;
  return DPD_OK;
}

// The steps of a window that is kept whole, and its bin sums.
int stored_window(dpd_ctx *c) {
  Window &W = c->win;
  const StoreLayout l(c);
  const int64_t NF = c->NF, stride = (int64_t)(l.stride / 16);
  const StoredStep s0 = stored_step(c, 0);
  int rc = save_state(c, s0.X);
  if (rc) return rc;
  HIP_TRY(c, dpd::launch_store_walls(c->stream, c->NW + 1, W.steps, stride, c->pos[c->cur] + NF,
                                     c->vt + NF, s0.D + NF, s0.V + NF, (int64_t)(l.stride / 4),
                                     s0.idx_all + NF + c->NW, (int32_t)(NF + c->NW)));
  for (int t = 0; t < W.steps; ++t) {
    rc = stored_window_step(c, t, t == W.steps - 1);
    if (rc) return rc;
  }
  // the states after steps 1 .. steps - 1 start the next steps; the last is the context's
  if (W.steps > 1) {
    const float4 *x = stored_step(c, 1).X;
    HIP_TRY(c, dpd::launch_obs(c->stream, NF, W.steps - 1, stride, x, x + NF, W.axis, W.nbins,
                               W.scale, W.sums, W.counts));
  }
  HIP_TRY(c, dpd::launch_obs(c->stream, NF, 1, 0, c->pos[c->cur], c->vel[c->cur], W.axis, W.nbins,
                             W.scale, W.sums, W.counts));
  return DPD_OK;
}

// The preparation of step t's VJP from the arrays st, velocities' adjoints to vn.
dpd::AdjPrep adj_prep(dpd_ctx *c, const StoredStep &st, float4 *vn) {
  Window &W = c->win;
  const int64_t NF = c->NF;
  return {st.idx, st.D,  st.V, W.lw,       W.axis, W.nbins, W.scale, W.adj + 6 * NF,
          vn,     W.adj + 8 * NF, W.part_g};
}

// The VJP kernels of step t from its arrays st, prepared with the velocities' adjoints vn.
// With next, the preparation of the step before follows in the same launch, else B
// receives the adjoints of X_t.
int step_vjp(dpd_ctx *c, const StoredStep &st, uint64_t t, const float4 *vn, float4 *B,
             const dpd::AdjPrep *next, double *dphi) {
  Window &W = c->win;
  const int64_t NF = c->NF;
  hipStream_t s = c->stream;
  float4 *rn = W.adj + 6 * NF, *fbar = W.adj + 8 * NF;
  float4 *rt = W.adj + 9 * NF, *vtb = W.adj + 10 * NF;
  HIP_TRY(c, dpd::launch_force_vjp(s, c->wide ? 0 : c->fblock, c->boxes, c->ftiles, c->n_ftiles,
                                   NF, (int32_t)(NF + c->NW), st.D, st.V, st.idx, st.idx_all,
                                   st.start_all, fbar, rn, rt, vtb, W.dk0, t + 1, W.part_f));
  HIP_TRY(c, dpd::launch_integrate_vjp(s, c->boxes, NF, st.X, st.X + NF, st.X + 2 * NF, st.V, rt,
                                       vtb, vn, c->grid, c->grid_f64, dphi, B, B + NF,
                                       B + 2 * NF, next));
  return DPD_OK;
}

// The backward sweep of a window kept whole: A holds the adjoints of the last state (slot
// order; its memory is used), B receives those of the first.
int stored_sweep(dpd_ctx *c, float4 *A, float4 *B, double *dphi) {
  Window &W = c->win;
  const int64_t NF = c->NF;
  float4 *vn = W.adj + 7 * NF, *other = A;
  HIP_TRY(c, dpd::launch_adj_prep(c->stream, c->boxes, NF, 0, A, A + NF, A + 2 * NF,
                                  adj_prep(c, stored_step(c, W.steps - 1), vn)));
  for (int t = W.steps - 1; t >= 0; --t) {
    dpd::AdjPrep next{};
    if (t > 0) next = adj_prep(c, stored_step(c, t - 1), other);
    const int rc = step_vjp(c, stored_step(c, t), (uint64_t)t, vn, B, t > 0 ? &next : nullptr, dphi);
    if (rc) return rc;
    std::swap(vn, other);
  }
  return DPD_OK;
}

// Recomputed step t of a segment in the backward sweep: from the stored
// state X_t (3 x NF block x), redo the drift/bounce-back and the cell list
// of r_{t+1} in the order of X_t, then the three VJP kernels.  A holds the
// adjoints of X_{t+1} (slot order), B receives those of X_t.
int backward_step(dpd_ctx *c, const float4 *x, uint64_t t, const float4 *A, float4 *B,
                  double *dphi) {
  Window &W = c->win;
  const int64_t NF = c->NF;
  hipStream_t s = c->stream;
  HIP_TRY(c, hipMemcpyAsync(W.wpos, x, 16 * (size_t)NF, hipMemcpyDeviceToDevice, s));
  HIP_TRY(c, dpd::launch_integrate(s, c->ppt, c->boxes, c->itiles, c->n_itiles, W.wpos, W.wpos,
                                   x + NF, x + 2 * NF, c->vt, c->cell_of, c->rank_of, c->count, c->bits,
                                   c->use_mask, c->quad, c->grid_f64, c->status, NF, c->wcstart,
                                   0));
  int rc = scan_scatter_sort(c, s, nullptr, nullptr, false);
  if (rc) return rc;
  const StoredStep st = {const_cast<float4 *>(x), W.wpos,     c->vt,
                         c->idx,                  c->idx_all, c->start_all};
  float4 *vn = W.adj + 7 * NF;
  HIP_TRY(c, dpd::launch_adj_prep(s, c->boxes, NF, 0, A, A + NF, A + 2 * NF, adj_prep(c, st, vn)));
  return step_vjp(c, st, t, vn, B, nullptr, dphi);
}

int backward_impl(dpd_ctx *c, const double *dldp, double *grads, double *dphi) {
  Window &W = c->win;
  const int64_t NF = c->NF;
  hipStream_t s = c->stream;
  const int nb_f = dpd::force_vjp_blocks(c->n_ftiles), nb_g = dpd::adj_prep_blocks(NF);
  int rc = window_partials(c);
  if (rc) return rc;
  // keep the context's state; the sweep reuses the step buffers
  const int cur0 = c->cur;
  const uint64_t k_save = c->k;
  const int64_t steps_save = c->steps;
  const bool recompute = !W.full;
  if (recompute) {
    rc = save_state(c, W.save);
    if (rc) return rc;
    HIP_TRY(c,
            hipMemcpyAsync(W.status_save, c->status, sizeof(StatusBlock), hipMemcpyDeviceToDevice,
                           s));
  }
  const bool timing = c->timing;
  c->timing = false;

  float4 *A = W.adj, *B = W.adj + 3 * NF;
  HIP_TRY(c, dpd::launch_fill_zero(s, A, 48 * (size_t)NF));
  HIP_TRY(c, dpd::launch_fill_zero(s, W.part_f, 24 * (size_t)nb_f));
  HIP_TRY(c, dpd::launch_fill_zero(s, W.part_g, 24 * (size_t)nb_g));
  if (dphi) HIP_TRY(c, dpd::launch_fill_zero(s, dphi, 8 * (size_t)c->NGRID));
  HIP_TRY(c, dpd::launch_loss_weights(s, W.nbins, dldp, W.counts, W.lw));
  // walls and the pad of the sweep's position array
  HIP_TRY(c, hipMemcpyAsync(W.wpos + NF, c->pos[c->cur] + NF, 16 * (size_t)(c->NW + 1),
                            hipMemcpyDeviceToDevice, s));
  if (!recompute) {
    rc = stored_sweep(c, A, B, dphi);
    std::swap(A, B);
  }
  for (int seg = W.nck - 1; seg >= 0 && !rc && recompute; --seg) {
    const int t0 = seg * W.ckpt, t1 = std::min(W.steps, t0 + W.ckpt);
    rc = load_state(c, W.ck + (size_t)seg * 3 * NF);
    if (rc) break;
    c->k = W.k0 + (uint64_t)t0;
    HIP_TRY(c, dpd::launch_set_u64(s, c->dk, c->k));
    // recompute the segment, storing X_t for t0 <= t < t1
    for (int t = t0; t < t1 && !rc; ++t) {
      rc = save_state(c, W.seg + (size_t)(t - t0) * 3 * NF);
      if (!rc) rc = one_step(c);
    }
    for (int t = t1 - 1; t >= t0 && !rc; --t) {
      rc = backward_step(c, W.seg + (size_t)(t - t0) * 3 * NF, (uint64_t)t, A, B, dphi);
      std::swap(A, B);
    }
  }
  if (!rc) {
    // the refreshed starting force f0 = F(r0, v0; k0) + g
    const float4 *x0 = segment_start(c, 0);
    float4 *rt = W.adj + 9 * NF, *vtb = W.adj + 10 * NF, *fbar = W.adj + 8 * NF;
    const Replica &p = c->rep[0];
    HIP_TRY(c, hipMemcpyAsync(W.wpos, x0, 16 * (size_t)NF, hipMemcpyDeviceToDevice, s));
    HIP_TRY(c, dpd::launch_vt_from_v(s, NF, x0 + NF, c->vt));
    HIP_TRY(c, dpd::launch_bin(s, p.G, p.co, NF, W.wpos, c->cell_of, c->rank_of, c->count));
    rc = scan_scatter_sort(c, s, nullptr, nullptr, false);
    if (!rc) {
      HIP_TRY(c, dpd::launch_adj_prep(s, c->boxes, NF, 1, A, A + NF, A + 2 * NF,
                                      adj_prep(c, {}, nullptr)));
      HIP_TRY(c, dpd::launch_force_vjp(s, c->wide ? 0 : c->fblock, c->boxes, c->ftiles, c->n_ftiles, NF,
                                       (int32_t)(NF + c->NW), W.wpos, c->vt, c->idx, c->idx_all,
                                       c->start_all, fbar, nullptr, rt, vtb, W.dk0, 0, W.part_f));
      HIP_TRY(c, dpd::launch_reduce_partials(s, nb_f, W.part_f, nb_g, W.part_g, W.acc));
    }
  }
  // restore the context
  c->timing = timing;
  c->cur = cur0;
  c->k = k_save;
  c->steps = steps_save;
  if (recompute) {
    int r2 = load_state(c, W.save);
    if (!rc) rc = r2;
    HIP_TRY(c,
            hipMemcpyAsync(c->status, W.status_save, sizeof(StatusBlock), hipMemcpyDeviceToDevice,
                           s));
    HIP_TRY(c, dpd::launch_set_u64(s, c->dk, c->k));
  }
  if (rc) return rc;
  double acc[6];
  HIP_TRY(c, hipMemcpyAsync(acc, W.acc, sizeof acc, hipMemcpyDeviceToHost, s));
  HIP_TRY(c, hipStreamSynchronize(s));
  if (grads)
    for (int q = 0; q < 6; ++q) grads[q] = acc[q];
  return latched_error(c);
}

// The recorded window's trajectory again, segment by segment from its
// checkpoints as the backward sweep recomputes it.  State s (0: the
// window's start with its refreshed force, t + 1: after step t) of every
// particle in gid order into pos/vel/frc_log + 3 n s, the event codes of
// step t into ev_log + n t (walls: their positions and velocities, zero
// forces and events).  The context's state, k and counters are left as
// they were.
int trace_impl(dpd_ctx *c, float *pos_log, float *vel_log, float *frc_log, int32_t *ev_log) {
  Window &W = c->win;
  const int64_t NF = c->NF;
  const Replica &p = c->rep[0];
  hipStream_t s = c->stream;
  const int cur0 = c->cur;
  const uint64_t k_save = c->k;
  const int64_t steps_save = c->steps;
  int rc = save_state(c, W.save);
  if (rc) return rc;
  HIP_TRY(c, hipMemcpyAsync(W.status_save, c->status, sizeof(StatusBlock), hipMemcpyDeviceToDevice,
                           s));
  const bool timing = c->timing;
  c->timing = false;
  // state `st` of the trajectory into the logs (events of step st - 1)
  auto put = [&](int st) -> hipError_t {
    float *pl = pos_log ? pos_log + (size_t)3 * p.n * st : nullptr;
    float *vl = vel_log ? vel_log + (size_t)3 * p.n * st : nullptr;
    float *fl = frc_log ? frc_log + (size_t)3 * p.n * st : nullptr;
    int32_t *el = (ev_log && st > 0) ? ev_log + (size_t)p.n * (st - 1) : nullptr;
    return export_box(c, 0, pl, vl, fl, el, nullptr);
  };
  for (int seg = 0; seg < W.nck && !rc; ++seg) {
    const int t0 = seg * W.ckpt, t1 = std::min(W.steps, t0 + W.ckpt);
    rc = load_state(c, segment_start(c, seg));
    if (rc) break;
    c->k = W.k0 + (uint64_t)t0;
    HIP_TRY(c, dpd::launch_set_u64(s, c->dk, c->k));
    if (seg == 0) HIP_TRY(c, put(0));
    for (int t = t0; t < t1 && !rc; ++t) {
      rc = one_step(c);
      if (rc) break;
      HIP_TRY(c, put(t + 1));
    }
  }
  c->timing = timing;
  c->cur = cur0;
  c->k = k_save;
  c->steps = steps_save;
  int r2 = load_state(c, W.save);
  if (!rc) rc = r2;
  HIP_TRY(c, hipMemcpyAsync(c->status, W.status_save, sizeof(StatusBlock), hipMemcpyDeviceToDevice,
                           s));
  HIP_TRY(c, dpd::launch_set_u64(s, c->dk, c->k));
  HIP_TRY(c, hipStreamSynchronize(s));
  if (rc) return rc;
  return latched_error(c);
}

}  // namespace

extern "C" {

const char *dpd_last_error(const dpd_ctx *ctx) {
  return ctx ? ctx->err.c_str() : g_create_error.c_str();
}

const char *dpd_kernel_name(int32_t i) {
  if (i < 0 || i >= DPD_NUM_KERNELS) return "";
  return kKernelNames[i];
}

int dpd_create(const dpd_box *box, const dpd_particles *pp, const dpd_params *prm,
               const dpd_phi_grid *phi, const dpd_allocator *alloc, void *hip_stream,
               dpd_ctx **out) {
  return create_impl(1, box, pp, prm, phi, alloc, hip_stream, out);
}

int dpd_batch_create(int32_t nbox, const dpd_box *boxes, const dpd_particles *particles,
                     const dpd_params *params, const dpd_phi_grid *grids,
                     const dpd_allocator *alloc, void *hip_stream, dpd_ctx **out) {
  return create_impl(nbox, boxes, particles, params, grids, alloc, hip_stream, out);
}

int dpd_replica_count(const dpd_ctx *c) { return c ? c->R : DPD_E_INVAL; }

int dpd_step(dpd_ctx *c, int64_t nsteps) {
  if (!c) return DPD_E_INVAL;
  if (nsteps < 0) return fail(c, DPD_E_INVAL, "negative step count");
  if (c->vt2 && !c->captured) {
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(c->stream, &st) != hipSuccess) (void)hipGetLastError();
    c->captured = st != hipStreamCaptureStatusNone;
  }
  return run_steps(c, nsteps);
}

int dpd_use_graph(dpd_ctx *c, int32_t enable) {
  if (!c) return DPD_E_INVAL;
  if ((enable != 0) != c->use_graph) drop_graphs(c);
  c->use_graph = enable != 0;
  return DPD_OK;
}

int dpd_use_persistent(dpd_ctx *c, int32_t enable) {
  if (!c) return DPD_E_INVAL;
  if (!enable) {
    if (c->persistent) drop_graphs(c);
    c->persistent = false;
    return DPD_OK;
  }
  if (c->nbricks > 0)
    return fail(c, DPD_E_INVAL, "the persistent step needs the per-particle pair kernel");
  if (c->moving) return fail(c, DPD_E_INVAL, "the persistent step does not move walls");
  HIP_TRY(c, hipStreamSynchronize(c->stream));
  c->persistent = true;
  // (one particle per thread, the default of small contexts, takes longer there)
  int rc = c->ppt != 2 ? set_shapes(c, 2, c->fblock) : build_persistent(c);
  if (rc) {
    c->persistent = false;
    return rc;
  }
  drop_graphs(c);
  return DPD_OK;
}

int dpd_replica_forces(dpd_ctx *c, int32_t r, float *f_out) {
  if (!c) return DPD_E_INVAL;
  if (check_replica(c, r)) return DPD_E_INVAL;
  if (!f_out) return fail(c, DPD_E_INVAL, "f_out is NULL");
  HIP_TRY(c, export_box(c, r, nullptr, nullptr, f_out, nullptr, nullptr));
  HIP_TRY(c, hipStreamSynchronize(c->stream));
  return status_error(c, *c->note);
}

int dpd_forces(dpd_ctx *c, float *f_out) { return dpd_replica_forces(c, 0, f_out); }

int dpd_replica_state(dpd_ctx *c, int32_t r, float *pos, float *vel, int32_t *events,
                      int32_t *cell_of) {
  if (!c) return DPD_E_INVAL;
  if (check_replica(c, r)) return DPD_E_INVAL;
  HIP_TRY(c, export_box(c, r, pos, vel, nullptr, events, cell_of));
  HIP_TRY(c, hipStreamSynchronize(c->stream));
  return status_error(c, *c->note);
}

int dpd_get_state(dpd_ctx *c, float *pos, float *vel, int32_t *events, int32_t *cell_of) {
  return dpd_replica_state(c, 0, pos, vel, events, cell_of);
}

int dpd_replica_set_state(dpd_ctx *c, int32_t r, const float *pos, const float *vel,
                          const float *force, uint64_t k, int32_t on_device) {
  if (!c) return DPD_E_INVAL;
  if (check_replica(c, r)) return DPD_E_INVAL;
  if (!pos || !vel || !force) return fail(c, DPD_E_INVAL, "NULL state array");
  const Replica &p = c->rep[r];
  const size_t bytes = 12 * (size_t)p.n;
  const float *dp = pos, *dv = vel, *df = force;
  float *stage = nullptr;
  if (!on_device) {
    stage = (float *)dalloc(c, 3 * std::max<size_t>(bytes, 4));
    if (!stage) return fail(c, DPD_E_NOMEM, "staging allocation failed");
    HIP_TRY(c, hipMemcpyAsync(stage, pos, bytes, hipMemcpyHostToDevice, c->stream));
    HIP_TRY(c, hipMemcpyAsync(stage + 3 * p.n, vel, bytes, hipMemcpyHostToDevice, c->stream));
    HIP_TRY(c, hipMemcpyAsync(stage + 6 * p.n, force, bytes, hipMemcpyHostToDevice, c->stream));
    dp = stage;
    dv = stage + 3 * p.n;
    df = stage + 6 * p.n;
  }
  const int a = c->cur;
  HIP_TRY(c, dpd::launch_import(c->stream, p.nf, c->pos[a] + p.fo, c->vel[a] + p.fo,
                                c->frc[a] + p.fo, dp, dv, df));
  if (p.moving)
    HIP_TRY(c, dpd::launch_import_walls(c->stream, p.nw, c->pos[a] + c->NF + p.wo, dp));
  drop_graphs(c);
  c->gen += 1;
  int rc = resort(c);
  if (rc) return rc;
  c->k = k;
  HIP_TRY(c, hipMemcpyAsync(c->dk, &c->k, 8, hipMemcpyHostToDevice, c->stream));
  Status before;
  rc = read_status(c, before);
  if (rc) return rc;
  const void *g = (const char *)c->grid + (size_t)p.go * (c->grid_f64 ? 8 : 4);
  HIP_TRY(c, dpd::launch_check_phi(c->stream, p.G, g, c->grid_f64, p.nf, c->pos[c->cur] + p.fo,
                                   c->status));
  Status after;
  rc = read_status(c, after);
  if (rc) return rc;
  if (stage) dfree(c, stage);
  if (after.bad_phi != before.bad_phi)
    return fail(c, DPD_E_INVAL, "set_state: fluid particles at phi < 0");
  return DPD_OK;
}

int dpd_set_state(dpd_ctx *c, const float *pos, const float *vel, const float *force,
                  uint64_t k, int32_t on_device) {
  return dpd_replica_set_state(c, 0, pos, vel, force, k, on_device);
}

int dpd_replica_pairs(dpd_ctx *c, int32_t r, uint32_t *pairs, int64_t cap, int64_t *count) {
  if (!c || !count) return DPD_E_INVAL;
  if (check_replica(c, r)) return DPD_E_INVAL;
  if (cap < 0 || (cap > 0 && !pairs)) return fail(c, DPD_E_INVAL, "bad pair buffer");
  const Replica &p = c->rep[r];
  // rebuild the cell list so that it matches the current positions exactly
  HIP_TRY(c, dpd::launch_fill_zero(c->stream, c->pair_counter, 8));
  int rc = bin_all(c, c->stream);
  if (!rc) rc = scan_scatter_sort(c, c->stream);
  if (rc) return rc;
  HIP_TRY(c, dpd::launch_pairs(c->stream, p.G, p.P, p.co, p.fo, p.nf, c->pos[c->cur], c->idx,
                               c->idx_all, c->start_all, pairs, cap, c->pair_counter));
  unsigned long long cnt = 0;
  HIP_TRY(c, hipMemcpyAsync(&cnt, c->pair_counter, 8, hipMemcpyDeviceToHost, c->stream));
  HIP_TRY(c, hipStreamSynchronize(c->stream));
  *count = (int64_t)cnt;
  return latched_error(c);
}

int dpd_neighbor_pairs(dpd_ctx *c, uint32_t *pairs, int64_t cap, int64_t *count) {
  return dpd_replica_pairs(c, 0, pairs, cap, count);
}

int dpd_replica_profile(dpd_ctx *c, int32_t r, int32_t axis, int32_t nbins, double *out) {
  if (!c) return DPD_E_INVAL;
  if (check_replica(c, r)) return DPD_E_INVAL;
  if (axis < 0 || axis > 2 || nbins <= 0 || !out)
    return fail(c, DPD_E_INVAL, "bad profile arguments");
  const Replica &p = c->rep[r];
  HIP_TRY(c, dpd::launch_fill_zero(c->stream, out, 5 * 8 * (size_t)nbins));
  HIP_TRY(c, dpd::launch_profile(c->stream, p.G, p.nf, c->pos[c->cur] + p.fo,
                                 c->vel[c->cur] + p.fo, axis, nbins, out));
  return DPD_OK;
}

int dpd_profile(dpd_ctx *c, int32_t axis, int32_t nbins, double *out) {
  return dpd_replica_profile(c, 0, axis, nbins, out);
}

int dpd_counters(dpd_ctx *c, int64_t *out) {
  if (!c || !out) return DPD_E_INVAL;
  Status st;
  int rc = read_status(c, st);
  if (rc) return rc;
  int64_t flagged = 0;
  for (auto &p : c->rep) flagged += p.flagged_cubes;
  out[0] = c->steps;
  out[1] = (int64_t)c->k;
  out[2] = (int64_t)st.bounce;
  out[3] = (int64_t)st.fallback;
  out[4] = c->NF;
  out[5] = c->NW;
  out[6] = c->NCELL;
  out[7] = flagged;
  out[9] = (int64_t)st.unstable;
  // fluid particles now in flagged cubes (those that interpolate phi)
  HIP_TRY(c, dpd::launch_fill_zero(c->stream, &c->status->lookups, 8));
  for (auto &p : c->rep)
    HIP_TRY(c, dpd::launch_count_flagged(c->stream, p.G, c->grid_f64, p.nf,
                                         c->pos[c->cur] + p.fo, c->bits + p.bo,
                                         &c->status->lookups));
  rc = read_status(c, st);
  if (rc) return rc;
  out[8] = (int64_t)st.lookups;
  return DPD_OK;
}

int dpd_kernel_times(dpd_ctx *c, int32_t enable, double *out_ms, int64_t *out_launches) {
  if (!c) return DPD_E_INVAL;
  HIP_TRY(c, hipStreamSynchronize(c->stream));
  harvest_timings(c);
  if (out_ms)
    for (int i = 0; i < DPD_NUM_KERNELS; ++i) out_ms[i] = c->kernel_ms[i];
  if (out_launches)
    for (int i = 0; i < DPD_NUM_KERNELS; ++i) out_launches[i] = c->kernel_launches[i];
  if (enable && !c->timing) {
    for (int i = 0; i < DPD_NUM_KERNELS; ++i) {
      c->kernel_ms[i] = 0;
      c->kernel_launches[i] = 0;
    }
  }
  c->timing = enable != 0;
  return DPD_OK;
}

int dpd_autotune(dpd_ctx *c, int32_t steps, int32_t *shape_out, double *ms_out) {
  if (!c) return DPD_E_INVAL;
  if (steps < 1) return fail(c, DPD_E_INVAL, "autotune needs at least one step per trial");
  const int P = c->persistent ? 2 : wide_ppt(c);
  const int shapes[4][2] = {{P, 256}, {1, 256}, {P, 128}, {1, 128}};
  const std::string sig = tune_signature(c);
  const char *cache = std::getenv("DPD_TUNE_CACHE");
  int best = -1;
  double times[4] = {-1, -1, -1, -1};
  if (cache) {
    std::ifstream in(cache);
    std::string s;
    int ppt, blk;
    while (in >> s >> ppt >> blk) {
      if (s != sig) continue;
      for (int i = 0; i < 4; ++i)
        if (shapes[i][0] == ppt && shapes[i][1] == blk) best = i;
    }
  }
  if (best < 0) {
    // trials start from a saved copy of the state and leave it unchanged
    HIP_TRY(c, hipStreamSynchronize(c->stream));
    const int cur0 = c->cur;
    const uint64_t k0 = c->k;
    const int64_t steps0 = c->steps;
    const size_t np = 16 * (size_t)(c->NF + c->NW + 1), nv = 16 * (size_t)c->NF;
    const size_t nwv = c->moving ? 16 * (size_t)c->NW : 0;   // moving walls' velocities
    char *save = (char *)dalloc(c, np + 2 * nv + sizeof(StatusBlock) + nwv);
    if (!save) return fail(c, DPD_E_NOMEM, "autotune snapshot allocation failed");
    char *save_wv = save + np + 2 * nv + sizeof(StatusBlock);
    if (nwv)
      HIP_TRY(c, hipMemcpyAsync(save_wv, c->vt + c->NF, nwv, hipMemcpyDeviceToDevice, c->stream));
    HIP_TRY(c, hipMemcpyAsync(save, c->pos[cur0], np, hipMemcpyDeviceToDevice, c->stream));
    HIP_TRY(c, hipMemcpyAsync(save + np, c->vel[cur0], nv, hipMemcpyDeviceToDevice, c->stream));
    HIP_TRY(c, hipMemcpyAsync(save + np + nv, c->frc[cur0], nv, hipMemcpyDeviceToDevice,
                              c->stream));
    HIP_TRY(c, hipMemcpyAsync(save + np + 2 * nv, c->status, sizeof(StatusBlock),
                              hipMemcpyDeviceToDevice, c->stream));
    const bool timing = c->timing;
    c->timing = false;
    int rc = DPD_OK;
    // one trial of shape i from the saved state (which it restores)
    auto run_shape = [&](int i, double &t) -> int {
      rc = set_shapes(c, shapes[i][0], shapes[i][1]);
      float ms = 0.f;
      if (!rc) rc = trial(c, steps, &ms);
      t = ms / steps;
      // restore the saved state
      c->cur = cur0;
      c->k = k0;
      c->steps = steps0;
      HIP_TRY(c, hipMemcpyAsync(c->pos[cur0], save, np, hipMemcpyDeviceToDevice, c->stream));
      HIP_TRY(c, hipMemcpyAsync(c->vel[cur0], save + np, nv, hipMemcpyDeviceToDevice, c->stream));
      HIP_TRY(c, hipMemcpyAsync(c->frc[cur0], save + np + nv, nv, hipMemcpyDeviceToDevice,
                                c->stream));
      HIP_TRY(c, hipMemcpyAsync(c->status, save + np + 2 * nv, sizeof(StatusBlock),
                                hipMemcpyDeviceToDevice, c->stream));
      HIP_TRY(c, hipMemcpyAsync(c->dk, &c->k, 8, hipMemcpyHostToDevice, c->stream));
      if (nwv) {
        // the walls moved during the trial: their saved positions (above) and
        // velocities, and the cell list of that order
        HIP_TRY(c, hipMemcpyAsync(c->vt + c->NF, save_wv, nwv, hipMemcpyDeviceToDevice,
                                  c->stream));
        const int wrc = wall_pass(c, c->stream);
        if (wrc && !rc) rc = wrc;
      }
      return DPD_OK;
    };
    // The first trials of a run are slower (clocks and caches warm up), which
    // favoured whichever shape came last: one untimed round, then two rounds
    // in opposite orders, each shape keeping its faster time.
    const int order[3][4] = {{0, 1, 2, 3}, {0, 1, 2, 3}, {3, 2, 1, 0}};
    // the work-group size is that of k_force alone: not of the pair force with 16 lanes per
    // particle, in bricks, or in the persistent step, whose shapes with 128 are those with 256
    const bool blocks = !c->wide && !c->persistent && c->n_otiles > 0;
    for (int round = 0; round < 3 && !rc; ++round)
      for (int o = 0; o < 4 && !rc; ++o) {
        const int i = order[round][o];
        if (!blocks && shapes[i][1] == 128) continue;
        double t = -1.0;
        const int e = run_shape(i, t);
        if (e) {
          dfree(c, save);
          c->timing = timing;
          return e;
        }
        if (rc || round == 0) continue;
        if (times[i] < 0.0 || t < times[i]) times[i] = t;
      }
    if (!blocks) {
      times[2] = times[0];
      times[3] = times[1];
    }
    for (int i = 0; i < 4 && !rc; ++i)
      if (best < 0 || times[i] < times[best]) best = i;
    HIP_TRY(c, hipStreamSynchronize(c->stream));
    dfree(c, save);
    c->timing = timing;
    if (rc) return rc;
    if (cache) {
      std::ofstream o(cache, std::ios::app);
      o << sig << " " << shapes[best][0] << " " << shapes[best][1] << "\n";
    }
  }
  int rc = set_shapes(c, shapes[best][0], shapes[best][1]);
  if (rc) return rc;
  if (shape_out) {
    shape_out[0] = c->ppt;
    shape_out[1] = c->fblock;
  }
  if (ms_out)
    for (int i = 0; i < 4; ++i) ms_out[i] = times[i];
  return DPD_OK;
}

int dpd_set_params(dpd_ctx *c, int32_t r, const dpd_params *prm) {
  if (!c) return DPD_E_INVAL;
  if (check_replica(c, r)) return DPD_E_INVAL;
  if (!prm) return fail(c, DPD_E_INVAL, "params is NULL");
  const std::string e = check_params(*prm);
  if (!e.empty()) return fail(c, DPD_E_INVAL, e);
  Replica &p = c->rep[r];
  if (prm->rc != p.rc) return fail(c, DPD_E_INVAL, "rc fixes the cell grid and cannot change");
  if ((prm->flags & DPD_FLAG_NO_MASK) != (c->use_mask ? 0 : DPD_FLAG_NO_MASK))
    return fail(c, DPD_E_INVAL, "flags cannot change");
  make_kparams(*prm, p, p.P);
  HIP_TRY(c, hipMemcpyAsync((char *)c->boxes + sizeof(Box) * (size_t)r + offsetof(Box, P), &p.P,
                            sizeof(KParams), hipMemcpyHostToDevice, c->stream));
  // the integrate instance with the moving-wall and specular forms, if any
  // box needs it (a captured step holds the instance it was captured with)
  // and the force instance with the conservative force of Eq. 22-24
  bool reflect = false, sph = false;
  for (const Replica &q : c->rep) {
    reflect = reflect || q.P.reflect != 0;
    sph = sph || q.P.sph != 0;
  }
  if (reflect != c->reflect || sph != c->sph) {
    c->reflect = reflect;
    c->sph = sph;
    drop_graphs(c);
  }
  HIP_TRY(c, hipStreamSynchronize(c->stream));
  c->gen += 1;
  return DPD_OK;
}

int dpd_set_phi(dpd_ctx *c, int32_t r, const void *data, int32_t on_device) {
  if (!c) return DPD_E_INVAL;
  if (check_replica(c, r)) return DPD_E_INVAL;
  if (!data) return fail(c, DPD_E_INVAL, "phi data is NULL");
  const Replica &p = c->rep[r];
  const size_t es = c->grid_f64 ? 8 : 4;
  const int64_t nodes = (int64_t)p.ng[0] * p.ng[1] * p.ng[2];
  void *stage = dalloc(c, es * (size_t)nodes);
  if (!stage) return fail(c, DPD_E_NOMEM, "staging allocation failed");
  HIP_TRY(c, hipMemcpyAsync(stage, data, es * (size_t)nodes,
                            on_device ? hipMemcpyDeviceToDevice : hipMemcpyHostToDevice,
                            c->stream));
  Status before;
  int rc = read_status(c, before);
  if (rc) return rc;
  HIP_TRY(c, dpd::launch_check_grid(c->stream, stage, c->grid_f64, nodes, c->status));
  HIP_TRY(c, dpd::launch_check_phi(c->stream, p.G, stage, c->grid_f64, p.nf,
                                   c->pos[c->cur] + p.fo, c->status));
  Status after;
  rc = read_status(c, after);
  if (rc) return rc;
  if (after.bad_grid != before.bad_grid || after.bad_phi != before.bad_phi) {
    rc = write_status(c, before);
    if (rc) return rc;
    HIP_TRY(c, hipStreamSynchronize(c->stream));
    dfree(c, stage);
    return fail(c, DPD_E_INVAL, after.bad_grid != before.bad_grid
                                    ? "non-finite phi values"
                                    : "fluid particles would sit at phi < 0");
  }
  void *g = (char *)c->grid + (size_t)p.go * es;
  HIP_TRY(c, hipMemcpyAsync(g, stage, es * (size_t)nodes, hipMemcpyDeviceToDevice, c->stream));
  HIP_TRY(c, dpd::launch_cube_mask(c->stream, p.G, g, c->grid_f64, p.nwords, c->bits + p.bo));
  HIP_TRY(c, dpd::launch_build_quad(c->stream, p.G, g, c->grid_f64,
                                    (char *)c->quad + 4 * (size_t)p.go * es));
  std::vector<uint32_t> hb((size_t)p.nwords);
  HIP_TRY(c, hipMemcpyAsync(hb.data(), c->bits + p.bo, 4 * (size_t)p.nwords,
                            hipMemcpyDeviceToHost, c->stream));
  HIP_TRY(c, hipStreamSynchronize(c->stream));
  dfree(c, stage);
  int64_t m = 0;
  for (uint32_t w : hb) m += __builtin_popcount(w);
  c->rep[r].flagged_cubes = m;
  c->gen += 1;
  return DPD_OK;
}

int dpd_window_forward(dpd_ctx *c, int32_t steps, int32_t ckpt, int32_t axis, int32_t nbins,
                       double *profile, int64_t *counts) {
  if (!c) return DPD_E_INVAL;
  if (c->R != 1) return fail(c, DPD_E_STATE, "the adjoint form needs a single-box context");
  if (c->rep[0].P.reflect)
    return fail(c, DPD_E_INVAL, "the adjoint form covers resting walls with bounce-back only");
  if (c->rep[0].P.sph)
    return fail(c, DPD_E_INVAL, "the adjoint form covers the linear conservative force only");
  if (steps < 1 || ckpt < 1 || ckpt > steps)
    return fail(c, DPD_E_INVAL, "need steps >= 1 and 1 <= ckpt <= steps");
  if (axis < 0 || axis > 2 || nbins < 1 || nbins > dpd::kMaxBins)
    return fail(c, DPD_E_INVAL, "bad axis or bin count");
  Window &W = c->win;
  W.valid = false;
  int rc = window_alloc(c, steps, ckpt, nbins);
  if (rc) return rc;
  W.steps = steps;
  W.ckpt = ckpt;
  W.nck = (steps + ckpt - 1) / ckpt;
  W.axis = axis;
  W.nbins = nbins;
  W.scale = (float)((double)nbins / c->rep[0].L[axis]);
  rc = refresh_forces(c);
  if (rc) return rc;
  W.k0 = c->k;
  HIP_TRY(c, dpd::launch_set_u64(c->stream, W.dk0, W.k0));
  HIP_TRY(c, dpd::launch_fill_zero(c->stream, W.sums, 8 * (size_t)nbins));
  HIP_TRY(c, dpd::launch_fill_zero(c->stream, W.counts, 8 * (size_t)nbins));
  if (W.full) {
    rc = stored_window(c);
    if (rc) return rc;
  }
  for (int t = 0; t < steps && !W.full; ++t) {
    if (t % ckpt == 0) {
      rc = save_state(c, W.ck + (size_t)(t / ckpt) * 3 * c->NF);
      if (rc) return rc;
    }
    rc = one_step(c);
    if (rc) return rc;
    HIP_TRY(c, dpd::launch_obs(c->stream, c->NF, 1, 0, c->pos[c->cur], c->vel[c->cur], axis, nbins,
                               W.scale, W.sums, W.counts));
  }
  HIP_TRY(c, dpd::launch_obs_final(c->stream, nbins, W.sums, W.counts, profile, counts));
  rc = latched_error(c);
  if (rc) return rc;
  W.valid = true;
  W.gen = c->gen;
  return DPD_OK;
}

int dpd_backward(dpd_ctx *c, const double *dL_dprofile, double *grads, double *dL_dphi) {
  if (!c) return DPD_E_INVAL;
  if (!c->win.valid) return fail(c, DPD_E_STATE, "backward needs a recorded window");
  if (c->win.gen != c->gen)
    return fail(c, DPD_E_STATE, "parameters, phi or state changed since the window was recorded");
  if (!dL_dprofile) return fail(c, DPD_E_INVAL, "dL_dprofile is NULL");
  return backward_impl(c, dL_dprofile, grads, dL_dphi);
}

int dpd_window_trace(dpd_ctx *c, float *pos_log, float *vel_log, float *frc_log,
                     int32_t *ev_log) {
  if (!c) return DPD_E_INVAL;
  if (!c->win.valid) return fail(c, DPD_E_STATE, "trace needs a recorded window");
  if (c->win.gen != c->gen)
    return fail(c, DPD_E_STATE, "parameters, phi or state changed since the window was recorded");
  return trace_impl(c, pos_log, vel_log, frc_log, ev_log);
}

int dpd_sync(dpd_ctx *c) {
  if (!c) return DPD_E_INVAL;
  return latched_error(c);
}

void dpd_destroy(dpd_ctx *c) {
  if (!c) return;
  (void)hipStreamSynchronize(c->stream);
  release_all(c);
  delete c;
}

int dpd_pair_random(uint64_t seed, uint64_t k, uint32_t replica, const uint32_t *gi,
                    const uint32_t *gj, int64_t n, uint32_t *words, float *xi, void *hip_stream) {
  if (n < 0 || (n > 0 && (!gi || !gj))) return DPD_E_INVAL;
  if (replica >= 65536u) return DPD_E_INVAL;
  hipError_t e = dpd::launch_pair_random((hipStream_t)hip_stream, seed, k, replica, gi, gj, n,
                                         words, xi);
  return e == hipSuccess ? DPD_OK : DPD_E_DEVICE;
}

int dpd_copy_probe(void *dst, const void *src, size_t bytes, void *hip_stream) {
  if (!dst || !src) return DPD_E_INVAL;
  hipError_t e = dpd::launch_copy((hipStream_t)hip_stream, dst, src, bytes);
  return e == hipSuccess ? DPD_OK : DPD_E_DEVICE;
}

int dpd_valu_probe(int32_t kind, int64_t waves, int32_t iters, float *out, void *hip_stream) {
  if (kind < 0 || kind > 3 || waves <= 0 || iters < 0 || !out) return DPD_E_INVAL;
  if (waves * 64 / 256 > INT32_MAX) return DPD_E_INVAL;
  hipError_t e = dpd::launch_valu_probe((hipStream_t)hip_stream, kind, waves, iters, out);
  return e == hipSuccess ? DPD_OK : DPD_E_DEVICE;
}

// ---- Snapshots ----
// Blob: header, then the cell-sorted device arrays of the current state:
// positions of fluid and walls (NF + NW float4, gid bits in w), fluid
// velocities with the last event code (NF float4), fluid forces (NF float4)
// and wall velocities (NW float4).
namespace {
struct SnapHeader {
  char magic[8];
  uint32_t version, R;
  int64_t NF, NW, NCELL, NGRID;
  uint64_t k;
  int64_t steps;
  uint64_t wall_hash;   // FNV-1a of the wall positions (resting walls must match)
  Status status;
};
constexpr char kSnapMagic[8] = {'D', 'P', 'D', 'S', 'N', 'A', 'P', '1'};
constexpr uint32_t kSnapVersion = 1;

uint64_t fnv1a(const void *p, size_t n) {
  const unsigned char *b = (const unsigned char *)p;
  uint64_t h = 1469598103934665603ull;
  for (size_t i = 0; i < n; ++i) h = (h ^ b[i]) * 1099511628211ull;
  return h;
}

size_t snap_bytes(const dpd_ctx *c) {
  return sizeof(SnapHeader) + (size_t)c->R * 4 * sizeof(int64_t) +
         16 * (size_t)(2 * c->NF + 2 * c->NW + c->NF);
}
}  // namespace

int64_t dpd_snapshot_size(const dpd_ctx *c) {
  if (!c) return DPD_E_INVAL;
  return (int64_t)snap_bytes(c);
}

int dpd_snapshot_io(dpd_ctx *c, int32_t dir, void *blob) {
  if (!c) return DPD_E_INVAL;
  if (!blob) return fail(c, DPD_E_INVAL, "snapshot blob is NULL");
  if (dir != 0 && dir != 1) return fail(c, DPD_E_INVAL, "dir must be 0 (save) or 1 (restore)");
  const int a = c->cur;
  char *p = (char *)blob;
  SnapHeader *hd = (SnapHeader *)p;
  int64_t *layout = (int64_t *)(p + sizeof(SnapHeader));
  char *arr = p + sizeof(SnapHeader) + (size_t)c->R * 4 * sizeof(int64_t);
  const size_t bpos = 16 * (size_t)(c->NF + c->NW), bf = 16 * (size_t)c->NF,
               bw = 16 * (size_t)c->NW;
  char *apos = arr, *avel = arr + bpos, *afrc = avel + bf, *awv = afrc + bf;
  // the walls as they are in the context now (for the hash)
  std::vector<float4> walls((size_t)c->NW);
  if (c->NW)
    HIP_TRY(c, hipMemcpyAsync(walls.data(), c->pos[a] + c->NF, bw, hipMemcpyDeviceToHost,
                              c->stream));
  if (dir == 0) {
    Status st;
    int rc = read_status(c, st);   // synchronises
    if (rc) return rc;
    memcpy(hd->magic, kSnapMagic, 8);
    hd->version = kSnapVersion;
    hd->R = (uint32_t)c->R;
    hd->NF = c->NF;
    hd->NW = c->NW;
    hd->NCELL = c->NCELL;
    hd->NGRID = c->NGRID;
    hd->k = c->k;
    hd->steps = c->steps;
    hd->wall_hash = fnv1a(walls.data(), bw);
    hd->status = st;
    for (int r = 0; r < c->R; ++r) {
      layout[4 * r + 0] = c->rep[r].nf;
      layout[4 * r + 1] = c->rep[r].nw;
      layout[4 * r + 2] = c->rep[r].ncell;
      layout[4 * r + 3] = c->rep[r].moving ? 1 : 0;
    }
    HIP_TRY(c, hipMemcpyAsync(apos, c->pos[a], bpos, hipMemcpyDeviceToHost, c->stream));
    HIP_TRY(c, hipMemcpyAsync(avel, c->vel[a], bf, hipMemcpyDeviceToHost, c->stream));
    HIP_TRY(c, hipMemcpyAsync(afrc, c->frc[a], bf, hipMemcpyDeviceToHost, c->stream));
    if (c->NW)
      HIP_TRY(c, hipMemcpyAsync(awv, c->vt + c->NF, bw, hipMemcpyDeviceToHost, c->stream));
    HIP_TRY(c, hipStreamSynchronize(c->stream));
    return DPD_OK;
  }
  // restore: the blob must describe this context's layout
  if (memcmp(hd->magic, kSnapMagic, 8) != 0 || hd->version != kSnapVersion)
    return fail(c, DPD_E_INVAL, "not a snapshot of this library version");
  if (hd->R != (uint32_t)c->R || hd->NF != c->NF || hd->NW != c->NW || hd->NCELL != c->NCELL ||
      hd->NGRID != c->NGRID)
    return fail(c, DPD_E_INVAL, "snapshot of a context with another layout");
  bool any_moving = false;
  for (int r = 0; r < c->R; ++r) {
    const Replica &q = c->rep[r];
    if (layout[4 * r + 0] != q.nf || layout[4 * r + 1] != q.nw ||
        layout[4 * r + 2] != q.ncell || layout[4 * r + 3] != (q.moving ? 1 : 0))
      return fail(c, DPD_E_INVAL, "snapshot of a context with other boxes");
    any_moving = any_moving || q.moving;
  }
  HIP_TRY(c, hipStreamSynchronize(c->stream));
  // resting walls never move: the snapshot's must be this context's
  if (!any_moving && c->NW && fnv1a(walls.data(), bw) != hd->wall_hash)
    return fail(c, DPD_E_INVAL, "snapshot of a context with other wall particles");
  drop_graphs(c);
  HIP_TRY(c, hipMemcpyAsync(c->pos[a], apos, bpos, hipMemcpyHostToDevice, c->stream));
  if (c->NW)
    HIP_TRY(c, hipMemcpyAsync(c->pos[1 - a] + c->NF, apos + bf, bw, hipMemcpyHostToDevice,
                              c->stream));
  HIP_TRY(c, hipMemcpyAsync(c->vel[a], avel, bf, hipMemcpyHostToDevice, c->stream));
  HIP_TRY(c, hipMemcpyAsync(c->frc[a], afrc, bf, hipMemcpyHostToDevice, c->stream));
  if (c->NW)
    HIP_TRY(c, hipMemcpyAsync(c->vt + c->NF, awv, bw, hipMemcpyHostToDevice, c->stream));
  {
    int rc = write_status(c, hd->status);
    if (rc) return rc;
  }
  c->k = hd->k;
  c->steps = hd->steps;
  HIP_TRY(c, hipMemcpyAsync(c->dk, &c->k, 8, hipMemcpyHostToDevice, c->stream));
  // moving walls: their cell runs follow the restored positions (the sort
  // within cells keeps the restored order)
  if (c->moving) {
    int rc = wall_pass(c, c->stream);
    if (rc) return rc;
  }
  c->gen += 1;
  HIP_TRY(c, hipStreamSynchronize(c->stream));
  return latched_error(c);
}

int dpd_phi_relax(void *phi, void *work, int32_t dtype, const int32_t n[3], const double h[3],
                  double eps, double dtau, int32_t iters, double *residual, void *hip_stream) {
  return dpd::phi_relax_run(phi, work, dtype, n, h, eps, dtau, iters, residual, hip_stream);
}

}  // extern "C"

// Argument checks and launches of dpd_phi_relax (also the body of the
// allocation-free variant, which passes its static scratch as `work`).
int dpd::fail_global(int code, const char *msg) { return fail(nullptr, code, msg); }

int dpd::phi_relax_check(const void *phi, int32_t dtype, const int32_t n[3], const double h[3],
                         double eps, double dtau, int32_t iters) {
  if (!phi || !n || !h) return fail(nullptr, DPD_E_INVAL, "NULL argument");
  if (dtype != 4 && dtype != 8) return fail(nullptr, DPD_E_INVAL, "dtype must be 4 or 8");
  for (int a = 0; a < 3; ++a) {
    if (n[a] < 1) return fail(nullptr, DPD_E_INVAL, "grid sizes must be >= 1");
    if (!(std::isfinite(h[a]) && h[a] > 0)) return fail(nullptr, DPD_E_INVAL, "h must be > 0");
  }
  if ((int64_t)n[0] * n[1] > INT32_MAX)
    return fail(nullptr, DPD_E_INVAL, "n[0] n[1] must be < 2^31");
  if (!(std::isfinite(eps) && eps > 0)) return fail(nullptr, DPD_E_INVAL, "eps must be > 0");
  double stiff = 0;
  for (int a = 0; a < 3; ++a) stiff += (eps / h[a]) * (eps / h[a]);
  if (!(std::isfinite(dtau) && dtau > 0 && dtau <= 1.0 / (2.0 * stiff)))
    return fail(nullptr, DPD_E_INVAL, "need 0 < dtau <= 1 / (2 sum (eps/h)^2)");
  if (iters < 0) return fail(nullptr, DPD_E_INVAL, "iters must be >= 0");
  if (dpd::phi_relax_blocks(n) > INT32_MAX) return fail(nullptr, DPD_E_INVAL, "grid too large");
  return DPD_OK;
}

int dpd::phi_relax_run(void *phi, void *work, int32_t dtype, const int32_t n[3],
                       const double h[3], double eps, double dtau, int32_t iters,
                       double *residual, void *hip_stream) {
  const int chk = phi_relax_check(phi, dtype, n, h, eps, dtau, iters);
  if (chk) return chk;
  if (!work) return fail(nullptr, DPD_E_INVAL, "NULL argument");
  hipStream_t s = (hipStream_t)hip_stream;
  const size_t es = (size_t)dtype;
  const size_t nodes = (size_t)n[0] * n[1] * n[2];
  // Eq. 15 in the grid's units: lap' = eps^2 lap, grad' = eps grad
  const double coef[8] = {eps * eps / (h[0] * h[0]), eps * eps / (h[1] * h[1]),
                          eps * eps / (h[2] * h[2]), eps / (2 * h[0]), eps / (2 * h[1]),
                          eps / (2 * h[2]), 1e-4, dtau};
  void *res = (char *)work + nodes * es;
  void *cur = phi, *nxt = work;
  hipError_t e = hipSuccess;
  for (int32_t it = 0; it < iters && e == hipSuccess; ++it) {
    const bool last = residual && it == iters - 1;
    if (last) e = dpd::launch_fill_zero(s, res, es);
    if (e == hipSuccess)
      e = dpd::launch_phi_relax(s, dtype == 8, cur, nxt, n, coef, last ? res : nullptr);
    std::swap(cur, nxt);
  }
  if (e == hipSuccess && cur != phi) e = hipMemcpyAsync(phi, cur, nodes * es, hipMemcpyDeviceToDevice, s);
  if (e != hipSuccess) return hip_fail(nullptr, e, "dpd_phi_relax");
  if (residual) {
    *residual = 0.0;
    if (iters > 0) {
      uint64_t bits = 0;
      e = hipMemcpyAsync(&bits, res, es, hipMemcpyDeviceToHost, s);
      if (e == hipSuccess) e = hipStreamSynchronize(s);
      if (e != hipSuccess) return hip_fail(nullptr, e, "dpd_phi_relax residual");
      if (dtype == 8) {
        double v;
        memcpy(&v, &bits, 8);
        *residual = v;
      } else {
        float v;
        uint32_t b32 = (uint32_t)bits;
        memcpy(&v, &b32, 4);
        *residual = v;
      }
    }
  }
  return DPD_OK;
}
