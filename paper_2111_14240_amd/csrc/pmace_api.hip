// C ABI of libpmace.so (declared in include/pmace.h).
//
// Host responsibilities: argument validation, the workspace layout, the order
// of the set-up (its tables and lists are built on the device), and launching
// iterations (one reconstruction's, or a batch's on several streams).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <new>
#include <utility>
#include <vector>

#include "pmace.h"
#include "pmace_internal.hpp"

using pmace::Recon;

namespace {
std::mutex g_slots_mu;
void* g_slots[pmace::kHostSlots];   // the free ones
size_t g_free_slots = 0, g_made_slots = 0;
}  // namespace

namespace pmace {
void* take_host_slot() {
  {
    std::lock_guard<std::mutex> lk(g_slots_mu);
    if (g_free_slots > 0) return g_slots[--g_free_slots];
    if (g_made_slots == kHostSlots) return nullptr;
    ++g_made_slots;
  }
  void* p = nullptr;
  if (hipHostMalloc(&p, kHostSlot, hipHostMallocPortable | hipHostMallocMapped) == hipSuccess) return p;
  (void)hipGetLastError();
  std::lock_guard<std::mutex> lk(g_slots_mu);
  --g_made_slots;
  return nullptr;
}

void give_host_slot(void* slot) {
  if (!slot) return;
  std::lock_guard<std::mutex> lk(g_slots_mu);
  g_slots[g_free_slots++] = slot;
}
}  // namespace pmace

namespace {

constexpr size_t kAlign = 256;
// Patch sides run by the fused one-workgroup agent; larger ones (160, 192,
// 256) by the three-pass agent.
constexpr int kSmallNp[] = {32, 48, 64, 96, 128};
constexpr int kClasses = 5;
inline size_t align_up(size_t x) { return (x + kAlign - 1) & ~(kAlign - 1); }

bool graphs_enabled() {
  const char* e = std::getenv("PMACE_NO_GRAPH");
  return !(e && e[0] == '1');
}

// A stream-ordered iteration captured once and replayed.
struct Graph {
  hipGraph_t g = nullptr;
  hipGraphExec_t x = nullptr;
  void release() {
    if (x) (void)hipGraphExecDestroy(x);
    if (g) (void)hipGraphDestroy(g);
    x = nullptr;
    g = nullptr;
  }
};

}  // namespace

struct pmace_ctx {
  pmace_params prm;
  hipStream_t stream;
  int device;
  Recon h;                        // host copy of the device descriptor
  Recon* dev;                     // device descriptor (in the workspace)
  int2* ritems;                   // device: (0, b) NRMSE reduction items
  int* fitem;                     // device: {0}
  int ngitems;                    // gather tiles of all chunks
  std::vector<int2> chunk_tiles;  // host: per chunk (first gather tile, count)
  std::vector<int2> chunk_rows;   // host, row-spectrum states: per chunk (first row item, count)
  Graph graph;                    // several iterations back to back (pmace_iterate)
  bool graph_tried;
  long long asked;                // iterations pmace_iterate has been asked for
  bool batched;                   // has been a batch member: its stop flag may be set
  pmace_status sticky;            // first asynchronous failure seen
  unsigned long long resets;      // times the host cleared the stop flag
  // batches holding a copy of this context's descriptor (and its index there):
  // pmace_set_reference updates those copies too
  std::vector<std::pair<pmace_batch*, int>> holders;
};

// Streams beside a batch's own, with the events that fork and join them: three,
// as a process has four hardware queues by default and a fourth would share
// one with the batch's stream (a 4-iteration pass of 16 mixed members with 2
// lanes 1782 us, 3 1712, 4 1826, 8 1819).
constexpr int kLanes = 3;
struct Lanes {
  int device;
  hipStream_t s[kLanes];
  hipEvent_t fork, join[kLanes];
};

struct pmace_batch {
  int n;
  hipStream_t stream;
  std::vector<pmace_ctx*> ctxs;
  Recon* recs;                 // device: member descriptors
  int2* items[kClasses];       // device: agent items per fused patch size (kSmallNp)
  int nitems[kClasses];
  bool zeros[kClasses];        // some member's probe has exact zeros
  int ppw[kClasses];           // patches per workgroup of each class's merged agent launch
  int2* gitems[kClasses];      // device: gather items per class
  int ngitems[kClasses];
  int2* ritems;                // device: (member, block) NRMSE items
  int* fitems;                 // device: member indices
  pmace::PollItem* polled;     // device: what a poll reads of each member
  pmace_stop_rule rule;
  // Members that run as chains of their own (Np > 128, or the split agent):
  // indices, and each member's reduction items and entry of fitems; those of
  // the other members (nsmall of them) come first in both.
  std::vector<int> chains;
  std::vector<int2> rspan;     // (first reduction item, count) per member
  std::vector<int> fpos;       // its entry of fitems, per member
  std::vector<int> run;        // the chains launched by a call (room for all of them)
  int nsmall, nsmall_ritems;
  Lanes* lanes;                // where the chains run side by side, or null
  long long iters;             // iterations launched by this batch
  // Np > 128 members a poll found stopped: their kernel chains are left out
  // of the launches (they would only read the flag and exit), until the host
  // clears the member's flag (pmace_iterate, pmace_set_reference), seen as a
  // change of its reset count from the one recorded here.
  std::vector<char> pruned;
  std::vector<unsigned long long> pruned_at;
};

namespace {

bool np_supported(int np) {
  for (int s : kSmallNp)
    if (np == s) return true;
  return np == 160 || np == 192 || np == 256;
}
bool np_large(int np) { return np > 128; }

bool rowspec_allowed(const pmace_params& p);

// Positions per chunk: Np <= 128 runs all positions in one fused launch;
// Np > 128 stages chunk*Np^2 spectra between its passes.
int chunk_of(const pmace_params& p) {
  int c = p.num_pos;
  // default: the tuned bound for 256-point patches (one for the three-pass
  // agent, one for the row-spectrum agent), scaled so that every patch side
  // stages about the same bytes per chunk
  if (np_large(p.np)) {
    const long long c256 = rowspec_allowed(p) ? PMACE_CHUNK256_RS : PMACE_CHUNK256;
    c = p.chunk > 0 ? p.chunk : (int)(c256 * 256 * 256 / ((long long)p.np * p.np));
  }
  if (c > p.num_pos) c = p.num_pos;
  // the same number of chunks, evened out (no small last chunk)
  const int n = (p.num_pos + c - 1) / c;
  return (p.num_pos + n - 1) / n;
}
int num_chunks(const pmace_params& p) {
  const int c = chunk_of(p);
  return (p.num_pos + c - 1) / c;
}
// Upper bounds of the gather tables (depend on sizes only, not on positions).
size_t max_tiles(const pmace_params& p) {
  return (size_t)num_chunks(p) * ((p.n1 + pmace::GT_R - 1) / pmace::GT_R) *
         ((p.n2 + pmace::GT_C - 1) / pmace::GT_C);
}
size_t max_list(const pmace_params& p) {
  return (size_t)p.num_pos * ((p.np - 1) / pmace::GT_R + 2) * ((p.np - 1) / pmace::GT_C + 2);
}
int num_red(const pmace_params& p) {
  return (int)(((size_t)p.n1 * p.n2 + pmace::RED_PX - 1) / pmace::RED_PX);
}

pmace_status check_params(const pmace_params* p) {
  if (!p) return PMACE_EINVAL;
  if (p->np < 1 || p->num_pos < 1 || p->n1 < p->np || p->n2 < p->np) return PMACE_EINVAL;
  if (!(std::isfinite(p->alpha) && p->alpha >= 0.f)) return PMACE_EINVAL;
  if (!(std::isfinite(p->kappa) && p->kappa >= 0.f)) return PMACE_EINVAL;
  if (!(std::isfinite(p->rho) && p->rho > 0.f && p->rho < 1.f)) return PMACE_EINVAL;
  constexpr uint32_t kAgents = PMACE_STAGED_AGENT | PMACE_SPLIT_AGENT | PMACE_ROWSPEC_AGENT;
  if (p->flags & ~(PMACE_CENTERED_DC | kAgents)) return PMACE_EINVAL;
  const uint32_t ag = p->flags & kAgents;
  if (ag & (ag - 1)) return PMACE_EINVAL;  // at most one agent asked for
  if (p->chunk < 0) return PMACE_EINVAL;
  if (p->method != PMACE_METHOD_PMACE && p->method != PMACE_METHOD_SHARP_PLUS) return PMACE_EINVAL;
  if (p->method == PMACE_METHOD_SHARP_PLUS && !(std::isfinite(p->beta) && p->beta >= 0.f && p->beta <= 1.f))
    return PMACE_EINVAL;
  if ((long long)p->n1 * p->n2 > (1LL << 30)) return PMACE_EINVAL;
  if (!np_supported(p->np)) return PMACE_EUNSUPPORTED;
  if (p->ppw < 0 || (p->ppw > 0 && ((p->ppw & (p->ppw - 1)) != 0 || p->ppw > pmace::max_ppw(p->np))))
    return PMACE_EINVAL;
  return PMACE_OK;
}

// Section offsets inside the workspace (relative to the aligned base).
struct Layout {
  size_t t, ys, pos, d, pc, dinv, gw, omega64, laminv, num, sold, xbar, xhat, stage, tiles, list, status, desc,
      ritems, red, tw, fit, dr, zmask, qtiles, qlist, citems, clist, order, total;
};

// Patch sides whose default agent is the split (coset-block) one: a build
// choice measured by the tuner (bit 0: Np = 128, bit 1: 192, bit 2: 256).
#ifndef PMACE_SPLIT_SIDES
#define PMACE_SPLIT_SIDES 2
#endif
bool split_default(int np) {
  const int bit = np == 128 ? 1 : np == 192 ? 2 : np == 256 ? 4 : 0;
  return (PMACE_SPLIT_SIDES & bit) != 0;
}
// The split agent may run: PMACE with Np in {128, 192, 256} when asked for,
// or by default where the build chose it, unless the other agent is asked
// for.  Whether it does also needs a probe without exact zeros (known at init).
bool split_allowed(const pmace_params& p) {
  if (p.method != PMACE_METHOD_PMACE) return false;
  if (p.np != 128 && p.np != 192 && p.np != 256) return false;
  if (p.flags & PMACE_SPLIT_AGENT) return true;
  if (p.flags & (PMACE_STAGED_AGENT | PMACE_ROWSPEC_AGENT)) return false;
  return split_default(p.np);
}
// Patch sides whose default agent keeps row-spectrum states (bit 0: Np = 160,
// bit 1: 192, bit 2: 256), where the split agent is not the default: a build
// choice measured by the tuner.
#ifndef PMACE_ROWSPEC_SIDES
#define PMACE_ROWSPEC_SIDES 0
#endif
bool rowspec_default(int np) {
  const int bit = np == 160 ? 1 : np == 192 ? 2 : np == 256 ? 4 : 0;
  return (PMACE_ROWSPEC_SIDES & bit) != 0;
}
// SHARP+ on the row-spectrum agent by default where PMACE is (1), or only
// when asked for (0): a build choice measured by the tuner.
#ifndef PMACE_ROWSPEC_SHARP
#define PMACE_ROWSPEC_SHARP 0
#endif
// The row-spectrum agent may run: Np > 128 when asked for, or by default
// where the build chose it and no other agent is asked for or chosen.  PMACE
// also needs a probe without exact zeros (known at init; its d = 0 rule acts
// per pixel); SHARP+ has no such rule.
bool rowspec_allowed(const pmace_params& p) {
  if (!np_large(p.np)) return false;
  if (p.flags & PMACE_ROWSPEC_AGENT) return true;
  if (p.flags & (PMACE_STAGED_AGENT | PMACE_SPLIT_AGENT)) return false;
  if (p.method == PMACE_METHOD_SHARP_PLUS && !PMACE_ROWSPEC_SHARP) return false;
  return !split_allowed(p) && rowspec_default(p.np);
}
// Bounds of its consensus tables (sizes only): every (chunk, object row,
// segment) item, and an entry per patch row and segment it meets (at most two,
// as a segment is at least 256 wide).
int cr_segments(const pmace_params& p) { return (p.n2 + pmace::CR_W - 1) / pmace::CR_W; }
size_t cr_items(const pmace_params& p) { return (size_t)num_chunks(p) * p.n1 * cr_segments(p); }
size_t cr_list(const pmace_params& p) { return (size_t)p.num_pos * p.np * std::min(2, cr_segments(p)); }
// Base tiles of the split consensus: rows [0, qrows), columns [0, qcols), the
// quadrant-0 blocks of all positions lie in [0, n1 - M) x [0, n2 - M).
int split_rows(const pmace_params& p) {
  const int M = p.np / 2;
  return (p.n1 - M + pmace::QT_R - 1) / pmace::QT_R * pmace::QT_R;
}
int split_cols(const pmace_params& p) {
  const int M = p.np / 2;
  return (p.n2 - M + pmace::QT_C - 1) / pmace::QT_C * pmace::QT_C;
}
size_t split_tiles(const pmace_params& p) {
  return (size_t)(split_rows(p) / pmace::QT_R) * (split_cols(p) / pmace::QT_C);
}
size_t split_list(const pmace_params& p) {
  const int M = p.np / 2;
  return (size_t)p.num_pos * ((M - 1) / pmace::QT_R + 2) * ((M - 1) / pmace::QT_C + 2);
}

// Stage buffer: Np > 128 keeps a chunk's spectra between its passes; SHARP+
// keeps its overlap numerators there; PMACE with Np <= 128 needs none.
size_t stage_patches(const pmace_params& p) {
  if (np_large(p.np)) return (size_t)chunk_of(p);
  return p.method == PMACE_METHOD_SHARP_PLUS ? (size_t)chunk_of(p) : 0;
}

// Data-fit partial sums per patch: one, or one per column block for Np > 128.
int fit_bpp(const pmace_params& p) { return np_large(p.np) ? p.np / PMACE_CB : 1; }

// Launch order of one row of the split consensus's base tiles t[first, end),
// left to right, so that each XCD runs side-by-side tiles (as setup_tiles_k
// does for the gather tiles).  Only which workgroup sums which pixel changes;
// every pixel's sum is the same.
void xcd_runs(std::vector<int4>& t, size_t first, size_t end) {
  const size_t q = (end - first) / 8;
  if (q == 0) return;
  const std::vector<int4> row(t.begin() + first, t.begin() + first + 8 * q);
  for (size_t b = 0; b < 8 * q; ++b) t[first + b] = row[(b % 8) * q + b / 8];
}

// Which cells of a grid some of a set of rectangles meets: a difference in
// both directions for each rectangle, summed up by close(), which returns how
// many cells are met.
struct Cover {
  int nr, nc;
  std::vector<int> d;
  Cover(int r, int c) : nr(r), nc(c), d((size_t)(r + 1) * (c + 1), 0) {}
  int& cell(int r, int c) { return d[(size_t)r * (nc + 1) + c]; }
  void add(int r0, int r1, int c0, int c1) {  // inclusive
    ++cell(r0, c0);
    --cell(r0, c1 + 1);
    --cell(r1 + 1, c0);
    ++cell(r1 + 1, c1 + 1);
  }
  int close() {
    int met = 0;
    for (int r = 0; r < nr; ++r) {
      int* row = &cell(r, 0);
      const int* up = r > 0 ? row - (nc + 1) : row;
      int run = 0;
      for (int c = 0; c < nc; ++c) {
        run += row[c];
        row[c] = run + (r > 0 ? up[c] : 0);
        met += row[c] > 0;
      }
    }
    return met;
  }
  bool at(int r, int c) { return cell(r, c) > 0; }
};
// A chunk's empty gather tiles or row items are left out where they are this
// share of all, and so many that the iterations gain the 10 us and more that
// the copy of the host's lists and its wait add to the set-up: an empty tile
// takes an iteration 2 ns (fused with the image update) or 0.5, an empty row
// item 0.4.  For Np > 128 the share alone decides: each XCD has a run of every
// tile row, and an empty column leaves one of them short (1600 positions of
// 160^2 with 2 of 32 columns empty, three-pass: gather 29.1 -> 27.4 us a chunk).
constexpr double kEmptyShare = 1.0 / 16.0;
constexpr int kEmptyTiles = 256, kEmptyItems = 1024;
bool leave_out(int all, int kept, int least) { return all - kept >= std::max(least, (int)(kEmptyShare * all)); }

// The places of a chunk's gather tiles without those that list nothing, row by
// row, ordered over the XCDs as setup_tiles_k orders whole rows.
std::vector<int> tile_slots(Cover& tiles, bool xcd) {
  std::vector<int> slots((size_t)tiles.nr * tiles.nc, -1);
  int first = 0;
  for (int r = 0; r < tiles.nr; ++r) {
    int n = 0, k = 0;
    for (int c = 0; c < tiles.nc; ++c) n += tiles.at(r, c);
    const int q = n / 8;
    for (int c = 0; c < tiles.nc; ++c) {
      if (!tiles.at(r, c)) continue;
      int slot = xcd && k < 8 * q ? (k % q) * 8 + k / q : k;
      if (!xcd && n % 8 == 0) slot = (k + r) % n;
      slots[(size_t)r * tiles.nc + c] = first + slot;
      ++k;
    }
    first += n;
  }
  return slots;
}

Layout layout_of(const pmace_params& p) {
  Layout L;
  const size_t P = (size_t)p.num_pos * p.np * p.np;
  const size_t npx = (size_t)p.n1 * p.n2;
  const size_t np2 = (size_t)p.np * p.np;
  size_t o = 0;
  L.t = o;       o = align_up(o + P * 8);
  L.ys = o;      o = align_up(o + P * 4);
  // status word, stop flag, finish item, track[8] at +32, list cursors at +96;
  // the positions follow, so the set-up reads both back in one copy
  L.status = o;  o += kAlign;
  L.pos = o;     o = align_up(o + (size_t)p.num_pos * 8);
  L.d = o;       o = align_up(o + np2 * 8);
  L.pc = o;      o = align_up(o + np2 * 16);
  L.dinv = o;    o = align_up(o + np2 * 8);
  L.gw = o;      o = align_up(o + np2 * 8);
  L.omega64 = o; o = align_up(o + np2 * 8);
  L.laminv = o;  o = align_up(o + npx * 4);
  L.num = o;     o = align_up(o + npx * 8);
  L.sold = o;    o = align_up(o + npx * 8);
  L.xbar = o;    o = align_up(o + npx * 8);
  L.xhat = o;    o = align_up(o + npx * 8);
  // the staged spectra and the split layout's partial sums never coexist
  const bool sp = split_allowed(p);
  L.stage = o;   o = align_up(o + std::max(stage_patches(p) * np2 * 8, sp ? 4 * npx * 8 : (size_t)0));
  L.tiles = o;   o = align_up(o + max_tiles(p) * 16);
  L.list = o;    o = align_up(o + max_list(p) * 8);
  L.desc = o;    o = align_up(o + sizeof(Recon));
  L.ritems = o;  o = align_up(o + (size_t)num_red(p) * 8);
  L.red = o;     o = align_up(o + (size_t)num_red(p) * 32);
  L.tw = o;      o = align_up(o + 256 * 8);
  L.fit = o;     o = align_up(o + (size_t)p.num_pos * std::max(fit_bpp(p), sp ? 4 : 0) * 8);
  L.dr = o;      o = align_up(o + (sp ? np2 * 8 : 0));
  L.zmask = o;   o = align_up(o + (size_t)p.np * 16 * 8);
  L.qtiles = o;  o = align_up(o + (sp ? split_tiles(p) * 16 : 0));
  L.qlist = o;   o = align_up(o + (sp ? split_list(p) * 4 : 0));
  const bool rs = rowspec_allowed(p);
  L.citems = o;  o = align_up(o + (rs ? cr_items(p) * 16 : 0));
  L.clist = o;   o = align_up(o + (rs ? cr_list(p) * 16 : 0));
  L.order = o;   o = align_up(o + (rs ? (size_t)p.num_pos * 16 : 0));
  L.total = o;
  return L;
}

#define PM_HIP(call)                            \
  do {                                          \
    hipError_t e_ = (call);                     \
    if (e_ != hipSuccess) return PMACE_EDEVICE; \
  } while (0)

pmace_status record(pmace_ctx* c, pmace_status s) {
  if (s != PMACE_OK && c->sticky == PMACE_OK) c->sticky = s;
  return s;
}

// Waits for a figure that the last launch wrote to the slot (none: reads it
// back from the device word it also left it in).
pmace_status read_figure(pmace_ctx* c, pmace::HostSlot& slot, const double* dev, double* out) {
  if (!slot.p && hipMemcpyAsync(out, dev, 8, hipMemcpyDeviceToHost, c->stream) != hipSuccess)
    return record(c, PMACE_EDEVICE);
  if (!slot.wait(c->stream)) return record(c, PMACE_EDEVICE);
  if (slot.p) *out = *static_cast<const double*>(slot.p);
  return PMACE_OK;
}

// A member that runs as its own chain of kernels (three-pass or split agent).
bool own_chain(const pmace_ctx* c) { return np_large(c->prm.np) || c->h.split; }

pmace_status enqueue_iteration(pmace_ctx* c, hipStream_t st) {
  if (c->h.split)
    PM_HIP(pmace::launch_split_iteration(c->h, 0, st));
  else if (np_large(c->prm.np))
    PM_HIP(pmace::launch_large_iteration(c->h, nullptr, c->chunk_tiles.data(), c->chunk_rows.data(), st));
  else
    PM_HIP(pmace::launch_small_iteration(c->prm.np, c->h, c->ngitems, st));
  return PMACE_OK;
}

// Capture `body(stream)` into g (on a private capture stream; the graph is
// then launched on the caller's stream).
template <class F>
pmace_status capture(Graph& g, F body) {
  hipStream_t cs = nullptr;
  PM_HIP(hipStreamCreateWithFlags(&cs, hipStreamNonBlocking));
  pmace_status s = PMACE_OK;
  if (hipStreamBeginCapture(cs, hipStreamCaptureModeThreadLocal) != hipSuccess) {
    s = PMACE_EDEVICE;
  } else {
    s = body(cs);
    hipGraph_t graph = nullptr;
    const hipError_t e = hipStreamEndCapture(cs, &graph);
    if (s == PMACE_OK && (e != hipSuccess || !graph)) s = PMACE_EDEVICE;
    if (s == PMACE_OK && hipGraphInstantiate(&g.x, graph, nullptr, nullptr, 0) != hipSuccess)
      s = PMACE_EDEVICE;
    g.g = graph;
    if (s != PMACE_OK) g.release();
  }
  (void)hipStreamDestroy(cs);
  return s;
}

bool capturing(hipStream_t st) {
  hipStreamCaptureStatus s = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(st, &s) == hipSuccess) return s != hipStreamCaptureStatusNone;
  (void)hipGetLastError();
  return false;
}

__global__ void clear_flag_k(int* flag) { *flag = 0; }

// Reset the stop flag and the NRMSE history of a reconstruction.
__global__ void reset_tracking_k(int* done, double* track) {
  *done = 0;
  track[0] = 0.0;
  track[1] = __builtin_inf();
  track[2] = __builtin_inf();
  track[3] = 0.0;
  track[4] = __builtin_inf();
  track[5] = __builtin_inf();
  track[6] = __builtin_inf();
}

// Copy a member's host descriptor into a batch's descriptor array.
hipError_t batch_recs_update(pmace_batch* b, int i, const Recon& h, hipStream_t st);
// Drop a destroyed member's entry from a batch (the batch can then only be destroyed).
void batch_forget(pmace_batch* b, int i);

}  // namespace

extern "C" {

const char* pmace_status_str(pmace_status s) {
  switch (s) {
    case PMACE_OK: return "ok";
    case PMACE_EINVAL: return "invalid argument";
    case PMACE_EUNSUPPORTED: return "unsupported configuration";
    case PMACE_ENOMEM: return "workspace too small";
    case PMACE_EDEVICE: return "HIP device error";
    case PMACE_ESTATE: return "invalid context state";
    case PMACE_EDIVERGED: return "consensus image not finite";
  }
  return "unknown status";
}

size_t pmace_footprint(const pmace_params* p) {
  if (check_params(p) != PMACE_OK) return 0;
  return layout_of(*p).total + kAlign;  // slack to align an arbitrary base
}

pmace_status pmace_init(const pmace_params* params, const void* probe_d, const int32_t* pos_d,
                        const float* intensity_d, const void* x0_d, void* workspace_d,
                        size_t ws_bytes, void* hip_stream, pmace_ctx** out) try {
  if (!out) return PMACE_EINVAL;
  *out = nullptr;
  pmace_status ps = check_params(params);
  if (ps != PMACE_OK) return ps;
  if (!probe_d || !pos_d || !intensity_d || !workspace_d) return PMACE_EINVAL;
  const pmace_params p = *params;
  if (ws_bytes < pmace_footprint(&p)) return PMACE_ENOMEM;
  hipStream_t st = reinterpret_cast<hipStream_t>(hip_stream);

  const int np = p.np, J = p.num_pos, n1 = p.n1, n2 = p.n2;
  const bool sharp = p.method == PMACE_METHOD_SHARP_PLUS;
  const double inv_np2 = 1.0 / ((double)np * np);

  // What copies in flight may still read or write outlives the context, whose
  // release waits for them.
  const size_t back_bytes = kAlign + (size_t)J * 8;
  pmace::HostSlot slot(back_bytes);
  std::vector<int32_t> pageable;
  std::vector<int4> qtiles;
  std::vector<int> qlist;
  std::vector<std::vector<int>> slots;
  std::vector<std::vector<int2>> rows;
  struct Guard {
    pmace_ctx* c;
    ~Guard() { pmace_destroy(c); }
  } guard{new (std::nothrow) pmace_ctx()};
  pmace_ctx* c = guard.c;
  if (!c) return PMACE_ENOMEM;
  c->prm = p;
  c->stream = st;
  c->sticky = PMACE_OK;
  c->graph_tried = false;
  c->asked = 0;
  c->batched = false;
  c->resets = 0;
  if (hipGetDevice(&c->device) != hipSuccess) return PMACE_EDEVICE;

  const Layout L = layout_of(p);
  char* base = reinterpret_cast<char*>(align_up(reinterpret_cast<size_t>(workspace_d)));
  Recon& h = c->h;
  std::memset(&h, 0, sizeof(Recon));
  h.t = reinterpret_cast<float2*>(base + L.t);
  h.ys = reinterpret_cast<float*>(base + L.ys);
  h.pos = reinterpret_cast<int2*>(base + L.pos);
  h.d = reinterpret_cast<float2*>(base + L.d);
  h.pc = reinterpret_cast<float4*>(base + L.pc);
  h.gw = reinterpret_cast<float2*>(base + L.gw);
  h.omega64 = reinterpret_cast<double*>(base + L.omega64);
  h.dinv = reinterpret_cast<float2*>(base + L.dinv);
  h.laminv = reinterpret_cast<float*>(base + L.laminv);
  h.num = reinterpret_cast<float2*>(base + L.num);
  h.sold = reinterpret_cast<float2*>(base + L.sold);
  h.xbar = reinterpret_cast<float2*>(base + L.xbar);
  h.xhat = reinterpret_cast<float2*>(base + L.xhat);
  h.stage = reinterpret_cast<float2*>(base + L.stage);
  h.tiles = reinterpret_cast<int4*>(base + L.tiles);
  h.tile_list = reinterpret_cast<int2*>(base + L.list);
  h.status = reinterpret_cast<unsigned*>(base + L.status);
  h.done = reinterpret_cast<int*>(base + L.status + 4);
  c->fitem = reinterpret_cast<int*>(base + L.status + 8);
  h.track = reinterpret_cast<double*>(base + L.status + 32);
  h.cursor = reinterpret_cast<int*>(base + L.status + 96);
  h.red = reinterpret_cast<double*>(base + L.red);
  h.twn = reinterpret_cast<float2*>(base + L.tw);
  h.fit = reinterpret_cast<double*>(base + L.fit);
  h.dr = reinterpret_cast<float2*>(base + L.dr);
  h.zmask = reinterpret_cast<unsigned long long*>(base + L.zmask);
  h.part = h.stage;   // the split layout keeps its partial sums where the stage would be
  h.qtiles = reinterpret_cast<int4*>(base + L.qtiles);
  h.qlist = reinterpret_cast<int*>(base + L.qlist);
  h.qrows = split_rows(p);
  h.qcols = split_cols(p);
  h.citems = reinterpret_cast<int4*>(base + L.citems);
  h.clist = reinterpret_cast<int4*>(base + L.clist);
  h.order = reinterpret_cast<int4*>(base + L.order);
  h.xref = nullptr;
  h.mask = nullptr;
  h.n1 = n1;
  h.n2 = n2;
  h.np = np;
  h.np2f = (float)((double)np * np);
  h.J = J;
  h.method = p.method;
  if (sharp) {
    h.beta = p.beta;
    h.a = 0.f;
    h.two_rho = 2.f * p.beta;
    h.rho = 1.f;
    h.ka = (float)((1.0 - 2.0 * (double)p.beta) * inv_np2);
    h.yfac = 1.f;
  } else {
    h.beta = 0.f;
    h.a = p.alpha / (1.f + p.alpha);
    h.two_rho = 2.f * p.rho;
    h.rho = p.rho;
    h.ka = 0.f;
    h.yfac = (float)(1.0 + (double)p.alpha);
    const double rho = p.rho, a = (double)p.alpha / (1.0 + (double)p.alpha);
    h.sb = (float)((1.0 - 2.0 * rho * a) * inv_np2);
    h.s2r = (float)(2.0 * rho * inv_np2);
    h.cx = (float)(2.0 * (1.0 - rho));
    h.co = (float)((1.0 - rho) / rho);
    h.cn = (float)(1.0 / rho);
  }
  const int chunk = chunk_of(p), nch = num_chunks(p);
  h.chunk = chunk;
  h.n_red = num_red(p);
  h.ppw = p.ppw > 0 ? p.ppw : pmace::default_ppw(p.np);
  c->dev = reinterpret_cast<Recon*>(base + L.desc);
  c->ritems = reinterpret_cast<int2*>(base + L.ritems);

  // Everything that reads the caller's arrays; then the status word and the
  // positions (checked on the device) come to the host in one copy.
  pmace::SetupInputs in;
  in.probe = reinterpret_cast<const float2*>(probe_d);
  in.pos = reinterpret_cast<const int2*>(pos_d);
  in.z = intensity_d;
  in.x0 = reinterpret_cast<const float2*>(x0_d);
  in.yscale = (float)((double)np / (sharp ? 1.0 : 1.0 + (double)p.alpha));
  in.centered = (p.flags & PMACE_CENTERED_DC) ? 1 : 0;
  in.kappa = (double)p.kappa;
  in.rho = (double)p.rho;
  in.split_allowed = split_allowed(p) ? 1 : 0;
  in.rowspec_allowed = rowspec_allowed(p) ? 1 : 0;
  if (pmace::launch_setup_inputs(h, in, c->fitem, st) != hipSuccess) return PMACE_EDEVICE;
  int32_t* back = static_cast<int32_t*>(slot.p);
  if (!back) {
    pageable.resize(back_bytes / 4);
    back = pageable.data();
  }
  const auto read_back = [&](size_t bytes) {
    if (slot.p) (void)slot.use<void>();
    return hipMemcpyAsync(back, base + L.status, bytes, hipMemcpyDeviceToHost, st) == hipSuccess && slot.wait(st);
  };
  if (!read_back(back_bytes)) return PMACE_EDEVICE;
  const int32_t* pos = back + kAlign / 4;
  constexpr unsigned kBad = pmace::kStatusBadIntensity | pmace::kStatusBadProbe | pmace::kStatusBadPosition;
  unsigned status = (unsigned)back[0];
  if (status & kBad) return PMACE_EINVAL;
  h.has_zero = !sharp && (status & pmace::kStatusProbeZero) ? 1 : 0;
  h.split = in.split_allowed && !h.has_zero ? 1 : 0;
  h.rowspec = in.rowspec_allowed && !h.has_zero ? 1 : 0;
  h.fit_bpp = h.split ? 4 : fit_bpp(p);
  // Non-temporal stage: for 256-point rows from three quarters of the 256 MB
  // Infinity Cache on (4 iterations: 200 positions, 100 MiB, 501 us without and
  // 520 with it; 300, 150 MiB, 764 and 772; 600, 300 MiB, 1566 and 1499; 900,
  // 450 MiB, 2341 and 2256; a solve of 400, 200 MiB, 1542 and 1519); for the
  // shorter rows of the other sides only from twice the cache on (960 of 192^2,
  // 270 MiB: 1484 and 1532).
  const double stage_mib = (double)std::min(chunk, p.num_pos) * np * np * 8.0 / (1 << 20);
  h.nt_stage = h.rowspec && stage_mib > (np == 256 ? 192.0 : 512.0) ? 1 : 0;

  // Split layout: the base tiles of its consensus, each with the positions
  // whose quadrant-0 block meets it in ascending order.
  const int M = np / 2;
  if (h.split) {
    const int qr = split_rows(p) / pmace::QT_R, qc = split_cols(p) / pmace::QT_C;
    std::vector<std::vector<int>> per_tile((size_t)qr * qc);
    for (int j = 0; j < J; ++j) {
      const int r = pos[2 * j], cc = pos[2 * j + 1];
      for (int tr = r / pmace::QT_R; tr <= (r + M - 1) / pmace::QT_R && tr < qr; ++tr)
        for (int tc = cc / pmace::QT_C; tc <= (cc + M - 1) / pmace::QT_C && tc < qc; ++tc)
          per_tile[(size_t)tr * qc + tc].push_back(j);
    }
    for (int tr = 0; tr < qr; ++tr) {
      const size_t row0 = qtiles.size();
      for (int tc = 0; tc < qc; ++tc) {
        const auto& l = per_tile[(size_t)tr * qc + tc];
        qtiles.push_back(make_int4((int)qlist.size(), (int)l.size(), tr * pmace::QT_R, tc * pmace::QT_C));
        qlist.insert(qlist.end(), l.begin(), l.end());
      }
      xcd_runs(qtiles, row0, qtiles.size());
    }
    if (qtiles.size() > split_tiles(p) || qlist.size() > split_list(p)) return PMACE_EDEVICE;
    h.nqt = (int)qtiles.size();
    if (hipMemcpyAsync(h.qtiles, qtiles.data(), qtiles.size() * 16, hipMemcpyHostToDevice, st) != hipSuccess ||
        (!qlist.empty() &&
         hipMemcpyAsync(h.qlist, qlist.data(), qlist.size() * 4, hipMemcpyHostToDevice, st) != hipSuccess))
      return PMACE_EDEVICE;
  }
  // (where the split agent is allowed the amplitudes and states had to wait)
  if (in.split_allowed && pmace::launch_setup_states(h, in, st) != hipSuccess) return PMACE_EDEVICE;

  // The rows that each chunk covers give its gather tiles (GT_R x GT_C object
  // pixels) and row items; their lists are built on the device.  On a sparse
  // or unordered scan many list no position: those that the iterations walk
  // (the row-spectrum agent its items, the split agent neither) are left out
  // here.  (64 positions of 64^2 on 4096^2: an iteration 152 us with all of
  // them at work, 39 ending at once, 15.6 left out; 200 of 160^2, unordered on
  // 2048 x 4096 in chunks of 25, three-pass: 595, 510, 377.)
  const int tiles_c = (n2 + pmace::GT_C - 1) / pmace::GT_C, nseg = cr_segments(p);
  size_t listed = 0;   // bytes of slots and rows whose copies have not been waited for
  c->chunk_tiles.assign(nch, make_int2(0, 0));
  c->chunk_rows.assign(nch, make_int2(0, 0));
  int tile0 = 0, item0 = 0;
  for (int g = 0; g < nch; ++g) {
    const int ja = g * chunk, jb = std::min(J, ja + chunk);
    int lo = n1, hi = 0;
    for (int j = ja; j < jb; ++j) {
      lo = std::min(lo, pos[2 * j]);
      hi = std::max(hi, pos[2 * j] + np);
    }
    const int tiles_r = (hi - lo + pmace::GT_R - 1) / pmace::GT_R;
    int ntiles = tiles_r * tiles_c, nitems = h.rowspec ? (hi - lo) * nseg : 0;
    pmace::SetupChunk k{ja, jb, lo, tiles_r, tile0, 0, 0, item0, nullptr, nullptr};
    const int least = np_large(np) ? 1 : kEmptyTiles;
    if (!h.rowspec && !h.split && ntiles > least) {
      Cover tiles(tiles_r, tiles_c);
      for (int j = ja; j < jb; ++j) {
        const int r = pos[2 * j] - lo, cc = pos[2 * j + 1];
        tiles.add(r / pmace::GT_R, (r + np - 1) / pmace::GT_R, cc / pmace::GT_C, (cc + np - 1) / pmace::GT_C);
      }
      const int kept = tiles.close();
      if (leave_out(ntiles, kept, least)) {
        slots.push_back(tile_slots(tiles, np_large(np)));
        k.slots = slots.back().data();
        listed += slots.back().size() * sizeof(int);
        ntiles = kept;
      }
    }
    if (nitems > kEmptyItems) {
      Cover segs(hi - lo, nseg);
      for (int j = ja; j < jb; ++j) {
        const int r = pos[2 * j] - lo, cc = pos[2 * j + 1];
        segs.add(r, r + np - 1, cc / pmace::CR_W, (cc + np - 1) / pmace::CR_W);
      }
      const int kept = segs.close();
      if (leave_out(nitems, kept, kEmptyItems)) {
        rows.emplace_back();
        rows.back().reserve(kept);
        for (int sg = 0; sg < nseg; ++sg)
          for (int r = 0; r < hi - lo; ++r)
            if (segs.at(r, sg)) rows.back().push_back(make_int2(lo + r, sg * pmace::CR_W));
        k.rows = rows.back().data();
        listed += rows.back().size() * sizeof(int2);
        nitems = kept;
      }
    }
    k.ntiles = ntiles;
    k.nitems = nitems;
    if (pmace::launch_setup_lists(h, k, tiles_c, nseg, pmace::cr_round(np), st) != hipSuccess)
      return PMACE_EDEVICE;
    if (listed > ((size_t)64 << 20)) {  // (many chunks of a huge object)
      if (!slot.wait(st)) return PMACE_EDEVICE;
      slots.clear();
      rows.clear();
      listed = 0;
    }
    c->chunk_tiles[g] = make_int2(tile0, ntiles);
    c->chunk_rows[g] = make_int2(item0, nitems);
    tile0 += ntiles;
    item0 += nitems;
  }
  c->ngitems = tile0;
  if (pmace::launch_setup_images(h, c->dev, c->ritems, st) != hipSuccess) return PMACE_EDEVICE;
  if (listed > 0 && !slot.wait(st)) return PMACE_EDEVICE;  // the lists above were still being read
  if (in.split_allowed) {  // the inputs were still being read
    if (!read_back(4)) return PMACE_EDEVICE;
    if ((unsigned)back[0] & kBad) return PMACE_EINVAL;
  }
  guard.c = nullptr;
  *out = c;
  return PMACE_OK;
} catch (...) {  // host memory for the lists
  return PMACE_ENOMEM;
}

pmace_status pmace_iterate(pmace_ctx* c, int32_t n_iter) {
  if (!c) return PMACE_ESTATE;
  if (n_iter < 0) return PMACE_EINVAL;
  if (n_iter == 0) return PMACE_OK;
  // a stop flag left by a batch would make its kernels skip this reconstruction
  // (a kernel, not a memset: a caller may be capturing this call)
  if (c->batched) {
    hipLaunchKernelGGL(clear_flag_k, dim3(1), dim3(1), 0, c->stream, c->h.done);
    if (hipGetLastError() != hipSuccess) return record(c, PMACE_EDEVICE);
  }
  ++c->resets;
  // Iterations are launched as they are: the host queues one in 5 to 7 us, the
  // shortest (36 positions of 32^2) runs in 8.  A graph of kGraphIters of them
  // closes the gaps between the smallest kernels (36 positions of 32^2: 8.0 ->
  // 7.2 us per iteration; 64 of 48^2: 11.3 -> 10.7; 144 of 64^2: 14.4 -> 13.9;
  // np 96 and 256: nothing, and a graph of one iteration is slower than its
  // launches at every size), but costs 100 to 300 us to capture, the first of
  // a process 3 to 4 ms, so it is made for Np <= 64 once kCaptureFrom
  // iterations have been asked for.  Under a caller's capture there are
  // launches only.
  constexpr int kGraphIters = 32;
  constexpr long long kCaptureFrom = 256;
  c->asked += n_iter;
  const bool whole = n_iter >= kGraphIters && c->asked >= kCaptureFrom && c->prm.np <= 64 && !capturing(c->stream);
  if (whole && !c->graph_tried && graphs_enabled()) {
    c->graph_tried = true;
    (void)capture(c->graph, [&](hipStream_t cs) {
      for (int i = 0; i < kGraphIters; ++i) {
        const pmace_status s = enqueue_iteration(c, cs);
        if (s != PMACE_OK) return s;
      }
      return PMACE_OK;
    });
  }
  int k = 0;
  if (whole && c->graph.x)
    for (; k + kGraphIters <= n_iter; k += kGraphIters)
      if (hipGraphLaunch(c->graph.x, c->stream) != hipSuccess) return record(c, PMACE_EDEVICE);
  for (; k < n_iter; ++k) {
    const pmace_status s = enqueue_iteration(c, c->stream);
    if (s != PMACE_OK) return record(c, s);
  }
  return PMACE_OK;
}

pmace_status pmace_reconstruct(pmace_ctx* c, void* xhat_d) {
  if (!c) return PMACE_ESTATE;
  if (!xhat_d) return PMACE_EINVAL;
  const size_t bytes = (size_t)c->prm.n1 * c->prm.n2 * 8;
  if (hipMemcpyAsync(xhat_d, c->h.xhat, bytes, hipMemcpyDeviceToDevice, c->stream) != hipSuccess)
    return record(c, PMACE_EDEVICE);
  return PMACE_OK;
}

pmace_status pmace_get_state(pmace_ctx* c, void* v_d) {
  if (!c) return PMACE_ESTATE;
  if (!v_d) return PMACE_EINVAL;
  if (pmace::launch_get_state(c->h, c->dev, reinterpret_cast<float2*>(v_d), c->stream) != hipSuccess)
    return record(c, PMACE_EDEVICE);
  return PMACE_OK;
}

pmace_status pmace_set_state(pmace_ctx* c, const void* v_d) {
  if (!c) return PMACE_ESTATE;
  if (!v_d) return PMACE_EINVAL;
  if (pmace::launch_set_state(c->h, c->dev, reinterpret_cast<const float2*>(v_d),
                              c->chunk_tiles.data(), c->stream) != hipSuccess)
    return record(c, PMACE_EDEVICE);
  return PMACE_OK;
}

pmace_status pmace_set_reference(pmace_ctx* c, const void* xref_d, const uint8_t* mask_d) {
  if (!c) return PMACE_ESTATE;
  c->h.xref = const_cast<float2*>(reinterpret_cast<const float2*>(xref_d));
  c->h.mask = xref_d ? const_cast<unsigned char*>(mask_d) : nullptr;
  if (hipMemcpyAsync(c->dev, &c->h, sizeof(Recon), hipMemcpyHostToDevice, c->stream) != hipSuccess)
    return record(c, PMACE_EDEVICE);
  // a batch reads its members through its own copies of their descriptors
  for (const auto& hb : c->holders)
    if (batch_recs_update(hb.first, hb.second, c->h, c->stream) != hipSuccess) return record(c, PMACE_EDEVICE);
  hipLaunchKernelGGL(reset_tracking_k, dim3(1), dim3(1), 0, c->stream, c->h.done, c->h.track);
  ++c->resets;
  if (hipGetLastError() != hipSuccess || hipStreamSynchronize(c->stream) != hipSuccess)
    return record(c, PMACE_EDEVICE);
  return PMACE_OK;
}

pmace_status pmace_nrmse(pmace_ctx* c, double* out) {
  if (!c) return PMACE_ESTATE;
  if (!out) return PMACE_EINVAL;
  if (!c->h.xref) return PMACE_ESTATE;
  pmace::HostSlot slot;
  if (pmace::launch_nrmse(c->dev, c->ritems, c->h.n_red, c->fitem, 1, 0, 0.f, 0, 0, slot.use<double>(), c->stream) !=
      hipSuccess)
    return record(c, PMACE_EDEVICE);
  return read_figure(c, slot, c->h.track + 1, out);
}

pmace_status pmace_set_stream(pmace_ctx* c, void* hip_stream) {
  if (!c) return PMACE_ESTATE;
  hipStream_t ns = reinterpret_cast<hipStream_t>(hip_stream);
  if (ns == c->stream) return PMACE_OK;
  // everything queued so far completes before the context's next work
  if (hipStreamSynchronize(c->stream) != hipSuccess) return record(c, PMACE_EDEVICE);
  c->stream = ns;
  return PMACE_OK;
}

pmace_status pmace_data_fit(pmace_ctx* c, double* out) {
  if (!c) return PMACE_ESTATE;
  if (!out) return PMACE_EINVAL;
  pmace::HostSlot slot;
  if (pmace::launch_fit_member(c->h, c->dev, 0, c->stream) != hipSuccess ||
      pmace::launch_fit_finish(c->dev, c->fitem, 1, 0, 0.f, 0, 0, slot.use<double>(), c->stream) != hipSuccess)
    return record(c, PMACE_EDEVICE);
  return read_figure(c, slot, c->h.track + 6, out);
}

pmace_status pmace_sync(pmace_ctx* c) {
  if (!c) return PMACE_ESTATE;
  unsigned word = 0;
  pmace::HostSlot slot;
  const unsigned* status = slot.p ? static_cast<unsigned*>(slot.p) : &word;
  if (hipMemcpyAsync(slot.p ? slot.use<void>() : &word, c->h.status, 4, hipMemcpyDeviceToHost, c->stream) !=
          hipSuccess ||
      !slot.wait(c->stream))
    return record(c, PMACE_EDEVICE);
  if (c->sticky != PMACE_OK) return c->sticky;
  if (*status & pmace::kStatusNonFinite) return record(c, PMACE_EDIVERGED);
  return PMACE_OK;
}

int32_t pmace_agent_kind(const pmace_ctx* c) {
  if (!c) return -1;
  if (c->h.split) return PMACE_AGENT_SPLIT;
  if (c->h.rowspec) return PMACE_AGENT_ROWSPEC;
  return np_large(c->prm.np) ? PMACE_AGENT_THREE_PASS : PMACE_AGENT_WHOLE_PATCH;
}

void pmace_destroy(pmace_ctx* c) {
  if (!c) return;
  // a batch still holding this context (a caller error) must not reach it
  for (const auto& hb : c->holders) batch_forget(hb.first, hb.second);
  (void)hipStreamSynchronize(c->stream);
  c->graph.release();
  delete c;
}

pmace_status pmace_fft2(int32_t np, int32_t count, const void* in_d, void* out_d, int32_t inverse,
                        void* hip_stream) {
  if (count < 0 || !in_d || !out_d) return PMACE_EINVAL;
  if (!np_supported(np)) return np < 1 ? PMACE_EINVAL : PMACE_EUNSUPPORTED;
  if (count == 0) return PMACE_OK;
  hipError_t e = pmace::launch_fft2(np, count, reinterpret_cast<const float2*>(in_d),
                                    reinterpret_cast<float2*>(out_d), inverse ? 1 : 0,
                                    reinterpret_cast<hipStream_t>(hip_stream));
  return e == hipSuccess ? PMACE_OK : PMACE_EDEVICE;
}

}  // extern "C"

// ---------------------------------------------------------------------------
// Batches
// ---------------------------------------------------------------------------
namespace {

int class_of(int np) {
  for (int k = 0; k < kClasses; ++k)
    if (np == kSmallNp[k]) return k;
  return -1;
}

struct BatchLayout {
  size_t recs, items[kClasses], gitems[kClasses], ritems, fitems, polled, total;
  int nitems[kClasses], ngitems[kClasses], nritems;
};

BatchLayout batch_layout(pmace_ctx* const* ctxs, int n) {
  BatchLayout L{};
  for (int i = 0; i < n; ++i) {
    const int k = own_chain(ctxs[i]) ? -1 : class_of(ctxs[i]->prm.np);
    if (k >= 0) {
      L.nitems[k] += ctxs[i]->prm.num_pos;
      L.ngitems[k] += ctxs[i]->ngitems;
    }
    L.nritems += ctxs[i]->h.n_red;
  }
  size_t o = 0;
  L.recs = o;    o = align_up(o + (size_t)n * sizeof(Recon));
  for (int k = 0; k < kClasses; ++k) {
    L.items[k] = o;  o = align_up(o + (size_t)L.nitems[k] * 8);
    L.gitems[k] = o; o = align_up(o + (size_t)L.ngitems[k] * 8);
  }
  L.ritems = o;  o = align_up(o + (size_t)L.nritems * 8);
  L.fitems = o;  o = align_up(o + (size_t)n * 4);
  L.polled = o;  o = align_up(o + (size_t)n * sizeof(pmace::PollItem));
  L.total = o;
  return L;
}

pmace_status check_members(pmace_ctx* const* ctxs, int32_t n) {
  if (!ctxs || n < 1) return PMACE_EINVAL;
  for (int i = 0; i < n; ++i) {
    if (!ctxs[i]) return PMACE_ESTATE;
    if (ctxs[i]->prm.method != PMACE_METHOD_PMACE) return PMACE_EUNSUPPORTED;
    if (ctxs[i]->stream != ctxs[0]->stream || ctxs[i]->device != ctxs[0]->device) return PMACE_EINVAL;
    for (int k = 0; k < i; ++k)
      if (ctxs[k] == ctxs[i]) return PMACE_EINVAL;
  }
  return PMACE_OK;
}

// One iteration of the members that share merged launches, and the stop rule's
// evaluation (check) or count.
pmace_status enqueue_small_members(pmace_batch* b, hipStream_t st, bool check) {
  const pmace_stop_rule& r = b->rule;
  for (int k = 0; k < kClasses; ++k)
    if (b->nitems[k] > 0)
      PM_HIP(pmace::launch_small_batch(kSmallNp[k], b->recs, b->items[k], b->nitems[k], b->gitems[k],
                                       b->ngitems[k], b->ppw[k], b->zeros[k], st));
  if (check && r.criterion == PMACE_STOP_NRMSE) {
    PM_HIP(pmace::launch_nrmse(b->recs, b->ritems, b->nsmall_ritems, b->fitems, b->nsmall, 1, r.tol, r.min_iter,
                               r.max_iter, nullptr, st));
  } else if (check) {
    for (int k = 0; k < kClasses; ++k)
      PM_HIP(pmace::launch_fit_batch(kSmallNp[k], b->recs, b->items[k], b->nitems[k], st));
    PM_HIP(pmace::launch_fit_finish(b->recs, b->fitems, b->nsmall, 1, r.tol, r.min_iter, r.max_iter, nullptr, st));
  } else {
    PM_HIP(pmace::launch_tick(b->recs, b->fitems, b->nsmall, r.max_iter, st));
  }
  return PMACE_OK;
}

// The same for member i, a chain of its own.
pmace_status enqueue_chain(pmace_batch* b, int i, hipStream_t st, bool check) {
  const pmace_ctx* c = b->ctxs[i];
  const pmace_stop_rule& r = b->rule;
  const int* fitem = b->fitems + b->fpos[i];
  if (c->h.split)
    PM_HIP(pmace::launch_split_iteration(c->h, 1, st));
  else
    PM_HIP(pmace::launch_large_iteration(c->h, b->recs + i, c->chunk_tiles.data(), c->chunk_rows.data(), st));
  if (check && r.criterion == PMACE_STOP_NRMSE) {
    PM_HIP(pmace::launch_nrmse(b->recs, b->ritems + b->rspan[i].x, b->rspan[i].y, fitem, 1, 1, r.tol, r.min_iter,
                               r.max_iter, nullptr, st));
  } else if (check) {
    PM_HIP(pmace::launch_fit_member(c->h, b->recs + i, 1, st));
    PM_HIP(pmace::launch_fit_finish(b->recs, fitem, 1, 1, r.tol, r.min_iter, r.max_iter, nullptr, st));
  } else {
    PM_HIP(pmace::launch_tick(b->recs, fitem, 1, r.max_iter, st));
  }
  return PMACE_OK;
}

// Sets of lanes: a batch holds one while it lives, and what it gives back is
// kept for the next, so that a server, which rebuilds its batch with every
// admission, neither makes nor destroys streams each time.
constexpr size_t kLaneSetsKept = 8;
std::mutex g_lanes_mu;
Lanes* g_lanes[kLaneSetsKept];
size_t g_nlanes = 0;

void destroy_lanes(Lanes* l) {
  for (int k = 0; k < kLanes; ++k) {
    if (l->s[k]) (void)hipStreamDestroy(l->s[k]);
    if (l->join[k]) (void)hipEventDestroy(l->join[k]);
  }
  if (l->fork) (void)hipEventDestroy(l->fork);
  delete l;
}

Lanes* take_lanes() {
  int device = 0;
  if (hipGetDevice(&device) != hipSuccess) return nullptr;
  {
    std::lock_guard<std::mutex> lk(g_lanes_mu);
    for (size_t i = g_nlanes; i-- > 0;)
      if (g_lanes[i]->device == device) {
        Lanes* l = g_lanes[i];
        g_lanes[i] = g_lanes[--g_nlanes];
        return l;
      }
  }
  Lanes* l = new (std::nothrow) Lanes();
  if (!l) return nullptr;
  l->device = device;
  bool ok = hipEventCreateWithFlags(&l->fork, hipEventDisableTiming) == hipSuccess;
  for (int k = 0; k < kLanes && ok; ++k)
    ok = hipStreamCreateWithFlags(&l->s[k], hipStreamNonBlocking) == hipSuccess &&
         hipEventCreateWithFlags(&l->join[k], hipEventDisableTiming) == hipSuccess;
  if (ok) return l;
  destroy_lanes(l);
  return nullptr;
}

// (Their work has been joined to a stream that has been waited for.)
void give_lanes(Lanes* l) {
  if (!l) return;
  {
    std::lock_guard<std::mutex> lk(g_lanes_mu);
    if (g_nlanes < kLaneSetsKept) {
      g_lanes[g_nlanes++] = l;
      return;
    }
  }
  destroy_lanes(l);
}

hipError_t batch_recs_update(pmace_batch* b, int i, const Recon& h, hipStream_t st) {
  return hipMemcpyAsync(b->recs + i, &h, sizeof(Recon), hipMemcpyHostToDevice, st);
}

void batch_forget(pmace_batch* b, int i) { b->ctxs[i] = nullptr; }

void batch_release(pmace_batch* b) {
  for (pmace_ctx* c : b->ctxs) {
    if (!c) continue;
    auto& hs = c->holders;
    for (size_t k = 0; k < hs.size();)
      if (hs[k].first == b) hs.erase(hs.begin() + (long)k);
      else ++k;
  }
  give_lanes(b->lanes);
  delete b;
}

}  // namespace

extern "C" {

size_t pmace_batch_footprint(pmace_ctx* const* ctxs, int32_t n) {
  if (check_members(ctxs, n) != PMACE_OK) return 0;
  return batch_layout(ctxs, n).total + kAlign;
}

pmace_status pmace_batch_create(pmace_ctx* const* ctxs, int32_t n, const pmace_stop_rule* rule,
                                void* workspace_d, size_t ws_bytes, pmace_batch** out) try {
  if (!out) return PMACE_EINVAL;
  *out = nullptr;
  pmace_status ps = check_members(ctxs, n);
  if (ps != PMACE_OK) return ps;
  if (!rule || !workspace_d || rule->min_iter < 0 || rule->max_iter < 1 || !std::isfinite(rule->tol) ||
      (rule->criterion != PMACE_STOP_NRMSE && rule->criterion != PMACE_STOP_DATA_FIT) ||
      rule->check_every < 0)
    return PMACE_EINVAL;
  const BatchLayout L = batch_layout(ctxs, n);
  if (ws_bytes < L.total + kAlign) return PMACE_ENOMEM;
  std::vector<Recon> recs(n);
  std::vector<int2> items[kClasses], gitems[kClasses], ritems;
  std::vector<int> fitems;
  struct Guard {
    pmace_batch* b;
    ~Guard() { pmace_batch_destroy(b); }
  } guard{new (std::nothrow) pmace_batch()};
  pmace_batch* b = guard.b;
  if (!b) return PMACE_ENOMEM;
  b->n = n;
  b->stream = ctxs[0]->stream;
  b->ctxs.assign(ctxs, ctxs + n);
  b->rule = *rule;
  if (b->rule.check_every == 0) b->rule.check_every = 1;
  b->iters = 0;
  b->pruned.assign(n, 0);
  b->pruned_at.assign(n, 0);
  char* base = reinterpret_cast<char*>(align_up(reinterpret_cast<size_t>(workspace_d)));
  b->recs = reinterpret_cast<Recon*>(base + L.recs);
  for (int i = 0; i < n; ++i) {
    recs[i] = ctxs[i]->h;
    if (own_chain(ctxs[i])) b->chains.push_back(i);
    else fitems.push_back(i);
  }
  b->nsmall = (int)fitems.size();
  fitems.insert(fitems.end(), b->chains.begin(), b->chains.end());
  b->run.reserve(b->chains.size());
  b->rspan.resize(n);
  b->fpos.resize(n);
  for (int f = 0; f < n; ++f) {
    const int i = fitems[f];
    pmace_ctx* c = ctxs[i];
    b->fpos[i] = f;
    b->rspan[i] = make_int2((int)ritems.size(), c->h.n_red);
    for (int r = 0; r < c->h.n_red; ++r) ritems.push_back(make_int2(i, r));
    if (f >= b->nsmall) continue;
    b->nsmall_ritems = (int)ritems.size();
    const int k = class_of(c->prm.np);
    b->zeros[k] = b->zeros[k] || c->h.has_zero;
    if (items[k].empty()) b->ppw[k] = c->h.ppw;   // the class takes its first member's choice
    for (int j = 0; j < c->prm.num_pos; ++j) items[k].push_back(make_int2(i, j));
    for (int t = 0; t < c->ngitems; ++t) gitems[k].push_back(make_int2(i, t));
  }
  if (b->chains.size() + (b->nsmall > 0) > 1) {   // else there is nothing to run side by side
    b->lanes = take_lanes();
    if (!b->lanes) return PMACE_EDEVICE;
  }
  hipStream_t st = b->stream;
  bool ok = hipMemcpyAsync(b->recs, recs.data(), (size_t)n * sizeof(Recon), hipMemcpyHostToDevice,
                           st) == hipSuccess;
  for (int k = 0; k < kClasses; ++k) {
    b->items[k] = reinterpret_cast<int2*>(base + L.items[k]);
    b->gitems[k] = reinterpret_cast<int2*>(base + L.gitems[k]);
    b->nitems[k] = (int)items[k].size();
    b->ngitems[k] = (int)gitems[k].size();
    if (!items[k].empty())
      ok = ok && hipMemcpyAsync(b->items[k], items[k].data(), items[k].size() * 8,
                                hipMemcpyHostToDevice, st) == hipSuccess;
    if (!gitems[k].empty())
      ok = ok && hipMemcpyAsync(b->gitems[k], gitems[k].data(), gitems[k].size() * 8,
                                hipMemcpyHostToDevice, st) == hipSuccess;
  }
  b->ritems = reinterpret_cast<int2*>(base + L.ritems);
  b->fitems = reinterpret_cast<int*>(base + L.fitems);
  b->polled = reinterpret_cast<pmace::PollItem*>(base + L.polled);
  ok = ok && hipMemcpyAsync(b->ritems, ritems.data(), ritems.size() * 8, hipMemcpyHostToDevice, st) ==
                 hipSuccess;
  ok = ok && hipMemcpyAsync(b->fitems, fitems.data(), (size_t)n * 4, hipMemcpyHostToDevice, st) ==
                 hipSuccess;
  ok = ok && hipStreamSynchronize(st) == hipSuccess;
  if (!ok) return PMACE_EDEVICE;
  for (int i = 0; i < n; ++i) {
    ctxs[i]->holders.emplace_back(b, i);
    ctxs[i]->batched = true;
  }
  guard.b = nullptr;
  *out = b;
  return PMACE_OK;
} catch (...) {  // host memory for the tables
  return PMACE_ENOMEM;
}

pmace_status pmace_batch_step(pmace_batch* b, int32_t n_iter) {
  if (!b) return PMACE_ESTATE;
  if (n_iter < 0) return PMACE_EINVAL;
  // a pruned member whose stop flag the host has cleared runs again
  std::vector<int>& run = b->run;
  run.clear();
  for (int i : b->chains) {
    if (b->pruned[i] && b->ctxs[i]->resets != b->pruned_at[i]) b->pruned[i] = 0;
    if (!b->pruned[i]) run.push_back(i);
  }
  // The chains depend on nothing but themselves, so they fork from the batch's
  // stream once a call and join it at the end, and each evaluates its own stop
  // rule (16 mixed members, a 4-iteration pass: 1712 us; with a fork and a join
  // around every iteration, for one evaluation over all members, 1955, and
  // those captured as a graph 1755).
  int nl = 0;
  if (b->lanes && n_iter > 0 && run.size() + (b->nsmall > 0) > 1) nl = (int)std::min(run.size(), (size_t)kLanes);
  if (nl) PM_HIP(hipEventRecord(b->lanes->fork, b->stream));
  for (int l = 0; l < nl; ++l) PM_HIP(hipStreamWaitEvent(b->lanes->s[l], b->lanes->fork, 0));
  pmace_status s = PMACE_OK;
  for (int k = 0; k < n_iter && s == PMACE_OK; ++k) {
    // the stop rule is evaluated after every check_every-th iteration of the batch
    const bool check = ++b->iters % b->rule.check_every == 0;
    if (b->nsmall > 0) s = enqueue_small_members(b, b->stream, check);
    for (size_t q = 0; q < run.size() && s == PMACE_OK; ++q)
      s = enqueue_chain(b, run[q], nl ? b->lanes->s[q % nl] : b->stream, check);
  }
  for (int l = 0; l < nl; ++l)   // also after a failed launch: what was queued is waited for with the stream
    if (hipEventRecord(b->lanes->join[l], b->lanes->s[l]) != hipSuccess ||
        hipStreamWaitEvent(b->stream, b->lanes->join[l], 0) != hipSuccess)
      s = PMACE_EDEVICE;
  return s;
}

pmace_status pmace_batch_poll_fit(pmace_batch* b, int32_t* done, double* nrmse, int32_t* iters,
                                  double* data_fit) try {
  if (!b) return PMACE_ESTATE;
  const size_t bytes = (size_t)b->n * sizeof(pmace::PollItem);
  pmace::HostSlot slot(bytes);  // (the kernel writes there itself)
  std::vector<pmace::PollItem> pageable(slot.p ? 0 : b->n);
  const pmace::PollItem* got = slot.p ? static_cast<pmace::PollItem*>(slot.p) : pageable.data();
  if (pmace::launch_poll(b->recs, b->n, slot.p ? slot.use<pmace::PollItem>() : b->polled, b->stream) != hipSuccess ||
      (!slot.p && hipMemcpyAsync(pageable.data(), b->polled, bytes, hipMemcpyDeviceToHost, b->stream) != hipSuccess) ||
      !slot.wait(b->stream))
    return PMACE_EDEVICE;
  for (int i : b->chains)
    if (got[i].done && !b->pruned[i]) {
      b->pruned[i] = 1;
      b->pruned_at[i] = b->ctxs[i]->resets;
    }
  for (int i = 0; i < b->n; ++i) {
    if (done) done[i] = got[i].done;
    if (nrmse) nrmse[i] = got[i].nrmse;
    if (iters) iters[i] = (int32_t)got[i].iters;
    if (data_fit) data_fit[i] = got[i].fit;
  }
  return PMACE_OK;
} catch (...) {  // host memory to read back through
  return PMACE_ENOMEM;
}

pmace_status pmace_batch_poll(pmace_batch* b, int32_t* done, double* nrmse, int32_t* iters) {
  return pmace_batch_poll_fit(b, done, nrmse, iters, nullptr);
}

void pmace_batch_destroy(pmace_batch* b) {
  if (!b) return;
  (void)hipStreamSynchronize(b->stream);
  batch_release(b);
}

}  // extern "C"
