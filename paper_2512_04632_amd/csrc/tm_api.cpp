// C ABI of the Turbo-Muon orthogonalizer: argument validation, per-stream
// workspace cache and the launch plan of Algorithms 1 and 2 (one launch per
// phase over the tiles of every matrix of the call).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <array>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <utility>
#include <vector>

#include "tm_internal.h"
#include "turbomuon.h"

namespace tmk {
hipError_t launch_elementwise_bf16(int kind, const Phase& P, hipStream_t st);
hipError_t launch_fast_bf16(int kind, int cfg, int step, const Phase& P, hipStream_t st);
hipError_t launch_split_f32(int kind, int cfg, int step, const Phase& P, hipStream_t st);
hipError_t launch_phase_f32(int kind, int cfg, const Phase& P, hipStream_t st);
hipError_t launch_opt(int apply, const OptPhase& P, hipStream_t st);
hipError_t launch_small_bf16(int F, int big, const SmallPhase& P, hipStream_t st);
}  // namespace tmk

namespace {

using tmk::Entry;
using tmk::Phase;

thread_local std::string g_last_error;

tm_status fail(tm_status s, const std::string& msg) {
  g_last_error = msg;
  return s;
}

// Default coefficients: the constant quintic triple, used for every iteration.
constexpr float kA = 3.4445f, kB = -4.7750f, kC = 2.0315f;

struct Workspace {
  void* ptr = nullptr;
  size_t bytes = 0;
  size_t refused = SIZE_MAX;   // smallest reserve (beyond what a call needed) that could not be had
  bool captured = false;       // used by a call under graph capture: never freed or reused in place
};

std::mutex g_mu;
using WsCache = std::map<std::pair<int, hipStream_t>, Workspace>;
WsCache g_ws;     // iteration workspace of every call
WsCache g_ws_u;   // bf16 update matrices of the optimizer step
std::map<int, bool> g_dev_ok;
// Workspaces replaced while a captured graph may still hold their address:
// freed only by tm_release_workspaces.
std::vector<void*> g_retired;

// Timing hooks: event pairs bracketing each launch while enabled.
struct TimedLaunch {
  int kind;
  hipEvent_t start, stop;
};
bool g_timing = false;
std::vector<TimedLaunch> g_timed;
static_assert(int(tmk::kNumKinds) == TM_NUM_PHASES, "one timing phase per kernel kind");
static_assert(tmk::kMaxIters == TM_MAX_ITERS, "the fused kernel's descriptor holds every iteration");
double g_time_ms[TM_NUM_PHASES];
int64_t g_time_n[TM_NUM_PHASES];

void collect_timing() {
  for (TimedLaunch& t : g_timed) {
    float ms = 0.f;
    if (hipEventSynchronize(t.stop) == hipSuccess &&
        hipEventElapsedTime(&ms, t.start, t.stop) == hipSuccess) {
      g_time_ms[t.kind] += double(ms);
      g_time_n[t.kind] += 1;
    }
    (void)hipEventDestroy(t.start);
    (void)hipEventDestroy(t.stop);
  }
  g_timed.clear();
}

// One matrix (or a batch of equal matrices stored back to back).
struct Item {
  char* x;
  uint32_t k, N;
  uint32_t kp, Np;     // padded workspace dims (set by the planner)
  uint32_t count;
  bool tall;
  bool direct;         // bf16: iteration 1 reads the caller's matrix in place of a padded copy
  bool pair;           // bf16: two iterations per update (see pair_rule)
};

// Which items a launch covers (the others get no blocks).
enum Cover { kCoverAll, kCoverTall, kCoverCopied };

tm_status check_device(int* dev) {
  hipError_t e = hipGetDevice(dev);
  if (e != hipSuccess) return fail(TM_ERR_HIP, std::string("hipGetDevice: ") + hipGetErrorString(e));
  auto it = g_dev_ok.find(*dev);
  if (it == g_dev_ok.end()) {
    hipDeviceProp_t prop;
    e = hipGetDeviceProperties(&prop, *dev);
    if (e != hipSuccess)
      return fail(TM_ERR_HIP, std::string("hipGetDeviceProperties: ") + hipGetErrorString(e));
    const bool ok = std::strncmp(prop.gcnArchName, "gfx950", 6) == 0;
    it = g_dev_ok.emplace(*dev, ok).first;
  }
  if (!it->second) return fail(TM_ERR_UNSUPPORTED, "device is not gfx950 (MI355X)");
  return TM_OK;
}

bool capturing(hipStream_t st) {
  hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(st, &cap) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  return cap != hipStreamCaptureStatusNone;
}

// Device memory of a workspace.  TM_TEST_FAIL_ALLOC in the environment refuses
// requests of at least that many bytes.
void* device_alloc(size_t bytes) {
  const char* refuse = std::getenv("TM_TEST_FAIL_ALLOC");
  if (refuse != nullptr && bytes >= std::strtoull(refuse, nullptr, 10)) return nullptr;
  void* p = nullptr;
  if (hipMalloc(&p, bytes) == hipSuccess) return p;
  (void)hipGetLastError();
  return nullptr;
}

// Grow the (device, stream) buffer of a cache to at least `bytes`, to `reserve`
// (>= bytes) where that can be had.  Under graph capture (`cap`) nothing may be
// allocated, freed or synchronised: the buffer must already be large enough, and
// it is then marked as captured.  A captured buffer keeps its address for the
// graphs that hold it: a later, larger eager call on that stream handle gets a new
// buffer, and the old one is retired (freed by tm_release_workspaces only).
tm_status get_workspace(int dev, hipStream_t st, size_t bytes, size_t reserve, bool cap, char** out,
                        WsCache& cache = g_ws) {
  Workspace& w = cache[{dev, st}];
  if (cap) {
    if (w.bytes < bytes)
      return fail(TM_ERR_UNSUPPORTED,
                  "the stream's workspace holds " + std::to_string(w.bytes) + " bytes, the call "
                  "needs " + std::to_string(bytes) + "; nothing can be allocated under graph "
                  "capture (make one call of this size on the stream before capturing)");
    w.captured = true;
    *out = static_cast<char*>(w.ptr);
    return TM_OK;
  }
  if (w.bytes < bytes || (w.bytes < reserve && reserve < w.refused)) {
    if (w.ptr && w.captured) {
      g_retired.push_back(w.ptr);
    } else if (w.ptr) {
      hipError_t e = hipStreamSynchronize(st);
      if (e != hipSuccess)
        return fail(TM_ERR_HIP, std::string("hipStreamSynchronize: ") + hipGetErrorString(e));
      (void)hipFree(w.ptr);
    }
    w = Workspace{nullptr, 0, w.refused, false};
    size_t size = std::max(bytes, reserve);
    void* p = device_alloc(size);
    if (p == nullptr && size > bytes) {
      w.refused = std::min(w.refused, size);   // not tried again by every later call
      size = bytes;
      p = device_alloc(size);
    }
    if (p == nullptr)
      return fail(TM_ERR_NO_MEMORY, "workspace allocation of " + std::to_string(bytes) + " bytes failed");
    w.ptr = p;
    w.bytes = size;
  }
  *out = static_cast<char*>(w.ptr);
  return TM_OK;
}

uint64_t item_ws(const Item& it, int esz) {
  return tmk::ws_layout(it.kp, it.Np, uint32_t(esz)).total * it.count;
}

// Generic (fp32) path: pick per phase the largest tile whose launch still
// spans one wave of the chip's 256 compute units; otherwise the smallest.
int choose_cfg_f32(int kind, const std::vector<Item>& items) {
  for (int cfg = 0; cfg < tmk::kNumCfg - 1; ++cfg) {
    uint64_t tiles = 0;
    for (const Item& it : items)
      tiles += uint64_t(it.count) * tmk::blocks_per_matrix(kind, cfg, it.k, it.N, it.kp, it.Np);
    if (tiles >= 256) return cfg;
  }
  return tmk::kNumCfg - 1;
}

// The items with neighbours of one shape joined: what the choice of a tile
// looks at (a group of many matrices has few shapes; choosing for each launch
// over every matrix would cost as much host time as a small call takes).
std::vector<Item> shapes_of(const std::vector<Item>& items) {
  std::vector<Item> out;
  for (const Item& it : items) {
    if (!out.empty() && out.back().k == it.k && out.back().N == it.N && out.back().kp == it.kp &&
        out.back().Np == it.Np && out.back().pair == it.pair)
      out.back().count += it.count;
    else
      out.push_back(it);
  }
  return out;
}

// Time of one matrix-core launch over `items` with a tile size, in
// microseconds without the launch itself.  A tile costs its compute unit f + r K
// (K elements of its contraction), and a launch at least its longest tile alone
// on a unit, f1 + r1 K.  Measured:
//   256: 13 + 0.024 K (one block per unit: pipeline fill and the 128 KB epilogue
//        are not hidden), in waves of one block per unit; a last wave of at most
//        a quarter runs as 128 sub-tiles;
//   128: 4 (with the mirrored store; update 1.5) + 0.0098 K;
//   64:  1.1 + 0.0039 K;   32 (one wave): 0.5 + 0.0021 K.
// Up to three blocks of 128 or 64 share a unit, so at most 768 start at once and
// the unit with the most of them ends last (528 of 64 with K = 2048: 23 us, 496
// with 1984: 16 us); more are dealt out as units come free.
double launch_us(int kind, int cfg, const std::vector<Item>& items, int segments) {
  struct Cost {
    double f, r, f1, r1;
  };
  const bool upd = kind == tmk::kKindUpdate;
  const Cost cost[4] = {{13.0, 0.024, 13.0, 0.024},
                        {upd ? 1.5 : 4.0, 0.0098, 4.5, 0.0095},
                        {1.1, 0.0039, 3.2, 0.0029},
                        {0.5, 0.0021, 0.5, 0.0021}};
  const Cost& c = cost[cfg];
  double sum = 0.0, tiles = 0.0, one = 0.0;
  for (const Item& it : items) {
    const double K = double(segments) * (kind == tmk::kKindGram ? it.Np : it.kp);
    const double n = double(it.count) * tmk::blocks_per_matrix(kind, cfg, it.k, it.N, it.kp, it.Np);
    tiles += n;
    sum += n * (c.f + c.r * K);
    one = std::max(one, c.f1 + c.r1 * K);
  }
  if (tiles == 0.0) return 0.0;
  const double waves = std::floor(tiles / 256.0), frac = tiles / 256.0 - waves;
  if (cfg == 0 && tiles > 256.0)
    return sum / tiles * (waves + (frac == 0.0 ? 0.0 : (frac <= 0.25 ? 0.45 : 1.0)));
  if ((cfg == 1 || cfg == 2) && tiles <= 768.0)
    return std::max(one, c.f + (sum / tiles - c.f) * std::ceil(tiles / 256.0));
  return std::max(one, sum / 256.0);
}

// The tile of a launch: cfg first .. last from the largest tile down, a
// smaller one where the model puts it 5% ahead (within that, the larger tile
// measured better: the 64 conv matrices' Gram on 240 tiles of 128 against 800
// of 64 by 9%).
int choose_cfg(int kind, int first, int last, const std::vector<Item>& items, int segments) {
  int best = first;
  double us = launch_us(kind, first, items, segments);
  for (int cfg = first + 1; cfg <= last; ++cfg) {
    const double t = launch_us(kind, cfg, items, segments);
    if (t < 0.95 * us) {
      best = cfg;
      us = t;
    }
  }
  return best;
}

// The layout tile of a call (its update's; the Gram and the k x k products may
// run smaller ones): of the tiles whose zero padding adds at most 30% to the
// call's products (the smallest always), the one with the shortest iteration, a
// smaller one again from 5% on.  One 4096 x 4096 fp32 matrix: 256 tiles of 256,
// one wave, instead of 1024 of 128; 1984 x 3072: 64 tiles without padding, whose
// Gram and polynomial save more than the update loses.
int choose_tile_cfg(const std::vector<Item>& items, int segments) {
  double real = 0.0;
  for (const Item& it : items)
    real += double(it.count) * (3.0 * it.k * double(it.k) * it.N + double(it.k) * it.k * it.k);
  int best = -1;
  double us = 0.0;
  for (int cfg = 0; cfg < tmk::kNumCfg; ++cfg) {
    std::vector<Item> laid = items;
    double padded = 0.0;
    bool pairs = false;
    for (Item& it : laid) {
      tmk::tiled_dims(it.k, it.N, uint32_t(tmk::cfg_tile(cfg)), &it.kp, &it.Np);
      padded += double(it.count) * (3.0 * it.kp * double(it.kp) * it.Np + double(it.kp) * it.kp * it.kp);
      pairs = pairs || it.pair;
    }
    if (padded > 1.3 * real && cfg < tmk::kNumCfg - 1) continue;
    auto shortest = [&](int kind) {
      return launch_us(kind, choose_cfg(kind, cfg, tmk::kCfgSym32, laid, segments), laid, segments);
    };
    const double t = launch_us(tmk::kKindUpdate, cfg, laid, segments) +
                     shortest(tmk::kKindGram) + (pairs ? 5.0 : 1.0) * shortest(tmk::kKindPoly);
    if (best < 0 || t < 0.95 * us) {
      best = cfg;
      us = t;
    }
  }
  return best;
}

// Workspace of `shapes` laid out on a tile size.
uint64_t laid_bytes(std::vector<Item> shapes, int cfg, int esz) {
  uint64_t total = 0;
  for (Item& it : shapes) {
    tmk::tiled_dims(it.k, it.N, uint32_t(tmk::cfg_tile(cfg)), &it.kp, &it.Np);
    total += item_ws(it, esz);
  }
  return total;
}

// The layout tile with the static scratch of the allocation-free entry point
// in view: a bf16 call that fits it on a smaller tile takes that one, whichever
// entry point it came by (equal launches, and tm_workspace_bytes tells which
// calls fit).  4 x 1044 x 1480: 67.8 MB on 128 tiles, 61.9 on 64; near the
// limit the padding of the larger tile is what decides.  With `limit`, the bytes
// that a call under capture or short of memory can have, also no tile beyond it
// but the smallest (whose layout is the smallest too): the results do not depend
// on the tile.
int layout_cfg(const std::vector<Item>& shapes, int esz, uint64_t limit = UINT64_MAX) {
  constexpr uint64_t kScratch = TM_NOALLOC_SCRATCH_BYTES;
  int cfg = choose_tile_cfg(shapes, esz == 4 ? 3 : 1);
  if (esz == 2 && laid_bytes(shapes, tmk::kNumCfg - 1, esz) <= kScratch) limit = std::min(limit, kScratch);
  while (limit != UINT64_MAX && cfg < tmk::kNumCfg - 1 && laid_bytes(shapes, cfg, esz) > limit) ++cfg;
  return cfg;
}

struct Plan {
  const std::vector<Item>* items;
  std::vector<uint64_t> ws_off;   // byte offset of each item's workspace region
  char* ws;
  int esz;
  hipStream_t st;
  int tcfg = 0;                   // bf16: the call's layout tile
  std::vector<Item> shapes;       // shapes_of(items)
  // tiles chosen so far for launches over all items of a class, by kind, smallest
  // tile and classes (-1: none yet)
  mutable int tile_of[tmk::kNumKinds][2][3];
  bool split = false;             // fp32 on fp16 planes (tm_fast.hip's kernels)
  float raise = 0.f;              // size that small rows are worked on at (raise_to); 0: their own
  bool timed = true;              // the timing hooks may bracket this call's launches
};

// Compute units of the MI355X: the blocks of one full wave of the large tiles.
constexpr int kWave = 256;

// K step (elements per ring stage) of a 4-wave or one-wave launch.  A 96 KB
// ring (128 for the 64 tile, 64 for the 128 tile) holds one block per compute
// unit, so it serves launches of at most one wave of blocks; a 48 KB ring (64
// for the 64 tile, 128 for the 32 tile) holds three, which suits a launch of
// any size; else 32 (the 128 tile's many-block launches).  Every K of the
// launch must be a multiple of the step (the Gram contracts over Np, the k x k
// products and the update over kp): halved until it is.  (The 256 tile's ring
// is fixed.)  A symmetric fp32 launch of different lengths also takes the 96 KB
// ring up to two waves of 64 tiles: its long tiles (three K segments) then have a
// unit each and the short ones fill the units as they come free (468 tiles 526 -> 519
// us a call, 486 tiles 687 -> 630; but 752 tiles 843 -> 867, and bf16's
// short ones gain nothing, 494 -> 552).
int k_step(int kind, int cfg, const Phase& P, bool split) {
  const int T = tmk::cfg_tile(cfg);
  int step = 32;
  if (T == 128 && P.total <= kWave) step = 64;
  if (T == 64) step = P.total <= kWave ? 128 : 64;
  if (T == 32) step = 128;
  if (split && T == 64 && (P.flags & tmk::kBySlice) && kind != tmk::kKindUpdate && P.total <= 2 * kWave)
    step = 128;
  for (int e = 0; e < P.nent; ++e) {
    const uint32_t K = kind == tmk::kKindGram ? P.e[e].Np : P.e[e].kp;
    while (P.e[e].tiles_per != 0u && K % uint32_t(step) != 0u) step /= 2;
  }
  return step;
}

// Enqueue one kernel launch of a prepared phase descriptor (timed when the
// timing hooks are on).
tm_status fire(const Plan& pl, int kind, int cfg, const Phase& P) {
  TimedLaunch tl{kind, nullptr, nullptr};
  if (g_timing && pl.timed && P.total > 0) {
    if (hipEventCreate(&tl.start) != hipSuccess || hipEventCreate(&tl.stop) != hipSuccess)
      return fail(TM_ERR_HIP, "hipEventCreate failed");
    (void)hipEventRecord(tl.start, pl.st);
  }
  if (P.total <= 0) return TM_OK;
  hipError_t e;
  const bool elementwise =
      kind == tmk::kKindFrob || kind == tmk::kKindAolVector || kind == tmk::kKindApplyScale;
  if (pl.esz == 4 && (!pl.split || elementwise))
    e = tmk::launch_phase_f32(kind, cfg, P, pl.st);
  else if (elementwise)
    e = tmk::launch_elementwise_bf16(kind, P, pl.st);
  else if (pl.split)
    e = tmk::launch_split_f32(kind, cfg, k_step(kind, cfg, P, pl.split), P, pl.st);
  else
    e = tmk::launch_fast_bf16(kind, cfg, k_step(kind, cfg, P, pl.split), P, pl.st);
  if (tl.start) {
    (void)hipEventRecord(tl.stop, pl.st);
    g_timed.push_back(tl);
  }
  if (e != hipSuccess) return fail(TM_ERR_HIP, std::string("kernel launch: ") + hipGetErrorString(e));
  return TM_OK;
}

// Entries of one launch: a run of positions [first, first + n) of the launch
// order.  A run of n > 1 single matrices of one shape whose workspace regions
// follow each other is one kPtrTab entry; otherwise n = 1.
struct Run {
  size_t first, n;
};

// Per-class operands of a bf16 matrix-core step (see Phase).
struct Step {
  int kind;
  uint32_t flags;
  int src = 0, dst = 0;       // Gram, update: Y slots
  int fac = tmk::kBufB;       // update: its k x k factor
  // k x k product: out = alpha L R + beta M + gamma I
  int l = 0, r = 0, m = tmk::kNoBuf, out = 0, mode = tmk::kSymBf16;
  float alpha = 0.f, beta = 0.f, gamma = 0.f;
};

// Tile of one matrix-core launch over `items` (those it covers), at most the
// layout tile.  A call that runs its update over all of its matrices in one
// launch keeps the layout tile.
int choose_step_cfg(int kind, uint32_t flags, int tcfg, const std::vector<Item>& items, bool whole,
                    int segments) {
  if (kind == tmk::kKindUpdate)
    return whole ? tcfg : choose_cfg(kind, tcfg, tmk::kNumCfg - 1, items, segments);
  // the first Gram's row partials and fp32 tiles want at least 64 columns
  const bool small = kind == tmk::kKindPoly || (flags & (tmk::kRowSum | tmk::kA32)) == 0u;
  return choose_cfg(kind, tcfg, small ? tmk::kCfgSym32 : tmk::kNumCfg - 1, items, segments);
}

// One launch of `kind` per chunk of at most kMaxEntries entries and kMaxPtrs
// table pointers.  bf16 matrix-core steps pass their operands by class in
// `steps` (a null one leaves its class out).
tm_status launch(const Plan& pl, int kind, int cfg, int src, int dst, float a, float b, float c,
                 uint32_t flags, int aux, Cover cover = kCoverAll,
                 const Step* const* steps = nullptr) {
  const std::vector<Item>& items = *pl.items;
  auto covered = [&](const Item& it) {
    return !((cover == kCoverTall && !it.tall) || (cover == kCoverCopied && it.direct) ||
             (steps != nullptr && steps[it.pair ? 1 : 0] == nullptr));
  };
  // Long tiles start first: update launches take their largest products first,
  // the symmetric ones their longest contractions (a group whose long ones come
  // last otherwise ends on them: 30 x 256 x 256 beside 3 x 1500 x 1700, 493 -> 422
  // us a call).  Every entry carries its own workspace offset.
  std::vector<size_t> idx(items.size());
  for (size_t i = 0; i < idx.size(); ++i) idx[i] = i;
  auto length = [&](const Item& it) {
    return kind == tmk::kKindUpdate ? double(it.k) * it.k * it.N * it.count
                                    : double(kind == tmk::kKindGram ? it.Np : it.kp);
  };
  if (kind == tmk::kKindUpdate || steps != nullptr)
    std::stable_sort(idx.begin(), idx.end(),
                     [&](size_t x, size_t y) { return length(items[x]) > length(items[y]); });
  auto joins = [&](size_t prev, size_t next) {
    const Item& u = items[idx[prev]];
    const Item& v = items[idx[next]];
    return u.count == 1u && v.count == 1u && u.k == v.k && u.N == v.N && u.kp == v.kp &&
           u.Np == v.Np && u.tall == v.tall && u.direct == v.direct && u.pair == v.pair &&
           pl.ws_off[idx[next]] == pl.ws_off[idx[prev]] + item_ws(u, pl.esz);
  };
  std::vector<std::vector<Run>> chunks(1);
  int ptrs = 0;
  for (size_t i = 0; i < idx.size(); ++i) {
    std::vector<Run>& ch = chunks.back();
    if (!ch.empty() && joins(i - 1, i)) {
      Run& r = ch.back();
      const int need = r.n == 1 ? 2 : 1;   // a run of two starts the table
      if (ptrs + need <= tmk::kMaxPtrs) {
        ++r.n;
        ptrs += need;
        continue;
      }
    }
    if (ch.size() == size_t(tmk::kMaxEntries) || ptrs == tmk::kMaxPtrs) {
      chunks.emplace_back();
      ptrs = 0;
    }
    chunks.back().push_back(Run{i, 1});
  }
  for (const std::vector<Run>& ch : chunks) {
    Phase P;
    std::memset(&P, 0, sizeof(P));
    // each launch picks its tile for the matrices that it covers (the last
    // launch of a split call may have much fewer); a product's arithmetic does
    // not depend on the tile size
    int ccfg = cfg;
    if (steps != nullptr && chunks.size() == 1) {
      const int classes = (steps[0] ? 1 : 0) + (steps[1] ? 2 : 0);
      const bool small = (flags & (tmk::kRowSum | tmk::kA32)) == 0u;
      int& memo = pl.tile_of[kind][small ? 1 : 0][classes - 1];
      if (memo < 0) {
        std::vector<Item> part;
        for (const Item& it : pl.shapes)
          if (covered(it)) part.push_back(it);
        memo = part.empty() ? 0
                            : choose_step_cfg(kind, flags, pl.tcfg, part,
                                              part.size() == pl.shapes.size(), pl.split ? 3 : 1);
      }
      ccfg = memo;
    } else if (steps != nullptr) {
      std::vector<Item> part;
      for (const Run& r : ch)
        for (size_t i = r.first; i < r.first + r.n; ++i)
          if (covered(items[idx[i]])) part.push_back(items[idx[i]]);
      if (part.empty()) continue;
      ccfg = choose_step_cfg(kind, flags, pl.tcfg, shapes_of(part), part.size() == items.size(),
                             pl.split ? 3 : 1);
    }
    uint64_t start = 0;
    uint32_t xp = 0;
    const size_t n = ch.size();
    for (size_t e = 0; e < n; ++e) {
      const Run& r = ch[e];
      const Item& it = items[idx[r.first]];
      Entry& E = P.e[e];
      E.x = it.x;
      E.ws256 = uint32_t(pl.ws_off[idx[r.first]] >> 8);
      E.k = it.k;
      E.N = it.N;
      E.kp = it.kp;
      E.Np = it.Np;
      E.count = r.n > 1 ? uint32_t(r.n) : it.count;
      E.flags = (it.tall ? tmk::kTall : 0u) | (it.direct ? tmk::kDirect : 0u) |
                (it.pair ? tmk::kPair : 0u);
      if (steps != nullptr && steps[it.pair ? 1 : 0] != nullptr) {
        const Step& st = *steps[it.pair ? 1 : 0];
        E.flags |= tmk::pack_ops(st.src, st.dst, st.fac, st.l, st.r, st.m, st.out);
      }
      if (r.n > 1) {
        E.flags |= tmk::kPtrTab;
        E.xbase = xp;
        for (size_t i = r.first; i < r.first + r.n; ++i) P.xp[xp++] = items[idx[i]].x;
      }
      E.tile_start = uint32_t(start);
      E.tiles_per = !covered(it) ? 0u : tmk::blocks_per_matrix(kind, ccfg, it.k, it.N, it.kp, it.Np);
      start += uint64_t(E.tiles_per) * E.count;
    }
    if (start >= (uint64_t(1) << 31))
      return fail(TM_ERR_UNSUPPORTED, "too many tiles in one launch");
    P.nent = int32_t(n);
    P.total = int32_t(start);
    P.ws = pl.ws;
    P.src = src;
    P.dst = dst;
    P.a = a;
    P.b = b;
    P.c = c;
    if (steps != nullptr) {
      const Step none{kind, 0u};
      const Step& s0 = steps[0] ? *steps[0] : none;
      const Step& s1 = steps[1] ? *steps[1] : none;
      P.a = s0.gamma, P.b = s0.beta, P.c = s0.alpha;
      P.a2 = s1.gamma, P.b2 = s1.beta, P.c2 = s1.alpha;
      P.symmode = !steps[0] ? s1.mode : (!steps[1] ? s0.mode : int(tmk::kSymMixed));
    }
    P.flags = flags;
    P.aux = aux;
    P.tail_base = 0;
    tm_status s = TM_OK;
    // A matrix-core launch whose entries' tiles differ in K gives every XCD an
    // eighth of each entry (kBySlice): the default chunks of consecutive tiles
    // would give the first XCDs all the long tiles of the launch.  us a call,
    // chunks and slices, both sorted: 30 x 256 x 256 with 3 x 1500 x 1700 422 and
    // 409; 6 x 2048 x 2048 with 4 of 2048 x 5632 2725 and 2640; dealing whole
    // matrices out in turn, where that is even, measures the same as slices (72
    // GPT-2 and 64 conv matrices within 0.4%).  Slices also stand in for the
    // sub-tiles of a nearly empty last wave (below), where the shortest tiles are
    // last: 20 x 1024 x 1024 with 8 x 1024 x 1800 902 us, with sub-tiles 952.
    // Not for entries of one matrix, which eight L2s then share, nor for many entries,
    // which every block walks through: groups of single matrices, slices and chunks, 40
    // shapes 480 and 361 us, 24 of them 294 and 244, 12 675 and 640, 6 404 and 388, 3 88
    // and 85; of three each, 40 shapes 1055 and 938, 24 680 and 632, 16 1342 and 1517 (360
    // and 337 with lengths closer together), 8 819 and 879.
    const bool mc = kind == tmk::kKindGram || kind == tmk::kKindPoly || kind == tmk::kKindUpdate;
    bool by_slice = false;
    if ((pl.esz == 2 || pl.split) && mc) {
      uint32_t kmin = UINT32_MAX, kmax = 0;
      uint64_t ents = 0, mats = 0;
      for (int e = 0; e < P.nent; ++e) {
        if (P.e[e].tiles_per == 0u) continue;
        const uint32_t K = kind == tmk::kKindGram ? P.e[e].Np : P.e[e].kp;
        kmin = std::min(kmin, K);
        kmax = std::max(kmax, K);
        ++ents;
        mats += P.e[e].count;
      }
      by_slice = kmin < kmax && ents <= 16 && 2 * mats >= 3 * ents;
      if (by_slice) P.flags |= tmk::kBySlice;
    }
    // bf16 matrix-core phases on 256 x 256 tiles whose last wave would be at
    // most a quarter full: the full waves run as usual, the remaining tiles as
    // 2 x 2 sub-tiles of 128 x 128 in a second launch that fits in one wave
    // (same per-element arithmetic, four times the blocks for the idle units);
    // an update tail of at most 16 tiles as 4 x 4 sub-tiles of 64 x 64.
    const int tail = (!by_slice && (pl.esz == 2 || pl.split) && ccfg == 0 && mc && P.total > kWave && P.total % kWave <= kWave / 4)
                         ? P.total % kWave
                         : 0;
    if (tail > 0) {
      P.total -= tail;
      s = fire(pl, kind, ccfg, P);
      Phase Q = P;
      const bool f4 = kind == tmk::kKindUpdate && 16 * tail <= kWave;
      Q.flags |= tmk::kTail | (f4 ? tmk::kTail4 : 0u);
      Q.tail_base = P.total;
      Q.total = (f4 ? 16 : 4) * tail;
      if (s == TM_OK) s = fire(pl, kind, f4 ? 2 : 1, Q);
    } else {
      s = fire(pl, kind, ccfg, P);
    }
    if (s != TM_OK) return s;
  }
  return TM_OK;
}

// Fused small-matrix path (bf16): a matrix qualifies when k <= 128 and its
// padded Y, A and B fit in the 160 KB of LDS of one compute unit.
constexpr uint64_t kSmallLdsBig = 160u * 1024u;   // variants of the fused kernel
constexpr uint64_t kSmallLdsLow = 64u * 1024u;    // (two workgroups per compute unit)

bool small_eligible(const Item& it) {
  return it.k <= uint32_t(tmk::kSmallMaxK) && tmk::small_lds_bytes(it.k, it.N) <= kSmallLdsBig;
}

// Every iteration of every matrix in one launch per (kp / 32, LDS variant)
// class and per chunk of kMaxSmallEntries entries / kMaxSmallPtrs pointers;
// consecutive single matrices of one shape share a kPtrTab entry.  No
// workspace: everything between reading X and writing the result stays in LDS.
tm_status plan_small(const Plan& pl, int iters, const float* coeffs, int precond) {
  const std::vector<Item>& items = *pl.items;
  for (int F = 1; F <= tmk::kSmallMaxK / 32; ++F)
    for (int big = 0; big < 2; ++big) {
      std::vector<size_t> idx;
      for (size_t i = 0; i < items.size(); ++i) {
        const Item& it = items[i];
        if (int(tmk::small_kp(it.k) / 32u) == F &&
            int(tmk::small_lds_bytes(it.k, it.N) > kSmallLdsLow) == big)
          idx.push_back(i);
      }
      size_t i = 0;
      while (i < idx.size()) {
        tmk::SmallPhase P;
        std::memset(&P, 0, sizeof(P));
        P.iters = iters;
        P.precond = precond;
        for (int t = 0; t < iters; ++t) {
          P.coef[t][0] = coeffs ? coeffs[3 * t] : kA;
          P.coef[t][1] = coeffs ? coeffs[3 * t + 1] : kB;
          P.coef[t][2] = coeffs ? coeffs[3 * t + 2] : kC;
        }
        uint64_t start = 0;
        int xp = 0;
        while (i < idx.size() && P.nent < tmk::kMaxSmallEntries) {
          const Item& it = items[idx[i]];
          Entry& E = P.e[P.nent];
          E.x = it.x;
          E.k = it.k;
          E.N = it.N;
          E.kp = tmk::small_kp(it.k);
          E.Np = tmk::small_np(it.N);
          E.flags = it.tall ? tmk::kTall : 0u;
          E.tile_start = uint32_t(start);
          E.tiles_per = 1u;
          E.count = it.count;
          ++i;
          // a run of single matrices of this shape: one pointer-table entry
          auto same = [&](size_t j) {
            const Item& v = items[idx[j]];
            return it.count == 1u && v.count == 1u && v.k == it.k && v.N == it.N && v.tall == it.tall;
          };
          if (i < idx.size() && same(i) && xp + 2 <= tmk::kMaxSmallPtrs) {
            E.flags |= tmk::kPtrTab;
            E.xbase = uint32_t(xp);
            P.xp[xp++] = it.x;
            while (i < idx.size() && same(i) && xp < tmk::kMaxSmallPtrs) P.xp[xp++] = items[idx[i++]].x;
            E.count = uint32_t(xp) - E.xbase;
          }
          start += E.count;
          ++P.nent;
          if (start >= (uint64_t(1) << 31))
            return fail(TM_ERR_UNSUPPORTED, "too many matrices in one launch");
        }
        P.total = int32_t(start);
        TimedLaunch tl{int(tmk::kKindSmall), nullptr, nullptr};
        if (g_timing && pl.timed) {
          if (hipEventCreate(&tl.start) != hipSuccess || hipEventCreate(&tl.stop) != hipSuccess)
            return fail(TM_ERR_HIP, "hipEventCreate failed");
          (void)hipEventRecord(tl.start, pl.st);
        }
        const hipError_t e = tmk::launch_small_bf16(F, big, P, pl.st);
        if (tl.start) {
          (void)hipEventRecord(tl.stop, pl.st);
          g_timed.push_back(tl);
        }
        if (e != hipSuccess) return fail(TM_ERR_HIP, std::string("kernel launch: ") + hipGetErrorString(e));
      }
    }
  return TM_OK;
}

uint32_t raise_flag(const Plan& pl) { return pl.raise > 0.f ? tmk::kRaise : 0u; }

// Scale vector s from the first Gram (its flags carry the row partials):
// AOL (Algorithm 2, second line) s_i = 1 / sqrt(row sum of |A0|); Schatten-4
// the uniform ||A0||_F^(-1/2), summed from the squares' row partials.  `part`
// is the column granularity of the row partials.
tm_status gram_scale(const Plan& pl, int precond, int part) {
  if (precond == TM_PRECOND_AOL)
    return launch(pl, tmk::kKindAolVector, 0, 0, 0, 0.f, 0.f, 0.f, 0u, part);
  tm_status s = launch(pl, tmk::kKindFrob, 0, 0, 0, 0.f, 0.f, 0.f, tmk::kFromPart, part);
  if (s == TM_OK)
    s = launch(pl, tmk::kKindAolVector, 0, 0, 0, pl.raise, 0.f, 0.f, tmk::kFrob | tmk::kS4 | raise_flag(pl), 0);
  return s;
}

// Row-partial flags of the first Gram for a pre-conditioning.
uint32_t first_gram_flags(int precond) {
  if (precond == TM_PRECOND_AOL) return tmk::kRowSum;
  if (precond == TM_PRECOND_SCHATTEN4) return tmk::kRowSum | tmk::kRowSq;
  return 0u;
}

// Scale vector s of a call that has formed its first Gram (gram_scale; for
// Algorithm 1 the trace of the first Gram, ||X0||_F^2).
tm_status first_scale(const Plan& pl, int precond, int part) {
  if (precond == TM_PRECOND_FROBENIUS)
    return launch(pl, tmk::kKindAolVector, 0, 0, 0, pl.raise, 0.f, 0.f, tmk::kFrob | tmk::kTrace | raise_flag(pl), 0);
  return gram_scale(pl, precond, part);
}

// Coefficients of iteration `it` (0-based).
struct Triple {
  float a, b, c;
};
Triple triple(const float* coeffs, int it) {
  return coeffs ? Triple{coeffs[3 * it], coeffs[3 * it + 1], coeffs[3 * it + 2]} : Triple{kA, kB, kC};
}

// Whether a call's k x k matrices stay within fp16's range (pairs, planes).  After
// any scaling sigma_max(X1) <= 1, so every A, T = B~ A and B~ of the call is
// bounded by its coefficients: with x the largest sigma^2, |B~| <= max |q| over
// [0, x], q(x) = a + b x + c x^2, and the next x is the largest x q(x)^2.  The call
// qualifies while A and T stay below 8 (32768 as stored, half of fp16's largest)
// and B~ below 32 (32768).  *growth: the most that all iterations together
// multiply a row by, the product of max |q| (at least 1 each).
bool half_ok(int iters, const float* coeffs, int precond, double top_b, double* growth) {
  *growth = 1.0;
  if (precond == TM_PRECOND_NONE) return false;
  double x = 1.02;   // the scale's own rounding
  for (int it = 0; it < iters; ++it) {
    const Triple t = triple(coeffs, it);
    const double a = t.a, b = t.b, c = t.c;
    auto q = [&](double v) { return a + b * v + c * v * v; };
    double top = std::max(std::fabs(a), std::fabs(q(x)));
    if (c != 0.0 && -b / (2 * c) > 0.0 && -b / (2 * c) < x) top = std::max(top, std::fabs(q(-b / (2 * c))));
    if (!(x <= 8.0 && top <= top_b && x * top <= 8.0)) return false;
    *growth *= std::max(top, 1.0);
    double nx = 0.0;
    constexpr int S = 128;
    for (int i = 1; i <= S; ++i) {
      const double v = x * i / S;
      nx = std::max(nx, v * q(v) * q(v));
    }
    x = 1.02 * nx;   // between the samples, and the rounding of the products
  }
  return x <= 8.0;
}

// Small rows under a uniform scale (Frobenius, Schatten-4), which AOL brings to
// like sizes: beside rows of size 1 their entries of A, B~ and Y fall below what
// fp16 (times kScaleA and so on) or two fp16 planes hold, so that a row of 2^-30 came
// out 100% (pairs) and 6e-3 (planes, 1024 x 2048) of itself off, and one of 2^-50 as
// zero.  They are therefore worked on at a size of `raise`, 2^-18 or so: s_i is s
// times a power of two, and the last update takes the factor out again (both
// exact).  To the other rows and to its own q(Y^T Y) such a row is the square of
// raise times the growth: 96 x 500 to 1024 x 2048, rows of 2^-10 to 2^-60, five
// iterations of a = 3.44 (growth 2^9): small rows are 4e-7 off (planes) and 6e-3
// (pairs), as the others are.  2^-14 is too large (1e-5), 2^-22 begins to show the
// formats' resolution (2e-6): from a growth of 2^14 on (8 iterations of the default
// coefficients) neither fits, and uniform scales keep the fp32 products and the
// step-by-step form.  0: no raise there.  (A row's size is that of its A0_ii: one whose
// squares underflow, below 1e-19 itself, stays as it is.)
float raise_to(double growth) {
  const int e = -8 - int(std::ceil(std::log2(growth)));
  return e < -22 ? 0.f : std::ldexp(1.f, std::min(e, -18));
}

// Two iterations per update (class 1).  Iterations k, k + 1 as printed take two
// Grams, two polynomials and two updates, (6 N + 2 k) k^2 operations.  As
// B~ and A are polynomials of one matrix, the second Gram is B~ A B~ and the
// two updates are one by Q = B~' B~: one Gram, five k x k products (A A,
// T = B~ A, B~ T, A' A', Q, upper halves) and one update, (3 N + 5 k) k^2.
// The k x k matrices are fp16 (11 bits against bf16's 8), and one bf16
// rounding of Y drops out: the error against 64 bits is about half of the
// step-by-step form's on every spectrum tried.  More than two would be
// fewer operations still, but the Gram's rounding error then grows by a^2 for
// every further iteration and passes the step-by-step form's on spectra with
// many small singular values.
// The line.  Pairs save 3 (N - k) k^2 operations per two iterations and add three
// dependent k x k products, each of a chain's 4 to 7 us below k = 1280 or so and
// of two waves of tiles and more above.  Times in pairs over step by step, four
// iterations, by N - k and matrices in the call (k = 64 to 8192 measured):
//            1280           1536           1792           2048           3072
//   k     1   4   24     1   4   24     1   4   24     1   4   24     1   4   24
//   256  1.04 1.00 1.02 1.03 0.98 1.01 1.01 0.96 1.00 0.99 0.93 0.96 0.94 0.90 0.89
//   512  1.03 1.01 0.88 1.03 1.00 0.87 0.98 0.95 0.83 0.98 0.93 0.85 0.94 0.90 0.67
//   768  1.06 1.00 0.87 1.05 0.97 0.84 1.02 0.94 0.83 0.99 0.87 0.78 1.03 0.84 0.73
//   1024 1.03 0.94 0.88 1.01 0.93 0.85 1.01 0.92 0.83 0.99 0.91 0.80 0.95 0.94 0.75
//   1280 1.01 0.97 0.93 1.01 0.95 0.90 1.00 0.93 0.88 0.92 0.75 0.84 0.88 0.79 0.79
//   2048 0.99 0.97      0.97 0.95      0.96 0.93      0.95 0.92      0.90 0.84
//   3072 1.07 0.96      1.07 0.94      1.04 0.93      1.01 0.92      0.93
//   8192 1.02           1.01           1.01           1.00           0.95
// So a lone matrix breaks even where N - k is about 2048 whatever k (above 8192 k / 4
// is assumed, as from 4096 to 8192), batches earlier.  Beside other matrices that go
// step by step the two chains share only some of their launches, which is up to 50 us
// more a call; three layers of four k x k, a k x N and an N x k matrix, pairs over step
// by step by N - k:
//   k      2048  2560  3072  4096        k      1024  1536  2048  2560  3072
//   256    1.17  1.15  1.12  1.08        1024         1.05  1.05  1.00  0.95
//   384    1.12  1.02  1.01  0.97        1152   1.08  1.03  1.00  0.97
//   512    1.04  1.01        0.96        1280         1.07  1.04  1.01  0.95
//   640    1.04  0.98  0.98              1408   1.02  0.98  0.95  0.93
//   768    1.02  0.95  0.92  0.83        1536   1.01  0.99  0.99        0.94
// (768 x 2688 1.02, 768 x 3072 0.96; 12 layers gain 3 to 10% at 2048 from k = 320 on; two
// layers of 2048, 3072 and 4096 at 2048 1.00, 0.98 and 0.98.)  So around 768, where the
// products of such a group fill a wave, the line is 3 k, up to 2560.  From 1280 on, where
// a few matrices fill the chip, it is k, up to 2048: 2 x 1555 x 3182 461 and 413 us,
// 9 x 1396 x 3144 (3 iterations) 846 and 784, against 2 to 5% in such mixed groups.
// Below 683 it is the lone matrix's: 16 x 256 x 2304 beside the other 3 x 3 convolutions of
// a ResNet, which run fused or in pairs, 464 and 416 us (but 12 x 256 x 256 with
// 2 x 256 x 2304 93 and 115); below 256 a call is too short to make up for a loss
// (8 x 128 x 512 with 2 x 192 x 2240 88 and 108).  Three iterations (one pair and one step) break
// even where four do (768: 1.00, 1024: 1.00, 2048: 0.98 at 2048); two alone twice as far
// (768 x 3840 1.20, 512 x 4608 1.00, 1024 x 5120 0.94) but from k = 1536 on (2048 x 4096 1.01
// and, 8 of them, 0.94).  The rule depends on the shape and iters alone, so that a
// matrix comes out the same from a single, a batched and a grouped call.
bool pair_rule(const Item& it, int iters) {
  const uint64_t k = it.k, d = uint64_t(it.N) - it.k;
  if (k < 256 || iters < 2) return false;
  const uint64_t line = k < 1280 ? std::max<uint64_t>(2048, std::min<uint64_t>(3 * k, 2560))
                                 : (k < 2048 ? k : std::max<uint64_t>(2048, k / 4));
  return d >= (iters == 2 && k < 1536 ? 4096 : line);
}

// fp32 matrices on fp16 planes.  Times on the fp32 products and on planes: 4096 x 4096
// 12.65 and 3.4 ms, 256 x 256 162 and 105 us, 600 of 64 x 64 1.20 and 0.15 ms, of
// 65 x 65 (128 x 128 as padded) 1.67 and 0.38, of 129 x 129 3.1 and 0.91, of 193 x 1000 10.7
// and 4.5; the closest of 400 calls from k = 64 to 385 64 x 96 x 96, 108.9 and 110.9 us.  Errors
// against 64 bits, planes over fp32: 0.31 to 0.86, median 0.51 (k = 64 to 1024, N = 1 to
// 9 k, every scale, 3 to 5 iterations): fewer roundings in the sums outweigh the planes'
// 22 to 23 bits.  The line is the smallest tile.  Planes are faster below it too (600 of
// 34 x 34 1.12 and 0.15 ms, one of 63 x 63 80 and 74 us), but there the padding of k
// alone is a workspace of up to (64 / k)^2 times the size, and short sums are not where
// planes gain accuracy (64 x 64: 0.62).
bool split_rule(const Item& it) { return it.k >= 64; }

// The k x k products and update of iterations [it, it + n) of one class (1:
// `pair`), n = 1 or 2, from A in kBufA; `scaled`: the update's factor times
// diag(s).
void block_steps(std::vector<Step>& out, bool pair, bool split, int it, int n, const float* coeffs, bool scaled,
                 int src, int dst, uint32_t update_flags) {
  const float sa = pair || split ? tmk::kScaleA : 1.f, sb = pair || split ? tmk::kScaleB : 1.f;
  auto product = [&](int l, int r, int m, int o, float al, float be, float ga, bool factor) {
    Step s{tmk::kKindPoly, 0u};
    s.l = l, s.r = r, s.m = m, s.out = o;
    s.alpha = al, s.beta = be, s.gamma = ga;
    s.mode = !pair ? (scaled ? tmk::kSymBf16Scaled : tmk::kSymBf16)
                   : (!factor ? tmk::kSymHalf : (scaled ? tmk::kSymFactorScaled : tmk::kSymFactor));
    out.push_back(s);
  };
  // B~ = b A + c A A + a I, times `f` (1 for a bf16 update's factor, else kScaleB)
  auto poly = [&](int i, int o, bool factor) {
    const Triple t = triple(coeffs, i);
    const float f = factor && !split ? 1.f : sb;
    product(tmk::kBufA, tmk::kBufA, tmk::kBufA, o, t.c * (f / (sa * sa)), t.b * (f / sa), t.a * f, factor);
  };
  Step u{tmk::kKindUpdate, update_flags};
  u.src = src;
  u.dst = dst;
  if (n == 1) {
    poly(it, tmk::kBufB, true);
  } else {
    poly(it, tmk::kBufB, false);
    product(tmk::kBufB, tmk::kBufA, tmk::kNoBuf, tmk::kBufT, 1.f / sb, 0.f, 0.f, false);   // T = B~ A
    product(tmk::kBufB, tmk::kBufT, tmk::kNoBuf, tmk::kBufA, 1.f / sb, 0.f, 0.f, false);   // A' = B~ T
    poly(it + 1, tmk::kBufT, false);                                                       // B~'
    product(tmk::kBufT, tmk::kBufB, tmk::kNoBuf, tmk::kBufA, 1.f / (sb * sb), 0.f, 0.f, true);   // Q
    u.fac = tmk::kBufA;
  }
  out.push_back(u);
}

// Runs the two classes' step lists, sharing launches where their kinds meet
// in order (a longest common subsequence): classes that run apart would each
// leave a partly filled last wave per launch.
tm_status run_steps(const Plan& pl, const std::vector<Step> (&seq)[2]) {
  const size_t n = seq[0].size(), m = seq[1].size();
  auto meet = [&](size_t i, size_t j) {
    const Step &a = seq[0][i], &b = seq[1][j];
    return a.kind == b.kind && a.flags == b.flags &&
           (a.kind != tmk::kKindPoly || (a.mode == tmk::kSymBf16 && b.mode == tmk::kSymHalf));
  };
  std::vector<int> best((n + 1) * (m + 1), 0);   // shared launches of the suffixes
  auto at = [&](size_t i, size_t j) -> int& { return best[i * (m + 1) + j]; };
  for (size_t i = n; i-- > 0;)
    for (size_t j = m; j-- > 0;)
      at(i, j) = meet(i, j) ? at(i + 1, j + 1) + 1 : std::max(at(i + 1, j), at(i, j + 1));
  size_t i = 0, j = 0;
  tm_status s = TM_OK;
  while (s == TM_OK && (i < n || j < m)) {
    const Step* st[2] = {nullptr, nullptr};
    if (i < n && j < m && meet(i, j)) {
      st[0] = &seq[0][i++];
      st[1] = &seq[1][j++];
    } else if (j == m || (i < n && at(i + 1, j) >= at(i, j + 1))) {
      st[0] = &seq[0][i++];
    } else {
      st[1] = &seq[1][j++];
    }
    const Step& any = st[0] ? *st[0] : *st[1];
    s = launch(pl, any.kind, 0, 0, 0, 0.f, 0.f, 0.f, any.flags, 0, kCoverAll, st);
  }
  return s;
}

// bf16, and fp32 on fp16 planes (Plan::split): zero-padded tiled workspace,
// matrix-core kernels of tm_fast.hip.
tm_status plan_tiled(const Plan& pl, int iters, const float* coeffs, int precond) {
  const bool frob = precond == TM_PRECOND_FROBENIUS;
  const bool from_gram = precond == TM_PRECOND_AOL || precond == TM_PRECOND_SCHATTEN4;
  const bool scaled = from_gram || frob;
  const uint32_t rflags = first_gram_flags(precond);
  const int part = tmk::kMinTile;   // the matrix-core Gram emits row partials per 64 columns
  // AOL with at most 16 row partials per row: the rescale pass sums s itself
  // (same order as the AOL-vector kernel), one launch fewer per call
  const bool fuse_s = precond == TM_PRECOND_AOL &&
                      std::all_of(pl.items->begin(), pl.items->end(),
                                  [&](const Item& it) { return it.kp <= uint32_t(16 * part); });
  tm_status s = TM_OK;
  if (pl.split) s = launch(pl, tmk::kKindLoadIn, tmk::kCfgRowMax, 0, 0, 0.f, 0.f, 0.f, 0u, 0);
  if (s == TM_OK && (iters > 0 || from_gram))
    s = launch(pl, tmk::kKindLoadIn, 0, 0, 0, 0.f, 0.f, 0.f, 0u, 0, kCoverCopied);
  if (s != TM_OK) return s;
  // the first Gram, of every matrix: A0 in fp32 where it is rescaled, then A1
  Step g0{tmk::kKindGram, rflags | (scaled ? tmk::kA32 : 0u)};
  g0.src = tmk::kSlotFirst;
  const Step* const both[2] = {&g0, &g0};
  auto gram = [&]() {
    return launch(pl, g0.kind, 0, 0, 0, 0.f, 0.f, 0.f, g0.flags, 0, kCoverAll, both);
  };
  if (iters == 0) {
    if (frob) {  // Algorithm 1, first line: s = 1 / ||X0||_F
      s = launch(pl, tmk::kKindFrob, 0, 0, 0, 0.f, 0.f, 0.f, 0u, 0);
      if (s == TM_OK) s = launch(pl, tmk::kKindAolVector, 0, 0, 0, 0.f, 0.f, 0.f, tmk::kFrob, 0);
    } else if (from_gram) {
      s = gram();
      if (s == TM_OK) s = gram_scale(pl, precond, part);
    }
    if (s == TM_OK && scaled) s = launch(pl, tmk::kKindApplyScale, 0, 0, 0, 0.f, 0.f, 0.f, 0u, 0);
    return s;
  }
  s = gram();
  if (s == TM_OK && scaled && !fuse_s) s = first_scale(pl, precond, part);
  if (s == TM_OK && scaled)         // A1 = diag(s) A0 diag(s), one rounding
    s = launch(pl, tmk::kKindScaleA, 0, 0, 0, 0.f, 0.f, 0.f, fuse_s ? tmk::kFuseS : 0u, part);
  if (s != TM_OK) return s;
  // The iterations, from A1.  The first block's factor is stored times diag(s)
  // and its update reads X0.
  std::vector<Step> seq[2];
  for (int cls = 0; cls < 2; ++cls) {
    if (std::none_of(pl.items->begin(), pl.items->end(),
                     [&](const Item& it) { return it.pair == (cls == 1); }))
      continue;
    int src = tmk::kSlotFirst;
    for (int it = 0; it < iters;) {
      const int n = cls == 1 ? std::min(2, iters - it) : 1;
      const int dst = it + n == iters ? tmk::kSlotFinal
                                      : (src == tmk::kSlotAlt1 ? tmk::kSlotAlt2 : tmk::kSlotAlt1);
      if (it > 0) {
        Step g{tmk::kKindGram, 0u};
        g.src = src;
        seq[cls].push_back(g);
      }
      block_steps(seq[cls], cls == 1, pl.split, it, n, coeffs, it == 0 && scaled, src, dst, raise_flag(pl));
      src = dst;
      it += n;
    }
  }
  return run_steps(pl, seq);
}

// fp32: generic kernels of tm_kernels.hip.
tm_status plan_f32(const Plan& pl, int iters, const float* coeffs, int precond) {
  const std::vector<Item>& items = *pl.items;
  tm_status s = TM_OK;
  const bool frob = precond == TM_PRECOND_FROBENIUS;
  const bool from_gram = precond == TM_PRECOND_AOL || precond == TM_PRECOND_SCHATTEN4;
  const bool scaled = from_gram || frob;
  const uint32_t rflags = first_gram_flags(precond);
  bool any_tall = false;
  for (const Item& it : items) any_tall = any_tall || it.tall;
  if (any_tall && (iters > 0 || from_gram)) {
    s = launch(pl, tmk::kKindTransposeIn, 0, 0, 0, 0.f, 0.f, 0.f, 0u, 0, kCoverTall);
    if (s != TM_OK) return s;
  }
  const int gcfg = choose_cfg_f32(tmk::kKindGram, items);
  const int pcfg = choose_cfg_f32(tmk::kKindPoly, items);
  const int ucfg = choose_cfg_f32(tmk::kKindUpdate, items);
  const int part = tmk::cfg_tile(gcfg);   // row partials per Gram tile column block

  if (iters == 0) {
    if (frob) {  // Algorithm 1, first line: s = 1 / ||X0||_F
      s = launch(pl, tmk::kKindFrob, 0, 0, 0, 0.f, 0.f, 0.f, 0u, 0);
      if (s == TM_OK) s = launch(pl, tmk::kKindAolVector, 0, 0, 0, 0.f, 0.f, 0.f, tmk::kFrob, 0);
      if (s != TM_OK) return s;
    }
    if (from_gram) {
      s = launch(pl, tmk::kKindGram, gcfg, tmk::kSlotFirst, 0, 0.f, 0.f, 0.f, rflags | tmk::kA32, 0);
      if (s == TM_OK) s = gram_scale(pl, precond, part);
      if (s != TM_OK) return s;
    }
    if (scaled) s = launch(pl, tmk::kKindApplyScale, 0, 0, 0, 0.f, 0.f, 0.f, 0u, 0);
    return s;
  }

  int src = tmk::kSlotFirst;
  for (int it = 1; it <= iters; ++it) {
    const float a = coeffs ? coeffs[3 * (it - 1)] : kA;
    const float b = coeffs ? coeffs[3 * (it - 1) + 1] : kB;
    const float c = coeffs ? coeffs[3 * (it - 1) + 2] : kC;
    // A single iteration would read and write the caller's buffer: it goes
    // through W1 and a final copy instead.
    const int dst = (it == iters && iters > 1) ? tmk::kSlotFinal
                                               : (it % 2 == 1 ? tmk::kSlotAlt1 : tmk::kSlotAlt2);
    const bool first = it == 1;
    const uint32_t scale = (first && scaled) ? tmk::kScale : 0u;
    const uint32_t gflags = (first ? rflags : 0u) | (scale ? tmk::kA32 : 0u);
    s = launch(pl, tmk::kKindGram, gcfg, src, 0, 0.f, 0.f, 0.f, gflags, 0);
    if (s == TM_OK && first && scaled) s = first_scale(pl, precond, part);
    if (s == TM_OK) s = launch(pl, tmk::kKindPoly, pcfg, 0, 0, a, b, c, scale, 0);
    if (s == TM_OK) s = launch(pl, tmk::kKindUpdate, ucfg, src, dst, a, b, c, scale, 0);
    if (s != TM_OK) return s;
    src = dst;
  }
  if (iters == 1) s = launch(pl, tmk::kKindCopyOut, 0, src, 0, 0.f, 0.f, 0.f, 0u, 0);
  return s;
}

// Workspace of a call in the form that needs the most, each on its smallest
// layout (fp32 on planes needs more than on the fp32 kernels).
uint64_t smallest_bytes(std::vector<Item> items, int esz) {
  uint64_t total = 0;
  for (Item& it : items) {
    if (esz == 2 || split_rule(it)) tmk::tiled_dims(it.k, it.N, tmk::kMinTile, &it.kp, &it.Np);
    else tmk::generic_dims(it.k, it.N, &it.kp, &it.Np);
    total += item_ws(it, esz);
  }
  return total;
}

// Plan and enqueue one call (g_mu held, device checked).  With ext_ws the
// call runs in that caller-provided device buffer of ext_bytes bytes (the
// allocation-free entry point) instead of the per-stream workspace cache, and
// its launches are never bracketed by the timing hooks' events.
tm_status run_locked(std::vector<Item>& items, int esz, int iters, const float* coeffs,
                     int precond, hipStream_t st, int dev, char* ext_ws = nullptr,
                     uint64_t ext_bytes = 0) {
  tm_status s = TM_OK;
  // bf16 calls made only of small matrices: the fused kernel, one launch
  // (TM_DISABLE_FUSED in the environment keeps them on the tiled kernels)
  if (esz == 2 && iters >= 1 && std::all_of(items.begin(), items.end(), small_eligible) &&
      std::getenv("TM_DISABLE_FUSED") == nullptr) {
    Plan pl;
    pl.items = &items;
    pl.esz = esz;
    pl.st = st;
    pl.ws = nullptr;
    pl.timed = ext_ws == nullptr;
    (void)dev;
    return plan_small(pl, iters, coeffs, precond);
  }
  // A call of more than kMaxEntries items runs every phase as several
  // launches; largest products first, so the last, partly filled launch
  // holds the shortest tiles.  Each matrix's arithmetic does not depend on
  // the launch it lands in.
  if (items.size() > size_t(tmk::kMaxEntries))
    std::stable_sort(items.begin(), items.end(), [](const Item& x, const Item& y) {
      return double(x.k) * x.k * x.N * x.count > double(y.k) * y.k * y.N * y.count;
    });
  const bool cap = ext_ws == nullptr && capturing(st);
  const bool uniform = precond != TM_PRECOND_AOL;
  double growth;
  const bool half = half_ok(iters, coeffs, precond, esz == 2 ? 32.0 : 16.0, &growth);
  const float raise = half && uniform ? raise_to(growth) : 0.f;
  // pairs (bf16), planes (fp32)
  const bool fp16 = half && (!uniform || raise > 0.f);
  // What a call of these shapes needs in any form (they differ by iters, coefficients
  // and precond), on the smallest tile: reserved by every call, so that one call serves
  // the capture of any other of the same or smaller shapes.
  const uint64_t every_form = smallest_bytes(items, esz);
  // A call whose matrices are pairs but for some in the fused kernel's range runs
  // those there, in one launch: step by step on tiles they would add about eight
  // launches to the pairs' chain.  (Bit for bit the same results.)
  std::vector<Item> small;
  if (esz == 2 && fp16 && std::getenv("TM_DISABLE_FUSED") == nullptr) {
    std::vector<Item> pairs;
    for (const Item& it : items) (pair_rule(it, iters) ? pairs : small).push_back(it);
    if (!pairs.empty() && std::all_of(small.begin(), small.end(), small_eligible)) items = pairs;
    else small.clear();
  }
  // parts of the call that run one after the other: bf16 is one, fp32 the
  // matrices on fp16 planes (`planes`) and the others
  std::vector<Item> part[2];
  Plan pl[2];
  auto lay_out = [&](bool planes, uint64_t limit) {
    uint64_t total = 0;
    for (int p = 0; p < 2; ++p) {
      part[p].clear();
      pl[p] = Plan();
    }
    for (const Item& it : items) part[esz == 2 || (planes && split_rule(it)) ? 0 : 1].push_back(it);
    uint64_t rest = 0;   // the other part's layout is what it is
    for (Item& it : part[1]) {
      tmk::generic_dims(it.k, it.N, &it.kp, &it.Np);
      rest += item_ws(it, esz);
    }
    for (int p = 0; p < 2; ++p) {
      if (part[p].empty()) continue;
      pl[p].items = &part[p];
      pl[p].esz = esz;
      pl[p].st = st;
      pl[p].split = p == 0 && esz == 4;
      if (p == 0) {
        bool any16 = pl[p].split;
        for (Item& it : part[p]) {
          it.pair = esz == 2 && fp16 && pair_rule(it, iters);
          any16 = any16 || it.pair;
        }
        pl[p].raise = any16 ? raise : 0.f;
        pl[p].tcfg = layout_cfg(shapes_of(part[p]), esz, limit == UINT64_MAX ? limit : limit - std::min(limit, rest));
        for (Item& it : part[p]) {
          tmk::tiled_dims(it.k, it.N, uint32_t(tmk::cfg_tile(pl[p].tcfg)), &it.kp, &it.Np);
          const int updates = it.pair ? (iters + 1) / 2 : iters;
          // A wide matrix that needs no padding is read in place by the first
          // update; a single update would read and write the caller's buffer in
          // the same launch, so it keeps the copy.
          it.direct = esz == 2 && !it.tall && it.kp == it.k && it.Np == it.N && updates != 1 &&
                      (reinterpret_cast<uintptr_t>(it.x) & 15u) == 0u;
        }
      }
      pl[p].shapes = shapes_of(part[p]);
      std::memset(pl[p].tile_of, -1, sizeof(pl[p].tile_of));
      for (const Item& it : part[p]) {
        pl[p].ws_off.push_back(total);
        total += item_ws(it, esz);
      }
    }
    return total;
  };
  const bool planes = esz == 4 && iters > 0 && fp16;
  uint64_t total = lay_out(planes, cap ? g_ws[{dev, st}].bytes : UINT64_MAX);
  if (total >= (uint64_t(1) << 40))   // entries hold offsets in 256-byte units
    return fail(TM_ERR_UNSUPPORTED, "workspace of more than 1 TB");
  char* ws = ext_ws;
  if (ext_ws != nullptr) {
    if (total > ext_bytes)
      return fail(TM_ERR_UNSUPPORTED, "the call needs " + std::to_string(total) +
                                          " bytes of scratch; the static scratch holds " +
                                          std::to_string(ext_bytes));
  } else {
    s = get_workspace(dev, st, size_t(total), size_t(every_form), cap, &ws);
    // short of memory: the layout with the least padding, then (fp32) the kernels
    // that need none
    for (int least = 0; least < (planes ? 2 : 1) && s == TM_ERR_NO_MEMORY; ++least) {
      total = lay_out(planes && least == 0, 0);
      s = get_workspace(dev, st, size_t(total), size_t(total), cap, &ws);
    }
    if (s != TM_OK) return s;
    g_last_error.clear();
  }
  // nothing is enqueued before this point, where the call can still fail
  if (!small.empty()) {
    Plan ps;
    ps.items = &small;
    ps.esz = esz;
    ps.st = st;
    ps.ws = nullptr;
    ps.timed = ext_ws == nullptr;
    s = plan_small(ps, iters, coeffs, precond);
  }
  for (int p = 0; p < 2 && s == TM_OK; ++p) {
    if (part[p].empty()) continue;
    pl[p].ws = ws;
    pl[p].timed = ext_ws == nullptr;
    s = p == 0 ? plan_tiled(pl[p], iters, coeffs, precond) : plan_f32(pl[p], iters, coeffs, precond);
  }
  return s;
}

tm_status run(std::vector<Item>& items, int esz, int iters, const float* coeffs, int precond,
              hipStream_t st) {
  if (items.empty()) return TM_OK;
  std::lock_guard<std::mutex> lock(g_mu);
  int dev = 0;
  tm_status s = check_device(&dev);
  if (s != TM_OK) return s;
  return run_locked(items, esz, iters, coeffs, precond, st, dev);
}

// Enqueue one elementwise optimizer launch per chunk of kMaxOptEntries
// matrices (timed as its own phase when the timing hooks are on).
tm_status launch_opt(int apply, const std::vector<tmk::OptEntry>& ents, const tmk::OptPhase& base,
                     hipStream_t st) {
  for (size_t b0 = 0; b0 < ents.size(); b0 += tmk::kMaxOptEntries) {
    tmk::OptPhase P = base;
    const size_t cnt = std::min(ents.size() - b0, size_t(tmk::kMaxOptEntries));
    uint64_t blocks = 0;
    for (size_t i = 0; i < cnt; ++i) {
      P.e[i] = ents[b0 + i];
      P.e[i].block_start = uint32_t(blocks);
      blocks += (P.e[i].size + tmk::kOptBlock - 1) / tmk::kOptBlock;
    }
    if (blocks >= (uint64_t(1) << 31)) return fail(TM_ERR_UNSUPPORTED, "too many blocks in one launch");
    P.nent = int32_t(cnt);
    P.total = uint32_t(blocks);
    TimedLaunch tl{apply ? int(tmk::kKindOptApply) : int(tmk::kKindOptMomentum), nullptr, nullptr};
    if (g_timing && P.total > 0) {
      if (hipEventCreate(&tl.start) != hipSuccess || hipEventCreate(&tl.stop) != hipSuccess)
        return fail(TM_ERR_HIP, "hipEventCreate failed");
      (void)hipEventRecord(tl.start, st);
    }
    const hipError_t e = tmk::launch_opt(apply, P, st);
    if (tl.start) {
      (void)hipEventRecord(tl.stop, st);
      g_timed.push_back(tl);
    }
    if (e != hipSuccess) return fail(TM_ERR_HIP, std::string("kernel launch: ") + hipGetErrorString(e));
  }
  return TM_OK;
}

tm_status check_common(int iters, const float* coeffs, int precond) {
  if (iters < 0 || iters > TM_MAX_ITERS)
    return fail(TM_ERR_INVALID_ARG, "iters out of range [0, " + std::to_string(TM_MAX_ITERS) + "]");
  if (precond != TM_PRECOND_NONE && precond != TM_PRECOND_FROBENIUS && precond != TM_PRECOND_AOL &&
      precond != TM_PRECOND_SCHATTEN4)
    return fail(TM_ERR_INVALID_ARG, "unknown precond " + std::to_string(precond));
  (void)coeffs;
  return TM_OK;
}

tm_status check_shape(int64_t m, int64_t n) {
  if (m < 1 || n < 1 || m > TM_MAX_DIM || n > TM_MAX_DIM)
    return fail(TM_ERR_INVALID_ARG, "matrix size " + std::to_string(m) + "x" + std::to_string(n) +
                                        " out of range [1, " + std::to_string(TM_MAX_DIM) + "]");
  return TM_OK;
}

Item make_item(void* X, int64_t m, int64_t n, int64_t count) {
  Item it;
  it.x = static_cast<char*>(X);
  it.tall = m > n;
  it.direct = false;
  it.pair = false;
  it.k = uint32_t(std::min(m, n));
  it.N = uint32_t(std::max(m, n));
  it.kp = it.k;
  it.Np = it.N;
  it.count = uint32_t(count);
  return it;
}

tm_status check_batched(void* X, int64_t m, int64_t n, int64_t batch, int iters,
                        const float* coeffs, int precond, int esz) {
  g_last_error.clear();
  tm_status s = check_common(iters, coeffs, precond);
  if (s != TM_OK) return s;
  if (batch < 0) return fail(TM_ERR_INVALID_ARG, "batch < 0");
  s = check_shape(m, n);
  if (s != TM_OK) return s;
  if (batch == 0) return TM_OK;
  if (X == nullptr) return fail(TM_ERR_INVALID_ARG, "X is NULL");
  if (reinterpret_cast<uintptr_t>(X) % uintptr_t(esz) != 0)
    return fail(TM_ERR_UNSUPPORTED, "X is not aligned to its element size");
  if (batch > INT32_MAX) return fail(TM_ERR_INVALID_ARG, "batch too large");
  return TM_OK;
}

tm_status batched(void* X, int64_t m, int64_t n, int64_t batch, int iters, const float* coeffs,
                  int precond, void* stream, int esz) {
  tm_status s = check_batched(X, m, n, batch, iters, coeffs, precond, esz);
  if (s != TM_OK || batch == 0) return s;
  std::vector<Item> items{make_item(X, m, n, batch)};
  return run(items, esz, iters, coeffs, precond, static_cast<hipStream_t>(stream));
}

tm_status grouped(void* const* X, const int64_t* m, const int64_t* n, int64_t count, int iters,
                  const float* coeffs, int precond, void* stream, int esz) {
  g_last_error.clear();
  tm_status s = check_common(iters, coeffs, precond);
  if (s != TM_OK) return s;
  if (count < 0) return fail(TM_ERR_INVALID_ARG, "count < 0");
  if (count == 0) return TM_OK;
  if (X == nullptr || m == nullptr || n == nullptr)
    return fail(TM_ERR_INVALID_ARG, "X, m or n is NULL");
  std::vector<Item> items;
  items.reserve(size_t(count));
  for (int64_t g = 0; g < count; ++g) {
    s = check_shape(m[g], n[g]);
    if (s != TM_OK) return fail(s, "matrix " + std::to_string(g) + ": " + g_last_error);
    if (X[g] == nullptr) return fail(TM_ERR_INVALID_ARG, "X[" + std::to_string(g) + "] is NULL");
    if (reinterpret_cast<uintptr_t>(X[g]) % uintptr_t(esz) != 0)
      return fail(TM_ERR_UNSUPPORTED, "X[" + std::to_string(g) + "] is not element aligned");
    items.push_back(make_item(X[g], m[g], n[g], 1));
  }
  return run(items, esz, iters, coeffs, precond, static_cast<hipStream_t>(stream));
}

}  // namespace

namespace tmk {

// Argument checks of tm_orthogonalize (nothing is enqueued).
tm_status check_batched_bf16(void* X, int64_t m, int64_t n, int64_t batch, int iters,
                             const float* coeffs, int precond) {
  return check_batched(X, m, n, batch, iters, coeffs, precond, 2);
}

// tm_orthogonalize in a caller-provided device buffer `ws` of `ws_bytes`
// (arguments already checked, batch > 0): the same plan and kernels as the
// cached-workspace call, so the results are bitwise equal to it.
tm_status run_batched_bf16_in(void* X, int64_t m, int64_t n, int64_t batch, int iters,
                              const float* coeffs, int precond, void* stream, char* ws,
                              uint64_t ws_bytes) {
  std::vector<Item> items{make_item(X, m, n, batch)};
  std::lock_guard<std::mutex> lock(g_mu);
  int dev = 0;
  tm_status s = check_device(&dev);
  if (s != TM_OK) return s;
  return run_locked(items, 2, iters, coeffs, precond, static_cast<hipStream_t>(stream), dev, ws,
                    ws_bytes);
}

// Record a failure for tm_last_error().
tm_status fail_with(tm_status s, const char* msg) { return fail(s, msg); }

}  // namespace tmk

extern "C" {

tm_status tm_orthogonalize(void* X, int64_t m, int64_t n, int64_t batch, int iters,
                           const float* coeffs, int precond, void* stream) {
  return batched(X, m, n, batch, iters, coeffs, precond, stream, 2);
}

tm_status tm_orthogonalize_f32(float* X, int64_t m, int64_t n, int64_t batch, int iters,
                               const float* coeffs, int precond, void* stream) {
  return batched(X, m, n, batch, iters, coeffs, precond, stream, 4);
}

tm_status tm_orthogonalize_grouped(void* const* X, const int64_t* m, const int64_t* n,
                                   int64_t count, int iters, const float* coeffs, int precond,
                                   void* stream) {
  return grouped(X, m, n, count, iters, coeffs, precond, stream, 2);
}

tm_status tm_orthogonalize_grouped_f32(float* const* X, const int64_t* m, const int64_t* n,
                                       int64_t count, int iters, const float* coeffs,
                                       int precond, void* stream) {
  return grouped(reinterpret_cast<void* const*>(X), m, n, count, iters, coeffs, precond, stream, 4);
}

tm_status tm_muon_step_grouped(float* const* W, const float* const* G, float* const* M,
                               const int64_t* m, const int64_t* n, int64_t count, float lr,
                               float momentum, int nesterov, float weight_decay, int shape_scale,
                               int iters, const float* coeffs, int precond, void* stream) {
  g_last_error.clear();
  tm_status s = check_common(iters, coeffs, precond);
  if (s != TM_OK) return s;
  if (count < 0) return fail(TM_ERR_INVALID_ARG, "count < 0");
  if (count == 0) return TM_OK;
  if (W == nullptr || G == nullptr || M == nullptr || m == nullptr || n == nullptr)
    return fail(TM_ERR_INVALID_ARG, "W, G, M, m or n is NULL");
  for (int64_t g = 0; g < count; ++g) {
    s = check_shape(m[g], n[g]);
    if (s != TM_OK) return fail(s, "matrix " + std::to_string(g) + ": " + g_last_error);
    if (W[g] == nullptr || G[g] == nullptr || M[g] == nullptr)
      return fail(TM_ERR_INVALID_ARG, "matrix " + std::to_string(g) + ": NULL pointer");
    if ((reinterpret_cast<uintptr_t>(W[g]) | reinterpret_cast<uintptr_t>(G[g]) |
         reinterpret_cast<uintptr_t>(M[g])) % 4u != 0)
      return fail(TM_ERR_UNSUPPORTED, "matrix " + std::to_string(g) + ": pointer not 4-byte aligned");
  }
  hipStream_t st = static_cast<hipStream_t>(stream);
  std::lock_guard<std::mutex> lock(g_mu);
  int dev = 0;
  s = check_device(&dev);
  if (s != TM_OK) return s;
  uint64_t ubytes = 0;
  for (int64_t g = 0; g < count; ++g) ubytes += tmk::align256(uint64_t(m[g]) * uint64_t(n[g]) * 2u);
  char* ubase = nullptr;
  s = get_workspace(dev, st, size_t(ubytes), size_t(ubytes), capturing(st), &ubase, g_ws_u);
  if (s != TM_OK) return s;
  std::vector<tmk::OptEntry> ents(static_cast<size_t>(count));
  std::vector<Item> items;
  items.reserve(size_t(count));
  uint64_t off = 0;
  for (int64_t g = 0; g < count; ++g) {
    tmk::OptEntry& E = ents[size_t(g)];
    std::memset(&E, 0, sizeof(E));
    E.w = W[g];
    E.g = G[g];
    E.m = M[g];
    E.u = reinterpret_cast<uint16_t*>(ubase + off);
    E.size = uint64_t(m[g]) * uint64_t(n[g]);
    E.vec = ((reinterpret_cast<uintptr_t>(W[g]) | reinterpret_cast<uintptr_t>(G[g]) |
              reinterpret_cast<uintptr_t>(M[g])) & 15u) == 0u;
    E.scale = shape_scale ? std::sqrt(std::max(1.0f, float(m[g]) / float(n[g]))) : 1.0f;
    items.push_back(make_item(E.u, m[g], n[g], 1));
    off += tmk::align256(E.size * 2u);
  }
  tmk::OptPhase base;
  std::memset(&base, 0, sizeof(base));
  base.lr = lr;
  base.mu = momentum;
  base.wd = weight_decay;
  base.nesterov = nesterov ? 1 : 0;
  s = launch_opt(0, ents, base, st);                                          // M, bf16 U
  if (s == TM_OK) s = run_locked(items, 2, iters, coeffs, precond, st, dev);  // U <- O
  if (s == TM_OK) s = launch_opt(1, ents, base, st);                          // W
  return s;
}

const float* tm_schedule_tail(const float* schedule, int rows, int iters) {
  g_last_error.clear();
  if (schedule == nullptr) {
    fail(TM_ERR_INVALID_ARG, "schedule is NULL");
    return nullptr;
  }
  if (rows < 1 || rows > TM_MAX_ITERS || iters < 0 || iters > rows) {
    fail(TM_ERR_INVALID_ARG, "need 1 <= rows <= " + std::to_string(TM_MAX_ITERS) +
                                 " and 0 <= iters <= rows (rows " + std::to_string(rows) +
                                 ", iters " + std::to_string(iters) + ")");
    return nullptr;
  }
  return schedule + 3 * (rows - iters);
}

uint64_t tm_workspace_bytes(const int64_t* m, const int64_t* n, int64_t count, int dtype_bytes) {
  if (m == nullptr || n == nullptr || count < 0 || (dtype_bytes != 2 && dtype_bytes != 4)) return 0;
  std::vector<Item> items;
  for (int64_t g = 0; g < count; ++g) {
    if (m[g] < 1 || n[g] < 1 || m[g] > TM_MAX_DIM || n[g] > TM_MAX_DIM) return 0;
    items.push_back(make_item(nullptr, m[g], n[g], 1));
  }
  // fp32: as if the coefficients allow the fp16 planes (the default ones do)
  std::vector<Item> tiled;
  uint64_t total = 0;
  for (Item& it : items) {
    if (dtype_bytes == 2 || split_rule(it)) {
      tiled.push_back(it);
    } else {
      tmk::generic_dims(it.k, it.N, &it.kp, &it.Np);
      total += item_ws(it, dtype_bytes);
    }
  }
  if (tiled.empty()) return total;
  // The tile depends on the form that iters and coeffs give the call: step by
  // step, with pairs, and pairs without the matrices of the fused kernel.
  auto bytes = [&](const std::vector<Item>& part) {
    const std::vector<Item> shapes = shapes_of(part);
    return shapes.empty() ? 0 : laid_bytes(shapes, layout_cfg(shapes, dtype_bytes), dtype_bytes);
  };
  uint64_t most = bytes(tiled);
  for (int iters = 2; dtype_bytes == 2 && iters <= 3; ++iters) {   // pair_rule's two lines
    std::vector<Item> pairs;
    for (Item& it : tiled) {
      it.pair = pair_rule(it, iters);
      if (it.pair) pairs.push_back(it);
    }
    most = std::max(most, std::max(bytes(tiled), bytes(pairs)));
  }
  total += most;
  return total;
}

tm_status tm_release_workspaces(void) {
  std::lock_guard<std::mutex> lock(g_mu);
  if (g_ws.empty() && g_ws_u.empty() && g_retired.empty()) return TM_OK;
  hipError_t e = hipDeviceSynchronize();
  for (WsCache* c : {&g_ws, &g_ws_u}) {
    for (auto& kv : *c)
      if (kv.second.ptr) (void)hipFree(kv.second.ptr);
    c->clear();
  }
  for (void* p : g_retired) (void)hipFree(p);
  g_retired.clear();
  if (e != hipSuccess) return fail(TM_ERR_HIP, std::string("hipDeviceSynchronize: ") + hipGetErrorString(e));
  return TM_OK;
}

tm_status tm_timing_enable(int enable) {
  std::lock_guard<std::mutex> lock(g_mu);
  g_timing = enable != 0;
  return TM_OK;
}

tm_status tm_timing_read(int phase, double* total_ms, int64_t* launches) {
  if (phase < 0 || phase >= TM_NUM_PHASES || total_ms == nullptr || launches == nullptr)
    return fail(TM_ERR_INVALID_ARG, "bad phase or null output");
  std::lock_guard<std::mutex> lock(g_mu);
  collect_timing();
  *total_ms = g_time_ms[phase];
  *launches = g_time_n[phase];
  return TM_OK;
}

tm_status tm_timing_reset(void) {
  std::lock_guard<std::mutex> lock(g_mu);
  collect_timing();
  for (int i = 0; i < TM_NUM_PHASES; ++i) {
    g_time_ms[i] = 0.0;
    g_time_n[i] = 0;
  }
  return TM_OK;
}

const char* tm_status_string(tm_status s) {
  switch (s) {
    case TM_OK: return "TM_OK";
    case TM_ERR_INVALID_ARG: return "TM_ERR_INVALID_ARG";
    case TM_ERR_UNSUPPORTED: return "TM_ERR_UNSUPPORTED";
    case TM_ERR_NO_MEMORY: return "TM_ERR_NO_MEMORY";
    case TM_ERR_HIP: return "TM_ERR_HIP";
  }
  return "TM_ERR_UNKNOWN";
}

const char* tm_last_error(void) { return g_last_error.c_str(); }

const char* tm_version(void) { return "0.1.0"; }

}  // extern "C"
