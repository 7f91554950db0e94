// Host side of libasv: argument checks, workspace layouts, tile selection and the launch
// sequences of one verification step, one draft step, the pruning of the draft trees, the
// tree-attention metadata and the commit. Every entry point is declared in include/asv.h.
#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <mutex>

#include <cstdio>

#include "asv.h"
#include "k_accept.h"
#include "k_draft.h"
#include "k_lmhead.h"
#include "k_reduce.h"
#include "k_tree.h"

namespace asv {
namespace {

constexpr size_t kAlign = 256;

// Vocabulary slabs of K1's plan, one workgroup tile and one record per slab and row. Up to 64 rows
// the ids are cut anew (cut_rows64), up to 512 where that pays (cut_wide).
constexpr int kSlab = 256;
constexpr int kPackRowsTarget = 256;   // rows per tile of the packed target LM-head weight
constexpr int kPackRowsDraft = 64;     // rows per tile of the packed draft LM-head weight

// Text of the most recent failure on this host thread (see asv_last_error).
thread_local char g_last_error[256] = "";

void set_error(const char* what, hipError_t e) {
  snprintf(g_last_error, sizeof(g_last_error), "%s: %s (%d)", what, hipGetErrorString(e),
           (int)e);
}

// ASV_OK when the launches enqueued so far succeeded, else ASV_EHIP with the error recorded.
int launch_status(const char* what) {
  const hipError_t e = hipGetLastError();
  if (e == hipSuccess) return ASV_OK;
  set_error(what, e);
  return ASV_EHIP;
}

size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }

// Tile families of K1. Few rows (the weight-streaming regime of small batches) use a 64-row
// tile so that all rows share one pass over W. Beyond 64 rows the plan minimises an estimate of
// the time: the rounds of workgroups over the CUs times the time of one tile, 62 : 80 : 98 for
// the 128-, 192- and 256-row tiles (per-round times of the spread loops on MI355X, with the
// packed weight); ties go to the larger tile. Interleaved comparisons at V = 151936 (records
// bit-identical across the tiles) agree with the single-family estimate at every row count
// measured from 150 to 3048 rows: e.g. at 540 rows three 192-row tiles beat three 256-row tiles
// by 17%, at 700 rows three 256-row tiles beat four 192-row tiles by 9%.
// A plan may split the slabs between two families in two launches: the first n1 slabs on
// family a, the rest on family b, n1 chosen so that family a fills whole rounds. At 378 rows
// and V = 151936, for instance, one 192-row family takes 1188 tiles, 4.64 rounds run as 5;
// 128-row tiles on 85 slabs (255 tiles, one round) and 192-row tiles on the other 509 (1018
// tiles, four rounds) leave no round a third empty.
enum class Tile { kRows64, kRows128, kRows192, kRows256 };

struct K1Plan {
  Tile a, b;       // slabs [0, n1) on tile a, [n1, S) on tile b
  int n1;          // == S: one launch of tile a
};


// Compute units of the current device, queried once per device.
int cu_count() {
  static std::atomic<int> cached[64];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
  int n = cached[dev].load(std::memory_order_relaxed);
  if (n <= 0) {
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        n <= 0)
      n = 256;
    cached[dev].store(n, std::memory_order_relaxed);
  }
  return n;
}

// est: the plan's estimate (beyond 64 rows).
K1Plan plan_k1(int N, int S, int cus, int64_t* est_out = nullptr) {
  if (N <= 64) return K1Plan{Tile::kRows64, Tile::kRows64, S};
  struct Family { Tile tile; int rows; int cost; };
  const Family families[3] = {{Tile::kRows128, 128, 62}, {Tile::kRows192, 192, 80},
                              {Tile::kRows256, 256, 98}};
  auto rounds = [&](int64_t tiles) { return (tiles + cus - 1) / cus; };
  K1Plan best{Tile::kRows128, Tile::kRows128, S};
  int64_t best_est = INT64_MAX;
  for (const Family& f : families) {
    const int64_t est = rounds((int64_t)((N + f.rows - 1) / f.rows) * S) * f.cost;
    if (est <= best_est) {
      best_est = est;
      best = K1Plan{f.tile, f.tile, S};
    }
  }
  // two families: family a fills k whole rounds on its slabs, family b takes the rest; taken
  // only when strictly better than every single family. The search stops at kMaxSplitRounds
  // rounds of family a (a launch that long gains nothing from a finer split, and the bound
  // keeps the host loop short for any size the checks accept).
  constexpr int64_t kMaxSplitRounds = 4096;
  for (const Family& fa : families) {
    const int64_t ra = (N + fa.rows - 1) / fa.rows;
    for (const Family& fb : families) {
      if (fb.rows == fa.rows) continue;
      const int64_t rb = (N + fb.rows - 1) / fb.rows;
      for (int64_t k = 1; k <= kMaxSplitRounds && k * cus < (int64_t)S * ra; ++k) {
        const int64_t n1 = k * cus / ra;
        if (n1 <= 0 || n1 >= S) continue;
        const int64_t est = rounds(n1 * ra) * fa.cost + rounds((S - n1) * rb) * fb.cost;
        if (est < best_est) {
          best_est = est;
          best = K1Plan{fa.tile, fb.tile, (int)n1};
        }
      }
    }
  }
  if (est_out) *est_out = best_est;
  return best;
}

// Order of a K1 launch's tiles. The blocks are dealt to the 8 XCDs in contiguous runs, and the
// concurrent tiles of an XCD (cus / 8 of them) share what they read through its L2: in the
// slab-major order about c / RT W slabs and all RT X row tiles per round of c tiles, blocked
// into groups of 4 row tiles, c / 4 slabs and 4 row tiles. Per round an XCD then reads about
// c / RT + RT or c / 4 + 4 slabs' and row tiles' worth of data from beyond its L2; the blocked
// order is taken where it reads less (at 256 CUs: more than 8 row tiles). Measured at 3048
// rows (12 row tiles): K1 1.3-1.6% faster, with blocks of 8 slabs x 4 row tiles.
void tile_blocking(int RT, int cus, int* blk_slabs, int* blk_rows) {
  constexpr int kRows = 4;
  const int c = std::max(1, cus / 8);
  *blk_slabs = 0;
  *blk_rows = 0;
  if (RT > kRows && (double)c / RT + RT > (double)c / kRows + kRows) {
    *blk_slabs = std::max(1, c / kRows);
    *blk_rows = kRows;
  }
}

// ---- The cut of the vocabulary up to 64 rows, where K1 streams W once and nothing else counts.
// 256-id slabs leave the chip short of work when there are few of them, and a short last round
// when they do not divide among the CUs: V = 32000 gave 125 workgroups, V = 151936 two rounds of
// which the second held 82. So the slabs are made as wide as an equal share of a CU's ids (one or
// two workgroups per CU, every CU the same bytes) while that fits a tile, and beyond it 128-id
// slabs fill whole rounds of two workgroups per CU and 64-id slabs share out the rest. Whole
// verify steps at 60 rows and H = 4096, before -> after, packed weight (the floor is a 7.2 TB/s
// read): V = 24000 80 -> 42 us (27), 32000 81 -> 48 (36), 40000 89 -> 58 (46), 64000 92 -> 83
// (73), 80000 118 -> 102 (91), 140000 220 -> 176 (159), 151936 223 -> 196 (173), 200000 260 -> 250
// (228); 100000 and 128256 are level.
enum class Stream64 {
  kDeep128,    // <= 128 ids, three slots, two workgroups per CU; the tail on 64 ids, four slots
  kSpread256,  // <= 256 ids, one workgroup per CU, three-slot spread loop
  kWide256,    // <= 256 ids, two slots, two workgroups per CU
};

// <ids, rows, waves along ids, waves along rows, ring depth, K loop, non-temporal W copies>
using Deep128 = TileFamily<128, 64, 4, 1, 3, 0, true>;
using Deep64 = TileFamily<64, 64, 4, 1, 4, 0, true>;
using Spread256 = TileFamily<256, 64, 2, 2, 3, 3, true>;
using Wide256 = TileFamily<256, 64, 4, 1, 2, 0, true>;

struct Cut64 {
  Stream64 kind;
  SlabCut cut;
  int S;         // slabs in all = records per row
  bool tail64;   // the tail's slabs hold at most 64 ids: they run on the 64-id tile
};

// Narrower slabs than this cost more in X copies and records than they share out.
constexpr int kMinCut = 32;
// Vocabularies beyond this keep 256-id slabs: at two workgroups per CU their last round is a
// small part of the launch, and their records stay as few as they were.
constexpr int kMaxCutVocab = 1 << 18;

// Most slabs of the cut up to 64 rows: one per 64 ids, but up to 256 of them one per 32. It grows
// with V, and from 16384 ids on the draft head needs no more workspace than 64-id slabs do.
int max_records64(int V) {
  return std::max((V + 63) / 64, std::min((V + kMinCut - 1) / kMinCut, 256));
}

Cut64 cut_rows64(int V, int cus) {
  // ids per slab when n slabs share `ids`, in whole groups of 8
  auto share = [](int ids, int n) { return std::max(kMinCut, ((ids + n - 1) / n + 7) / 8 * 8); };
  auto even = [&](Stream64 kind, int width) {
    const int S = (V + width - 1) / width;
    return Cut64{kind, SlabCut{S, width, width, 0, 0}, S, false};
  };
  auto bounded = [&](const Cut64& c) {
    return c.S <= max_records64(V) ? c : even(Stream64::kWide256, kSlab);
  };
  if (V > kMaxCutVocab) return even(Stream64::kWide256, kSlab);
  const int one = share(V, cus), two = share(V, 2 * cus);
  if (one <= 128) return bounded(even(Stream64::kDeep128, one));
  // one workgroup per CU is 4-7% ahead of two half as wide at 150-200 ids (V = 40000: 57 against
  // 62 us, 50000: 68-70 against 71-73) and 2% behind at 250 (V = 64000: 85 against 83)
  if (one <= 224) return even(Stream64::kSpread256, one);
  if (two <= 128) return bounded(even(Stream64::kDeep128, two));
  if (two <= 256) return even(Stream64::kWide256, two);
  const int n1 = V / (2 * cus * 128) * 2 * cus, rest = V - n1 * 128;
  const bool tail64 = rest <= 2 * cus * 64;
  const int tw = tail64 ? 64 : share(rest, 2 * cus);
  return bounded(
      Cut64{Stream64::kDeep128, SlabCut{n1, 128, tw, 0, 0}, n1 + (rest + tw - 1) / tw, tail64});
}

// ---- The cut of the vocabulary from 65 to 512 rows. A last round that 256-id slabs leave partly
// empty costs as much as a full one, and the plan's second family (more row tiles on the remaining
// slabs) a second launch and another pass over those slabs. Here the slabs fill whole rounds of
// one family, and the ids that remain are shared equally among the CUs, one narrower tile each, in
// the same launch. Behind two rounds and more the tail's slabs stay 256 ids wide, on 64-row tiles:
// the records, and with them row_lse, are then the plan's bit for bit. That costs time at 65 to 128
// rows: narrower tails there took K1 from 205-211 to 189-195 us (100 and 128 rows, V = 140000, after
// a read of 1 GiB), 1-7% less at 150 to 256 rows. The tail copies with the non-temporal hint,
// although its two to eight row tiles read each W slab through an XCD's L2. Without it: 190 rows at
// V = 151936 with the policy, on changing inputs, 257.5 -> 260.5 us; K1 alone 249 -> 244 us after a
// read of 1 GiB (0-2% less at 65 to 256 rows) and 252 -> 266 after a fill of it, whose dirty lines
// the copies without the hint push out; back-to-back steps 265 -> 247.
// Whole verify steps at H = 4096, packed weight, before -> after: 120 rows at
// V = 32000 68 -> 54 us, 73728 139 -> 120, 147456 222 -> 213; 190 rows at 32000 71 -> 61, 81920
// 149 -> 134, 147456 242 -> 233; 250 rows at 40960 95 -> 85, 98304 179 -> 176; 378 rows at 36864
// 122 -> 119; 500 rows at 40960 157 -> 151.
struct CutWide {
  int rows = 0;    // tree rows of a tile; 0: the plan's whole slabs are no worse
  int tail_ids, tail_rows;    // ids and tree rows of the tail's tiles
  SlabCut cut;
  int S;           // slabs in all = records per row
};

constexpr int kMaxCutRows = 512;
constexpr int kRows64Cost = 44;     // a round of 256 ids x 64 rows behind others, in the plan's units
constexpr int kMaxCutTail = 256;    // most slabs of a tail (the workspace holds as many records)

CutWide cut_wide(int N, int V, int cus, int64_t plan_est) {
  CutWide best;
  if (N <= 64 || N > kMaxCutRows || V > kMaxCutVocab) return best;
  struct Tail { int ids, cost; };
  struct Family { int rows, cost; Tail tails[3]; };
  // one round of tails in the plan's units; measured at 120, 190 and 250 rows after one and two
  // rounds: 30-34, 38-46 and 52-60 us (128 rows), 32-41, 50-55 and 70-71, 42-52, 57-64 and 85-87
  const Family families[3] = {{128, 62, {{64, 30}, {128, 44}, {192, 60}}},
                              {192, 80, {{64, 36}, {128, 54}, {192, 70}}},
                              {256, 98, {{64, 44}, {192, 90}, {0, 0}}}};    // its 128-id tail never wins
  int64_t best_est = plan_est;
  for (const Family& f : families) {
    const int RT = (N + f.rows - 1) / f.rows, per_round = cus / RT;    // slabs of one round
    if (RT > 2 || per_round < 1) continue;
    const int rounds = V / (kSlab * per_round), n_main = rounds * per_round;
    const int rest = V - n_main * kSlab;
    for (const Tail& t : f.tails) {
      const int width = std::max(kMinCut, ((rest + per_round - 1) / per_round + 7) / 8 * 8);
      const int n_tail = (rest + width - 1) / width;
      int64_t est = (int64_t)rounds * f.cost + t.cost;
      // two row tiles: level with the plan where the estimates are within 6% (378 rows at
      // V = 49152 136 against 134 us, 500 rows at 81920 275 against 265). Where the plan is three
      // 128-row tiles and the weight stays in the last-level cache, back-to-back steps are up to 12%
      // slower (300 rows, V = 40960, H = 2560 82 against 93 us); after a read of 1 GiB, as a target
      // forward leaves the cache, K1 is 1-9% faster (there 77 against 75 us)
      if (RT == 2) est = est * 53 / 50;
      if (rounds > 1 || rest == 0 || width > t.ids || n_tail > kMaxCutTail || est >= best_est)
        continue;
      best_est = est;
      best.rows = best.tail_rows = f.rows;
      best.tail_ids = t.ids;
      best.cut = SlabCut{n_main, kSlab, width, 0, 0};
      best.S = n_main + n_tail;
    }
    const int slabs = (rest + kSlab - 1) / kSlab, tail_RT = (N + 63) / 64;
    const int64_t est = (int64_t)rounds * f.cost +
                        ((int64_t)slabs * tail_RT + cus - 1) / cus * kRows64Cost;
    if (rounds > 1 && rest > 0 && est < best_est) {
      best_est = est;
      best.rows = f.rows;
      best.tail_rows = 64;
      best.tail_ids = kSlab;
      best.cut = SlabCut{n_main, kSlab, kSlab, 0, 0};
      best.S = n_main + slabs;
    }
  }
  return best;
}

// Most records that a step of up to N rows writes, whatever the device's CU count: the largest of
// what the three ranges of rows may write, so that it never falls as N or V grow and a workspace
// sized for the largest batch serves every smaller one.
size_t max_records(int N, int V) {
  const size_t whole = (V + kSlab - 1) / kSlab;
  const int cut_V = std::min(V, kMaxCutVocab);       // no cut beyond it
  size_t n = std::max((size_t)N * whole, (size_t)std::min(N, 64) * max_records64(cut_V));
  if (N > 64)
    n = std::max(n, (size_t)std::min(N, kMaxCutRows) *
                        ((cut_V + kSlab - 1) / kSlab + kMaxCutTail));
  return n;
}

// The plan's launches of at most this many row tiles copy W with the non-temporal hint (the one or
// two tiles of a slab read it about once); more row tiles share each W slab through an XCD's L2
// and keep the default policy. Against the earlier rule (the hint for tiles of up to 128 rows)
// in same-box A/Bs: 260, 300, 378 and 450 rows 3% faster, 150 rows 1.4%, 500 rows 1%; 128,
// 200 and 600 to 3048 rows level. The cuts always copy with the hint.
constexpr int kStreamWMaxRowTiles = 2;

int tile_rows_of(Tile t) {
  switch (t) {
    case Tile::kRows64: return 64;
    case Tile::kRows128: return 128;
    case Tile::kRows192: return 192;
    default: return 256;
  }
}

// The K1 launches of the plan over N rows and S whole slabs on `cus` CUs, one or two, each with its
// K loop, W copy policy and tile order. Returns the count.
int k1_launches(int N, int S, int cus, const K1Plan& plan, asv_k1_launch out[2]) {
  int n = 0;
  auto add = [&](Tile t, int slab0, int n_slabs) {
    asv_k1_launch& k = out[n++];
    k.tile_rows = tile_rows_of(t);
    k.slab0 = slab0;
    k.n_slabs = n_slabs;
    k.row_tiles = (N + k.tile_rows - 1) / k.tile_rows;
    switch (t) {
      case Tile::kRows64: k.k_loop = 0; break;
      case Tile::kRows128: k.k_loop = 3; break;
      default: k.k_loop = 2; break;
    }
    k.stream_w = k.row_tiles <= kStreamWMaxRowTiles ? 1 : 0;
    tile_blocking(k.row_tiles, cus, &k.blk_slabs, &k.blk_rows);
  };
  add(plan.a, 0, plan.n1);
  if (plan.n1 < S) add(plan.b, plan.n1, S - plan.n1);
  return n;
}

// The tile that asv_tuning.tile_rows asks for; false for a value that names no tile.
bool forced_tile(int rows, Tile* t) {
  switch (rows) {
    case 64: *t = Tile::kRows64; return true;
    case 128: *t = Tile::kRows128; return true;
    case 192: *t = Tile::kRows192; return true;
    case 256: *t = Tile::kRows256; return true;
    default: return false;
  }
}

// What K1 runs in a step of N rows: one launch over a cut of the vocabulary up to 64 rows (cut64)
// or, up to 512, where it is estimated to be faster (wide); else the plan's launches.
struct K1Step {
  asv_k1_launch plan[2];
  int n_plan;
  bool rows64;
  Cut64 cut64;
  CutWide wide;
  int S;           // records per row
};

// tile: the forced one, or null for the library's choice.
K1Step k1_step(int N, int V, int cus, const Tile* tile) {
  K1Step st{};
  st.S = (V + kSlab - 1) / kSlab;
  int64_t est = 0;           // no cut beyond 64 rows where the tile is forced
  const K1Plan plan = tile ? K1Plan{*tile, *tile, st.S} : plan_k1(N, st.S, cus, &est);
  st.n_plan = k1_launches(N, st.S, cus, plan, st.plan);
  st.rows64 = N <= 64 && plan.a == Tile::kRows64;
  if (st.rows64) {
    st.cut64 = cut_rows64(V, cus);
    st.S = st.cut64.S;
  } else {
    st.wide = cut_wide(N, V, cus, est);
    if (st.wide.rows) st.S = st.wide.S;
  }
  return st;
}

int tile_ids_of(Stream64 kind) { return kind == Stream64::kDeep128 ? 128 : kSlab; }

// A cut as asv_lmhead_cut describes it.
asv_lmhead_cut describe(const SlabCut& c, int S, int ids, int rows, int tail_ids, int tail_rows) {
  asv_lmhead_cut r{};
  r.records = S;
  if (c.n_main > 0) {
    r.main_slabs = c.n_main;
    r.main_ids = c.width;
    r.main_tile_ids = ids;
    r.main_tile_rows = rows;
  }
  if (S > c.n_main) {
    r.tail_slabs = S - c.n_main;
    r.tail_ids = c.tail_width;
    r.tail_tile_ids = tail_ids;
    r.tail_tile_rows = tail_rows;
  }
  return r;
}
asv_lmhead_cut describe(const Cut64& c, int ids, int rows) {
  return describe(c.cut, c.S, ids, rows, c.tail64 ? 64 : ids, rows);
}

struct Layout {
  int S = 0;       // vocabulary slabs of the plan
  int n_conf = 0;  // draft-confidence chunks per request
  size_t off_rec_m = 0, off_rec_s = 0, off_rec_a = 0, off_conf_m = 0, off_conf_s = 0;
  size_t off_cnt = 0;  // B + 1 ints: per-request completion counters, then the bad-offsets flag
  size_t bytes = 0;
};

Layout layout(int B, int N, int V) {
  Layout L;
  L.S = (V + kSlab - 1) / kSlab;
  L.n_conf = (V + kConfChunk - 1) / kConfChunk;
  const size_t rec = max_records(N, V) * 4;
  const size_t conf = (size_t)B * L.n_conf * 4;
  size_t at = 0;
  L.off_rec_m = at;  at += align_up(rec);
  L.off_rec_s = at;  at += align_up(rec);
  L.off_rec_a = at;  at += align_up(rec);
  L.off_conf_m = at; at += align_up(conf);
  L.off_conf_s = at; at += align_up(conf);
  L.off_cnt = at;    at += align_up((size_t)(B + 1) * 4);
  L.bytes = at;
  return L;
}

// Row and vocabulary indices (rounded up to whole tiles) and the LM-head kernel's workgroup
// count stay ints: N, V < 2^30, and for the 64-row tile, which has the most workgroups,
// ceil(V / 256) * ceil(N / 64) < 2^31.
bool grid_ok(int N, int V) {
  if (N >= (1 << 30) || V >= (1 << 30)) return false;
  const int64_t S = ((int64_t)V + kSlab - 1) / kSlab, RT = ((int64_t)N + 63) / 64;
  return S * RT < ((int64_t)1 << 31);
}

bool sizes_ok(int B, int N, int H, int V) {
  if (B < 0 || N < 0 || H <= 0 || V <= 0) return false;
  if ((B == 0) != (N == 0) || N < B) return false;
  if (H % kKAlign != 0 || H > (1 << 20)) return false;
  return grid_ok(N, V);
}

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

bool params_ok(const asv_params& p) {
  if (!(p.alpha > 0.f && p.alpha <= 1.f) || p.breaker_n < 1 || p.max_promotions < -1)
    return false;
  if (!(p.dcs_divisor > 0.f && p.dcs_divisor < __builtin_inff())) return false;
  if (!(p.temperature > 0.f && p.temperature < __builtin_inff())) return false;
  for (int k = 0; k < 3; ++k)
    if (p.shape_lo[k] < 1 || p.shape_hi[k] < 1 || p.shape_start[k] < 1) return false;
  return true;
}

// Launches `kernel` on `s`; with a start or stop event (measurement only) through
// hipExtLaunchKernelGGL, which sets the events to the dispatch's own start and end times.
template <typename F, typename... Args>
void launch_timed(F kernel, int grid, int threads, hipStream_t s, hipEvent_t start,
                  hipEvent_t stop, Args... args) {
  if (start || stop)
    hipExtLaunchKernelGGL(kernel, dim3(grid), dim3(threads), 0, s, start, stop, 0, args...);
  else
    kernel<<<grid, threads, 0, s>>>(args...);
}

LmheadArgs lmhead_args(const asv_verify_args* a, const Layout& L, char* ws, int S) {
  LmheadArgs r;
  r.X = a->hidden;
  r.W = a->w_lm;
  r.parent = a->parent;
  r.draft_tok = a->draft_tok;
  r.req_offsets = a->req_offsets;
  r.B = a->B;
  r.N = a->N;
  r.H = a->H;
  r.V = a->V;
  r.S = S;
  r.rec_m = reinterpret_cast<float*>(ws + L.off_rec_m);
  r.rec_s = reinterpret_cast<float*>(ws + L.off_rec_s);
  r.rec_a = reinterpret_cast<int32_t*>(ws + L.off_rec_a);
  r.drafted_logit = a->drafted_logit;
  r.done_cnt = reinterpret_cast<int32_t*>(ws + L.off_cnt);
  r.n_cnt = a->B + 1;
  r.w_packed = a->w_lm_layout == ASV_W_PACKED ? kPackRowsTarget : 0;
  return r;
}

struct K1Events {
  hipEvent_t start, stop;
};

// The main slabs of `cut` x k.row_tiles on family M and its tail's n_tail tiles on family T.
template <class M, class T = M>
void launch_lmhead(const LmheadArgs& g, const SlabCut& cut, int n_tail, const asv_k1_launch& k,
                   hipStream_t s, const K1Events& ev) {
  static_assert(M::BK == kPackDepth, "a stage is one packed column block");
  launch_timed(k_lmhead_partial<M, T>, cut.n_main * k.row_tiles + n_tail, M::C::kThreads, s,
               ev.start, ev.stop, g, cut, k.row_tiles, k.blk_slabs, k.blk_rows);
}

// One launch of the plan over whole 256-id slabs.
template <int TR, int WV, int WR, int NST, int LOOP>
void launch_slabs(const LmheadArgs& g, const asv_k1_launch& k, hipStream_t s,
                  const K1Events& ev) {
  const SlabCut cut{k.n_slabs, kSlab, kSlab, k.slab0, k.slab0 * kSlab};
  if (k.stream_w)
    launch_lmhead<TileFamily<kSlab, TR, WV, WR, NST, LOOP, true>>(g, cut, 0, k, s, ev);
  else
    launch_lmhead<TileFamily<kSlab, TR, WV, WR, NST, LOOP, false>>(g, cut, 0, k, s, ev);
}

// Up to 64 rows: one launch over the slabs of cut_rows64.
void launch_rows64(const LmheadArgs& g, const Cut64& c, const asv_k1_launch& k, hipStream_t s,
                   const K1Events& ev) {
  const int n_tail = c.S - c.cut.n_main;
  switch (c.kind) {
    case Stream64::kDeep128:
      if (c.tail64)
        launch_lmhead<Deep128, Deep64>(g, c.cut, n_tail, k, s, ev);
      else
        launch_lmhead<Deep128>(g, c.cut, n_tail, k, s, ev);
      break;
    case Stream64::kSpread256:
      launch_lmhead<Spread256>(g, c.cut, n_tail, k, s, ev);
      break;
    case Stream64::kWide256:
      launch_lmhead<Wide256>(g, c.cut, n_tail, k, s, ev);
      break;
  }
}

// The slabs of cut_wide: one launch of the family's 256-id tile, its tail on a narrower one (alone,
// where the vocabulary holds no whole round).
template <int TR, int NST, int TAIL_IDS, int TAIL_NST>
void launch_cut(const LmheadArgs& g, const CutWide& c, hipStream_t s, const K1Events& ev) {
  using M = TileFamily<kSlab, TR, 2, 2, NST, NST, true>;
  using T = TileFamily<TAIL_IDS, TR, 2, 2, TAIL_NST, TAIL_NST, true>;
  asv_k1_launch k{};
  k.row_tiles = (g.N + TR - 1) / TR;
  const int n_tail = (c.S - c.cut.n_main) * k.row_tiles;
  if (c.cut.n_main > 0)
    launch_lmhead<M, T>(g, c.cut, n_tail, k, s, ev);
  else
    launch_lmhead<T>(g, SlabCut{0, kSlab, c.cut.tail_width, 0, 0}, n_tail, k, s, ev);
}

template <int TR, int NST>
void launch_cut_rows(const LmheadArgs& g, const CutWide& c, hipStream_t s, const K1Events& ev) {
  if (c.tail_rows == 64) {
    using M = TileFamily<kSlab, TR, 2, 2, NST, NST, true>;
    asv_k1_launch k{};
    k.row_tiles = (g.N + TR - 1) / TR;
    launch_lmhead<M, Spread256>(g, c.cut, (c.S - c.cut.n_main) * ((g.N + 63) / 64), k, s, ev);
    return;
  }
  switch (c.tail_ids) {
    case 64: launch_cut<TR, NST, 64, 3>(g, c, s, ev); break;
    case 128:
      if constexpr (TR != 256) launch_cut<TR, NST, 128, 3>(g, c, s, ev);
      break;
    // three slots of 192 ids and 256 rows are 168 KB
    default: launch_cut<TR, NST, 192, TR == 256 ? 2 : 3>(g, c, s, ev); break;
  }
}

// Total bytes of the packed copy of a [V][H] weight whose K blocks hold V rounded up to
// `align` rows; false for sizes the LM-head kernels reject and for copies of 4 GiB or more,
// past the 32-bit offsets they use in it.
bool packed_size(int V, int H, int align, uint64_t* bytes) {
  if (V <= 0 || H <= 0 || H % kPackDepth != 0 || H > (1 << 20)) return false;
  const uint64_t Vp = ((uint64_t)V + align - 1) / align * align;
  const uint64_t total = Vp * (uint64_t)H * 2;
  if (total >= ((uint64_t)1 << 32)) return false;
  *bytes = total;
  return true;
}

// Pack w into tiles of PR rows (k_pack_tiles), after the checks both pack entry points share.
template <int PR>
int pack_tiles(const uint16_t* w, int V, int H, uint16_t* packed, uint64_t packed_bytes,
               void* stream) {
  constexpr int kAlign = PR > 128 ? PR : 128;
  uint64_t need = 0;
  if (!packed_size(V, H, kAlign, &need) || !w || !packed || !aligned16(w) ||
      !aligned16(packed) || packed_bytes < need)
    return ASV_EINVAL;
  const uintptr_t w0 = reinterpret_cast<uintptr_t>(w), p0 = reinterpret_cast<uintptr_t>(packed);
  if (w0 < p0 + need && p0 < w0 + (uint64_t)V * H * 2) return ASV_EINVAL;   // overlap
  (void)hipGetLastError();
  const int T = (int)((need / 2 / H) / PR);        // tiles per 64-column block
  const int tiles = T * (H / kPackDepth);
  k_pack_tiles<PR><<<tiles, kPackThreads, 0, reinterpret_cast<hipStream_t>(stream)>>>(
      reinterpret_cast<const uint4*>(w), reinterpret_cast<uint4*>(packed), V, H, T);
  return launch_status("k_pack_tiles");
}

AcceptArgs accept_args(const asv_verify_args* a, const Layout& L, char* ws, bool conf) {
  AcceptArgs r;
  r.B = a->B;
  r.N = a->N;
  r.V = a->V;
  r.off = a->req_offsets;
  r.parent = a->parent;
  r.tok = a->draft_tok;
  r.tau = a->tau;
  r.row_max = a->row_max;
  r.row_arg = a->row_argmax;
  r.g = a->drafted_logit;
  r.accept = a->accept;
  r.acc_len = a->accepted_len;
  r.bonus = a->bonus_token;
  r.path = a->accepted_path;
  r.conf_m = reinterpret_cast<const float*>(ws + L.off_conf_m);
  r.conf_s = reinterpret_cast<const float*>(ws + L.off_conf_s);
  r.n_conf = conf ? L.n_conf : 0;
  r.draft_conf = a->draft_conf;
  r.state = a->state;
  r.status = a->req_status;
  r.prm = a->params;
  return r;
}

// ---- draft side

// The draft LM head (K5) by draft rows R = 4B. Up to 64 rows it streams its weight like K1 and
// runs K1's cut and tiles (cut_rows64), except where the vocabulary leaves each CU one slab of 64
// ids: those run on a 64-id tile of 32 or 64 rows, which holds nothing that it doesn't read and
// fills its ring three stages ahead instead of two. Beyond, one workgroup per CU: an equal share of
// the ids where that fits a tile of 128, 192 or 256 ids (128 rows) or 128 ids (256 rows), else the
// rounds of the cheapest of these tiles.
enum class DraftTile {
  kRows32x64, kRows64x64, kRows64, kRows128x128, kRows128x192, kRows128x256, kRows256x128
};

struct DraftPlan {
  DraftTile tile;
  Cut64 cut;       // kRows64: all of it; else cut.cut and cut.S
  int row_tiles;
};

DraftPlan plan_draft(int R, int V, int cus) {
  auto slabs = [&](DraftTile tile, int width, int row_tiles) {
    const int S = (V + width - 1) / width;
    return DraftPlan{tile, Cut64{Stream64::kDeep128, SlabCut{S, width, width, 0, 0}, S, false},
                     row_tiles};
  };
  if (R <= 64) {
    // Whole draft steps at H = 4096, K1's cut against the 64-id tile: V = 16384 36.2 against 27.4 us
    // at 1 request, 39.2 against 30.8 at 16. Past one slab per CU some CUs run two: from 16640 ids
    // on 39.3 against 46.7 us at 16 requests, 36.4 against 37.5 at 4, but 36.5 against 35.1 at 1
    // and 36.3 against 35.9 at 2; 22000 ids are level there.
    if (V <= (int64_t)cus * (R <= 8 ? 80 : 64))
      return slabs(R <= 32 ? DraftTile::kRows32x64 : DraftTile::kRows64x64, 64, 1);
    return DraftPlan{DraftTile::kRows64, cut_rows64(V, cus), 1};
  }
  struct Family { DraftTile tile; int ids, rows, cost; };
  // cost of one round of tiles, in us at H = 4096 (MI355X)
  const Family families[4] = {{DraftTile::kRows128x128, 128, 128, 46},
                              {DraftTile::kRows128x192, 192, 128, 59},
                              {DraftTile::kRows128x256, 256, 128, 79},
                              {DraftTile::kRows256x128, 128, 256, 59}};
  DraftPlan best{};
  int64_t best_est = INT64_MAX;
  for (const Family& f : families) {
    const int RT = (R + f.rows - 1) / f.rows;
    const int64_t tiles = ((int64_t)V + f.ids - 1) / f.ids * RT, rounds = (tiles + cus - 1) / cus;
    const int64_t est = rounds * f.cost;
    if (est >= best_est) continue;
    best_est = est;
    // the slabs one round's row tiles leave room for, ids shared equally
    const int64_t n = std::max<int64_t>(1, rounds * cus / RT);
    const int width = (int)std::min<int64_t>(
        f.ids, std::max<int64_t>(128, ((V + n - 1) / n + 7) / 8 * 8));
    best = slabs(f.tile, width, RT);
  }
  return best;
}

struct DraftLayout {
  size_t off_k = 0, off_s = 0, bytes = 0;
};

// Most records that a draft step of up to R rows writes, whatever the device's CU count: never
// falling as R or V grow (see max_records).
size_t max_draft_records(int R, int V) {
  const size_t n = (size_t)std::min(R, 64) * max_records64(V);
  return R <= 64 ? n : std::max(n, (size_t)R * ((V + 127) / 128));
}

DraftLayout draft_layout(int B, int V) {
  DraftLayout L;
  const int R = B * kTopK;
  const size_t rec = max_draft_records(R, V);
  size_t at = 0;
  L.off_k = at; at += align_up(rec * kTopK * 8);
  L.off_s = at; at += align_up(rec * 4);
  L.bytes = at;
  return L;
}

bool draft_sizes_ok(int B, int H, int V) {
  if (B < 0 || H <= 0 || V < kTopK || V >= (1 << 30)) return false;
  if (H % kKAlign != 0 || H > (1 << 20)) return false;
  // 32-bit offsets inside a tile's buffer resource: all 4B rows of X and one slab of W
  if ((int64_t)B * kTopK * H * 2 >= (int64_t)1 << 31) return false;
  // the draft LM head's workgroup count stays an int: at most ceil(V / 64) slabs up to 64 rows
  // (or one per CU of a small V), ceil(V / 128) slabs of 128-row tiles beyond
  const int64_t R = (int64_t)B * kTopK, ids = R <= 64 ? 64 : 128;
  const int64_t row_tiles = R <= 64 ? 1 : (R + 127) / 128;
  return (V + ids - 1) / ids * row_tiles < ((int64_t)1 << 31);
}

template <class M, class T = M>
void launch_draft(const asv_draft_args* a, const DraftLayout& L, char* ws, const DraftPlan& p,
                  hipStream_t s, const K1Events& ev) {
  static_assert(M::BK == kPackDepth, "a stage is one packed column block");
  DraftArgs g;
  g.X = a->hidden;
  g.W = a->w_draft;
  g.R = a->B * kTopK;
  g.H = a->H;
  g.V = a->V;
  g.S = p.cut.S;
  g.rec_k = reinterpret_cast<uint64_t*>(ws + L.off_k);
  g.rec_s = reinterpret_cast<float*>(ws + L.off_s);
  g.w_packed = a->w_draft_layout == ASV_W_PACKED ? 128 : 0;
  const int n_main = p.cut.cut.n_main;
  launch_timed(k_draft_partial<M, T>, n_main * p.row_tiles + p.cut.S - n_main, M::C::kThreads, s,
               ev.start, ev.stop, g, p.cut.cut, p.row_tiles);
}

// ---- static scratch of asv_verify_noalloc

// The workspace of asv_verify_noalloc. In host code `scratch` names a host-side stand-in, not
// the device array: the device address comes from hipGetSymbolAddress, once per device (each
// GPU holds its own copy at its own address).
__device__ __align__(256) char scratch[ASV_STATIC_SCRATCH_BYTES];

constexpr int kMaxDevices = 64;

// Device address of `scratch` on the current device, or nullptr (error recorded).
void* scratch_address() {
  static std::mutex mu;
  static void* addr[kMaxDevices] = {};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) {
    set_error("hipGetDevice", e);
    return nullptr;
  }
  if (dev < 0 || dev >= kMaxDevices) {
    set_error("asv_verify_noalloc: device ordinal out of range", hipErrorInvalidDevice);
    return nullptr;
  }
  std::lock_guard<std::mutex> lock(mu);
  if (!addr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p) {
      set_error("hipGetSymbolAddress(scratch)", e != hipSuccess ? e : hipErrorInvalidSymbol);
      return nullptr;
    }
    addr[dev] = p;
  }
  return addr[dev];
}

}  // namespace
}  // namespace asv

using namespace asv;

extern "C" int asv_version(void) { return ASV_VERSION; }

extern "C" const char* asv_last_error(void) { return g_last_error; }

extern "C" const char* asv_status_string(int code) {
  switch (code) {
    case ASV_OK: return "ok";
    case ASV_EINVAL: return "invalid argument (size, null or misaligned pointer, parameter)";
    case ASV_EWORKSPACE: return "workspace too small or not 256-byte aligned";
    case ASV_EHIP: return "HIP runtime error or kernel launch failure";
    case ASV_ESCRATCH:
      return "the sizes need more workspace than the static scratch of asv_verify_noalloc";
    default: return "unknown asv status code";
  }
}

extern "C" int asv_workspace_bytes(int32_t B, int32_t N, int32_t H, int32_t V,
                                   uint64_t* bytes) {
  if (!bytes || !sizes_ok(B, N, H, V)) return ASV_EINVAL;
  *bytes = layout(B, N, V).bytes;
  return ASV_OK;
}

extern "C" int asv_state_init(asv_req_state* state, int32_t B, const asv_params* p,
                              void* stream) {
  if (B < 0 || !p || (B > 0 && !state) || !params_ok(*p)) return ASV_EINVAL;
  if (B == 0) return ASV_OK;
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  (void)hipGetLastError();
  k_state_init<<<(B + 255) / 256, 256, 0, s>>>(state, B, *p);
  return launch_status("k_state_init");
}

extern "C" int asv_tree_policy(const float* conf, asv_req_state* state, int32_t B,
                               const asv_params* p, void* stream) {
  if (B < 0 || !p || (B > 0 && !state) || !params_ok(*p)) return ASV_EINVAL;
  if (B == 0) return ASV_OK;
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  (void)hipGetLastError();
  k_tree_policy<<<(B + 255) / 256, 256, 0, s>>>(conf, state, B, *p);
  return launch_status("k_tree_policy");
}

extern "C" int asv_verify_tuned(const asv_verify_args* a, const asv_tuning* tuning,
                                void* workspace, uint64_t workspace_bytes, void* stream) {
  if (!a || !sizes_ok(a->B, a->N, a->H, a->V)) return ASV_EINVAL;
  const asv_tuning tu = tuning ? *tuning : asv_tuning{nullptr, nullptr, 0};
  Tile forced = Tile::kRows64;
  if (tu.tile_rows != 0 && !forced_tile(tu.tile_rows, &forced)) return ASV_EINVAL;
  if (a->w_lm_layout != ASV_W_ROW_MAJOR && a->w_lm_layout != ASV_W_PACKED) return ASV_EINVAL;
  uint64_t packed_bytes = 0;
  if (a->w_lm_layout == ASV_W_PACKED &&
      !packed_size(a->V, a->H, kPackRowsTarget, &packed_bytes))
    return ASV_EINVAL;
  if (a->B == 0) return ASV_OK;
  if (!a->hidden || !a->w_lm || !a->draft_tok || !a->parent || !a->req_offsets || !a->tau ||
      !a->row_max || !a->row_lse || !a->row_argmax || !a->drafted_logit || !a->accept ||
      !a->accepted_len || !a->bonus_token || !a->accepted_path || !a->req_status)
    return ASV_EINVAL;
  if (!aligned16(a->hidden) || !aligned16(a->w_lm)) return ASV_EINVAL;
  if (!params_ok(a->params)) return ASV_EINVAL;
  const Layout L = layout(a->B, a->N, a->V);
  if (!workspace || workspace_bytes < L.bytes ||
      (reinterpret_cast<uintptr_t>(workspace) % kAlign) != 0)
    return ASV_EWORKSPACE;

  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  char* ws = static_cast<char*>(workspace);
  const bool conf = a->draft_logits != nullptr;
  (void)hipGetLastError();

  const K1Step step = k1_step(a->N, a->V, cu_count(), tu.tile_rows != 0 ? &forced : nullptr);
  const Cut64& cut64 = step.cut64;
  const CutWide& wide = step.wide;
  const bool rows64 = step.rows64;
  LmheadArgs g = lmhead_args(a, L, ws, step.S);
  // K4 only needs the inputs: up to 64 rows its shares go to K1's tiles, one each, which saves its
  // launch (8 rows at V = 128256, one request: 165.6 -> 162.9 us), where there are enough tiles
  g.conf = ConfArgs{a->N, a->V, a->req_offsets, a->draft_logits,
                    reinterpret_cast<float*>(ws + L.off_conf_m),
                    reinterpret_cast<float*>(ws + L.off_conf_s), L.n_conf, 0};
  const int64_t shares = conf ? (int64_t)conf_shares(L.n_conf) * a->B : 0;
  if (rows64 && shares <= cut64.S) {
    g.conf.n_shares = (int)shares;
  } else if (conf) {
    ConfArgs c = g.conf;
    c.n_shares = (int)std::min<int64_t>(shares, INT32_MAX);
    k_draft_conf_partial<<<dim3(conf_shares(L.n_conf), a->B), kConfWaves * kWave, 0, s>>>(c);
    if (int rc = launch_status("k_draft_conf_partial")) return rc;
  }
  // timing events (measurement only): the start of the first launch, the end of the last
  const hipEvent_t ev_begin = reinterpret_cast<hipEvent_t>(tu.begin_event);
  const hipEvent_t ev_end = reinterpret_cast<hipEvent_t>(tu.end_event);
  switch (wide.rows) {
    case 128: launch_cut_rows<128, 3>(g, wide, s, K1Events{ev_begin, ev_end}); break;
    case 192: launch_cut_rows<192, 2>(g, wide, s, K1Events{ev_begin, ev_end}); break;
    case 256: launch_cut_rows<256, 2>(g, wide, s, K1Events{ev_begin, ev_end}); break;
    default: break;
  }
  for (int q = 0; q < step.n_plan && !wide.rows; ++q) {
    const asv_k1_launch& k = step.plan[q];
    const K1Events ev{q == 0 ? ev_begin : nullptr, q == step.n_plan - 1 ? ev_end : nullptr};
    // <tree rows, waves along vocab, waves along rows, ring depth, K loop>, each the fastest of
    // a sweep on MI355X for its row range. The 128-, 192- and 256-row tiles run the spread K
    // loops (copies spaced between the MFMAs), in interleaved comparisons 28% faster than the
    // burst ring at 378 rows and 20% at 2048 and 3048 rows.
    switch (k.tile_rows) {
      case 64:
        if (rows64)
          launch_rows64(g, cut64, k, s, ev);
        else
          launch_slabs<64, 4, 1, 2, 0>(g, k, s, ev);
        break;
      case 128: launch_slabs<128, 2, 2, 3, 3>(g, k, s, ev); break;
      case 192: launch_slabs<192, 2, 2, 2, 2>(g, k, s, ev); break;
      default: launch_slabs<256, 2, 2, 2, 2>(g, k, s, ev); break;
    }
  }
  if (int rc = launch_status("k_lmhead_partial")) return rc;

  const AcceptArgs acc = accept_args(a, L, ws, conf);
  const float* rec_m = reinterpret_cast<const float*>(ws + L.off_rec_m);
  const float* rec_s = reinterpret_cast<const float*>(ws + L.off_rec_s);
  const int32_t* rec_a = reinterpret_cast<const int32_t*>(ws + L.off_rec_a);
  int32_t* cnt = reinterpret_cast<int32_t*>(ws + L.off_cnt);
  if (a->B <= kFusedMaxB) {
    k_merge_accept<<<(a->N + kFinishWaves - 1) / kFinishWaves, kFinishWaves * kWave, 0, s>>>(
        step.S, rec_m, rec_s, rec_a, a->row_max, a->row_lse, a->row_argmax, cnt, acc);
    return launch_status("k_merge_accept");
  }
  k_slab_merge<<<(a->N + kMergeRowsPerBlock - 1) / kMergeRowsPerBlock,
                 kMergeRowsPerBlock * kWave, 0, s>>>(
      a->N, step.S, rec_m, rec_s, rec_a, a->row_max, a->row_lse, a->row_argmax, a->B,
      a->req_offsets, cnt + a->B);
  if (int rc = launch_status("k_slab_merge")) return rc;
  k_tree_accept<<<a->B, kWave, 0, s>>>(cnt + a->B, acc);
  return launch_status("k_tree_accept");
}

// The step of asv_k1_plan and asv_k1_cut; ASV_EINVAL for sizes asv_verify would reject.
static int checked_step(int N, int V, int cus, int tile_rows, K1Step* step) {
  if (N < 1 || V < 1 || cus < 1 || !grid_ok(N, V)) return ASV_EINVAL;
  Tile forced = Tile::kRows64;
  if (tile_rows != 0 && !forced_tile(tile_rows, &forced)) return ASV_EINVAL;
  *step = k1_step(N, V, cus, tile_rows != 0 ? &forced : nullptr);
  return ASV_OK;
}

extern "C" int asv_k1_plan(int32_t N, int32_t V, int32_t cus, int32_t tile_rows,
                           asv_k1_launch* launches, int32_t* n_launches) {
  K1Step step;
  if (!launches || !n_launches) return ASV_EINVAL;
  if (int rc = checked_step(N, V, cus, tile_rows, &step)) return rc;
  for (int q = 0; q < step.n_plan; ++q) launches[q] = step.plan[q];
  *n_launches = step.n_plan;
  return ASV_OK;
}

extern "C" int asv_k1_cut(int32_t N, int32_t V, int32_t cus, int32_t tile_rows,
                          asv_lmhead_cut* cut) {
  K1Step step;
  if (!cut) return ASV_EINVAL;
  if (int rc = checked_step(N, V, cus, tile_rows, &step)) return rc;
  const CutWide& w = step.wide;
  *cut = step.rows64 ? describe(step.cut64, tile_ids_of(step.cut64.kind), 64)
         : w.rows    ? describe(w.cut, w.S, kSlab, w.rows, w.tail_ids, w.tail_rows)
                     : asv_lmhead_cut{};
  return ASV_OK;
}

extern "C" int asv_draft_cut(int32_t B, int32_t V, int32_t cus, asv_lmhead_cut* cut) {
  if (B < 1 || cus < 1 || !cut || !draft_sizes_ok(B, kKAlign, V)) return ASV_EINVAL;
  const DraftPlan p = plan_draft(B * kTopK, V, cus);
  switch (p.tile) {
    case DraftTile::kRows32x64: *cut = describe(p.cut, 64, 32); break;
    case DraftTile::kRows64x64: *cut = describe(p.cut, 64, 64); break;
    case DraftTile::kRows64: *cut = describe(p.cut, tile_ids_of(p.cut.kind), 64); break;
    case DraftTile::kRows128x128: *cut = describe(p.cut, 128, 128); break;
    case DraftTile::kRows128x192: *cut = describe(p.cut, 192, 128); break;
    case DraftTile::kRows128x256: *cut = describe(p.cut, 256, 128); break;
    case DraftTile::kRows256x128: *cut = describe(p.cut, 128, 256); break;
  }
  return ASV_OK;
}

extern "C" int asv_verify(const asv_verify_args* a, void* workspace, uint64_t workspace_bytes,
                          void* stream) {
  return asv_verify_tuned(a, nullptr, workspace, workspace_bytes, stream);
}

extern "C" int asv_verify_noalloc(const asv_verify_args* a, void* stream) {
  if (!a || !sizes_ok(a->B, a->N, a->H, a->V)) return ASV_EINVAL;
  if (a->B == 0) return asv_verify_tuned(a, nullptr, nullptr, 0, stream);
  const size_t need = layout(a->B, a->N, a->V).bytes;
  if (need > ASV_STATIC_SCRATCH_BYTES) {
    snprintf(g_last_error, sizeof(g_last_error),
             "asv_verify_noalloc: %zu workspace bytes needed, the static scratch holds %u",
             need, ASV_STATIC_SCRATCH_BYTES);
    return ASV_ESCRATCH;
  }
  void* ws = scratch_address();
  if (!ws) return ASV_EHIP;
  return asv_verify_tuned(a, nullptr, ws, ASV_STATIC_SCRATCH_BYTES, stream);
}

extern "C" int asv_packed_lm_head_bytes(int32_t V, int32_t H, uint64_t* bytes) {
  if (!bytes || !packed_size(V, H, kPackRowsTarget, bytes)) return ASV_EINVAL;
  return ASV_OK;
}

extern "C" int asv_pack_lm_head(const uint16_t* w, int32_t V, int32_t H, uint16_t* packed,
                                uint64_t packed_bytes, void* stream) {
  return pack_tiles<kPackRowsTarget>(w, V, H, packed, packed_bytes, stream);
}

extern "C" int asv_packed_draft_head_bytes(int32_t V, int32_t H, uint64_t* bytes) {
  if (!bytes || V < kTopK || !packed_size(V, H, 128, bytes)) return ASV_EINVAL;
  return ASV_OK;
}

extern "C" int asv_pack_draft_head(const uint16_t* w, int32_t V, int32_t H, uint16_t* packed,
                                   uint64_t packed_bytes, void* stream) {
  if (V < kTopK) return ASV_EINVAL;
  return pack_tiles<kPackRowsDraft>(w, V, H, packed, packed_bytes, stream);
}

extern "C" int asv_draft_workspace_bytes(int32_t B, int32_t H, int32_t V, uint64_t* bytes) {
  if (!bytes || !draft_sizes_ok(B, H, V)) return ASV_EINVAL;
  *bytes = draft_layout(B, V).bytes;
  return ASV_OK;
}

extern "C" int asv_draft_step_tuned(const asv_draft_args* a, const asv_tuning* tuning,
                                    void* workspace, uint64_t workspace_bytes, void* stream) {
  if (!a || !draft_sizes_ok(a->B, a->H, a->V) || a->step < 0) return ASV_EINVAL;
  const asv_tuning tu = tuning ? *tuning : asv_tuning{nullptr, nullptr, 0};
  if (tu.tile_rows != 0) return ASV_EINVAL;
  if (a->w_draft_layout != ASV_W_ROW_MAJOR && a->w_draft_layout != ASV_W_PACKED)
    return ASV_EINVAL;
  uint64_t packed_bytes = 0;
  if (a->w_draft_layout == ASV_W_PACKED && !packed_size(a->V, a->H, 128, &packed_bytes))
    return ASV_EINVAL;
  if (a->B == 0) return ASV_OK;
  if (!a->hidden || !a->w_draft || !a->tree || !a->topk_id || !a->topk_logp || !a->row_lse ||
      !a->front_tok)
    return ASV_EINVAL;
  if (!aligned16(a->hidden) || !aligned16(a->w_draft)) return ASV_EINVAL;
  if (!a->state && a->step == 0) {
    const int ns = a->shape[0], tk = a->shape[1], nd = a->shape[2];
    if (!(ns >= 1 && tk >= 1 && tk <= kTopK && nd >= 1 && ns <= kPoolMax &&
          tk + (ns - 1) * tk * tk <= kPoolMax))
      return ASV_EINVAL;
  }
  const DraftLayout L = draft_layout(a->B, a->V);
  if (!workspace || workspace_bytes < L.bytes ||
      (reinterpret_cast<uintptr_t>(workspace) % kAlign) != 0)
    return ASV_EWORKSPACE;
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  char* ws = static_cast<char*>(workspace);
  (void)hipGetLastError();
  // timing events (measurement only): the start and the end of the draft LM head's launch
  const K1Events ev{reinterpret_cast<hipEvent_t>(tu.begin_event),
                    reinterpret_cast<hipEvent_t>(tu.end_event)};
  const DraftPlan p = plan_draft(a->B * kTopK, a->V, cu_count());
  switch (p.tile) {
    case DraftTile::kRows32x64:
      launch_draft<TileFamily<64, 32, 2, 1, 4, 0, true, Mfma32>>(a, L, ws, p, s, ev);
      break;
    case DraftTile::kRows64x64:
      launch_draft<TileFamily<64, 64, 2, 2, 4, 0, true, Mfma32>>(a, L, ws, p, s, ev);
      break;
    case DraftTile::kRows64:
      switch (p.cut.kind) {
        case Stream64::kDeep128:
          if (p.cut.tail64)
            launch_draft<Deep128, Deep64>(a, L, ws, p, s, ev);
          else
            launch_draft<Deep128>(a, L, ws, p, s, ev);
          break;
        case Stream64::kSpread256: launch_draft<Spread256>(a, L, ws, p, s, ev); break;
        case Stream64::kWide256: launch_draft<Wide256>(a, L, ws, p, s, ev); break;
      }
      break;
    // <ids, draft rows, waves along ids, waves along rows, ring depth, K loop, non-temporal W
    // copies, MFMA shape>. Eight waves: one workgroup per CU needs them to keep copies and MFMAs
    // in flight. The spread loop on the wider tiles (128 ids x 256 rows: 59 us a round against
    // 72 us with the burst ring); the 128x128 tile is MFMA-light and 2-5% faster on the burst
    // ring (32000 ids, 80 and 128 rows), where the 32x32 shape's cheaper epilogue (one lane
    // merge instead of two, on half as many row blocks) is worth another 1-3%. The hint pays on
    // the others (64000 ids, 128 rows: 294 -> 284 us for three steps; 256 rows: 450 -> 432).
    case DraftTile::kRows128x128:
      launch_draft<TileFamily<128, 128, 2, 4, 3, 0, false, Mfma32>>(a, L, ws, p, s, ev);
      break;
    case DraftTile::kRows128x192:
      launch_draft<TileFamily<192, 128, 2, 4, 3, 3, true>>(a, L, ws, p, s, ev);
      break;
    case DraftTile::kRows128x256:
      launch_draft<TileFamily<256, 128, 2, 4, 3, 3, true>>(a, L, ws, p, s, ev);
      break;
    case DraftTile::kRows256x128:
      launch_draft<TileFamily<128, 256, 2, 4, 3, 3, true>>(a, L, ws, p, s, ev);
      break;
  }
  if (int rc = launch_status("k_draft_partial")) return rc;
  DraftGrowArgs g;
  g.B = a->B;
  g.S = p.cut.S;
  g.step = a->step;
  g.rec_k = reinterpret_cast<const uint64_t*>(ws + L.off_k);
  g.rec_s = reinterpret_cast<const float*>(ws + L.off_s);
  g.vocab_map = a->vocab_map;
  g.state = a->state;
  for (int k = 0; k < 3; ++k) g.shape[k] = a->shape[k];
  g.tree = a->tree;
  g.topk_id = a->topk_id;
  g.topk_logp = a->topk_logp;
  g.row_lse = a->row_lse;
  g.front_tok = a->front_tok;
  g.draft_conf = a->draft_conf;
  // the records of a row in one round of loads: four a lane up to 256 of them, else eight
  if (g.S <= 4 * kWave)
    k_draft_grow<4><<<a->B, kDraftThreads, 0, s>>>(g);
  else
    k_draft_grow<8><<<a->B, kDraftThreads, 0, s>>>(g);
  return launch_status("k_draft_grow");
}

extern "C" int asv_draft_step(const asv_draft_args* a, void* workspace, uint64_t workspace_bytes,
                              void* stream) {
  return asv_draft_step_tuned(a, nullptr, workspace, workspace_bytes, stream);
}

extern "C" int asv_draft_prune(const asv_draft_tree* tree, int32_t B, const int32_t* root_tok,
                               int32_t n_cap, int32_t* parent, int32_t* draft_tok,
                               int32_t* req_offsets, int32_t* req_status, void* stream) {
  if (B < 0 || n_cap < 0) return ASV_EINVAL;
  if (B == 0) return ASV_OK;
  if (!tree || !parent || !draft_tok || !req_offsets || !req_status) return ASV_EINVAL;
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  (void)hipGetLastError();
  k_draft_prune<<<B, kPruneThreads, 0, s>>>(tree, root_tok, n_cap, parent, draft_tok,
                                            req_offsets, req_status);
  return launch_status("k_draft_prune");
}

extern "C" int asv_tree_meta(const int32_t* parent, const int32_t* req_offsets, int32_t B,
                             int32_t N, const int32_t* pos_base, int32_t mask_words,
                             int32_t* pos, uint32_t* mask, int32_t* req_status, void* stream) {
  if (B < 0 || N < B || (B == 0) != (N == 0)) return ASV_EINVAL;
  if (B == 0) return ASV_OK;
  if (!parent || !req_offsets || !req_status || (mask && mask_words < 1)) return ASV_EINVAL;
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  (void)hipGetLastError();
  k_tree_meta<<<B, kMetaThreads, 0, s>>>(parent, req_offsets, B, N, pos_base, mask_words, pos,
                                         mask, req_status);
  return launch_status("k_tree_meta");
}

extern "C" int asv_commit(const asv_commit_args* a, void* stream) {
  if (!a || a->B < 0 || a->N < a->B || (a->B == 0) != (a->N == 0)) return ASV_EINVAL;
  if (a->B == 0) return ASV_OK;
  if (!a->req_offsets || !a->draft_tok || !a->accepted_len || !a->accepted_path ||
      !a->bonus_token || !a->commit_off || !a->commit_tok || !a->commit_row || !a->req_status)
    return ASV_EINVAL;
  if (a->row_src) {
    if (!a->row_dst || a->row_bytes <= 0 || a->row_bytes % 4 != 0) return ASV_EINVAL;
    if ((reinterpret_cast<uintptr_t>(a->row_src) | reinterpret_cast<uintptr_t>(a->row_dst)) & 3)
      return ASV_EINVAL;
  }
  CommitArgs c;
  c.B = a->B;
  c.N = a->N;
  c.off = a->req_offsets;
  c.tok = a->draft_tok;
  c.acc_len = a->accepted_len;
  c.path = a->accepted_path;
  c.bonus = a->bonus_token;
  c.c_off = a->commit_off;
  c.c_tok = a->commit_tok;
  c.c_row = a->commit_row;
  c.src = static_cast<const char*>(a->row_src);
  c.dst = static_cast<char*>(a->row_dst);
  c.row_bytes = a->row_bytes;
  c.status = a->req_status;
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  (void)hipGetLastError();
  k_commit<<<dim3(a->B, c.src ? kCommitSplit : 1), kCommitThreads, 0, s>>>(c);
  return launch_status("k_commit");
}
