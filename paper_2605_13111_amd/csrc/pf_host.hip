// Host-side validation, sizing and planning of libpf.so (no kernels in this file).
#include <math.h>
#include <stdlib.h>
#include <string.h>
#include <algorithm>
#include <mutex>
#include <unordered_map>
#include <vector>
#include "pf_internal.h"

static bool aligned16(const void *p) { return (((uintptr_t)p) & 15u) == 0; }

static bool policy_ok(const pf_head_policy &p) {
  if (p.type != PF_ANCHOR && p.type != PF_WAVE && p.type != PF_VEIL) return false;
  if (p.type == PF_ANCHOR && (p.mode < PF_MODE_ALL || p.mode > PF_MODE_TOPK)) return false;
  if (p.sink < 0 || p.recent < 0 || p.cap < 0 || p.slots < 1) return false;
  if (p.type == PF_WAVE && p.period < 1) return false;
  if (p.type == PF_VEIL && p.cap > 0 && (p.cap > 64 || p.period < 1 || p.period > 64 || p.slots <= p.cap)) return false;
  return true;
}

int pf_validate_pool(const pf_pool *pool) {
  if (!pool) return PF_ERR_INVALID_ARG;
  if (pool->n_heads < 1 || pool->n_heads > PF_MAX_HEADS) return PF_ERR_INVALID_ARG;
  if (pool->tokens_per_frame < 1 || pool->total_slots < 1) return PF_ERR_INVALID_ARG;
  if (pool->dtype != 0) return PF_ERR_UNSUPPORTED;
  if (pool->head_dim != 64 && pool->head_dim != 128) return PF_ERR_UNSUPPORTED;
  if (!pool->k_pool || !pool->v_pool || !pool->policy_host || !pool->policy_dev || !pool->slot_base ||
      !pool->n_frames || !pool->frame_ids || !pool->frame_score || !pool->T_dev || !pool->sync)
    return PF_ERR_INVALID_ARG;
  if (!aligned16(pool->k_pool) || !aligned16(pool->v_pool)) return PF_ERR_INVALID_ARG;
  if (pool->T_host < 0) return PF_ERR_INVALID_ARG;
  long long total = 0;
  for (int h = 0; h < pool->n_heads; ++h) {
    if (!policy_ok(pool->policy_host[h])) return PF_ERR_INVALID_ARG;
    total += pool->policy_host[h].slots;
  }
  if (total != pool->total_slots) return PF_ERR_INVALID_ARG;
  // token offsets inside one head's key sequence are kept in 32-bit integers
  for (int h = 0; h < pool->n_heads; ++h)
    if ((long long)pool->policy_host[h].slots * pool->tokens_per_frame > (1ll << 30)) return PF_ERR_INVALID_ARG;
  return PF_OK;
}

// ---- process-wide tuning switches ---------------------------------------------------------------
// Defaults come from the environment (PF_ATTN_VARIANT, PF_ATTN_QUEUE, PF_SEG_TILES, PF_PLAN_UNIFORM), read once at
// first use; pf_set_tuning changes them afterwards.  Plain ints: a change races with calls running on other threads.
namespace {
struct Tuning {
  int attn_variant, attn_queue, seg_tiles, plan_uniform;
};
int env_int(const char *name, int dflt) {
  const char *e = getenv(name);
  return e ? atoi(e) : dflt;
}
Tuning &tuning() {
  static Tuning t = {env_int("PF_ATTN_VARIANT", -1), env_int("PF_ATTN_QUEUE", 1),
                     env_int("PF_SEG_TILES", 0), getenv("PF_PLAN_UNIFORM") ? 1 : 0};
  return t;
}
}  // namespace

extern "C" int pf_set_tuning(int attn_variant, int attn_queue, int seg_tiles, int plan_uniform) {
  if (attn_variant >= PF_NUM_VARIANTS || seg_tiles > (1 << 20)) return PF_ERR_INVALID_ARG;
  Tuning &t = tuning();
  if (attn_variant >= 0) t.attn_variant = attn_variant;
  if (attn_variant == -2) t.attn_variant = -1;       // the library's own choice again
  if (attn_queue >= 0) t.attn_queue = attn_queue != 0;
  if (seg_tiles >= 0) t.seg_tiles = seg_tiles;
  if (plan_uniform >= 0) t.plan_uniform = plan_uniform != 0;
  return PF_OK;
}

int pf_tuned_seg_tiles() { return tuning().seg_tiles > 0 ? tuning().seg_tiles : 0; }

int pf_resolve_seg_tiles(int seg_tiles) {
  if (seg_tiles <= 0) {
    seg_tiles = pf_tuned_seg_tiles();
    if (seg_tiles <= 0) seg_tiles = PF_DEFAULT_SEG_TILES;
  }
  return seg_tiles < PF_MIN_SEG_TILES ? PF_MIN_SEG_TILES : seg_tiles;
}

// ---- automatic segment lengths ------------------------------------------------------------------
// The launch is a list of blocks, one per (head, key segment, query tile); block i belongs to die i % 8.
//   * one block per workgroup (kernel 0): the hardware sends block i to die i % 8, and a die starts its next
//     block on the first compute unit that frees up;
//   * work queue (kernel 1): one resident workgroup per compute unit takes the next block of its die's list, and
//     from the next die's list once its own is empty.
// With three or four blocks per compute unit the finish time depends strongly on how the blocks pack, so the
// plan is chosen by replaying the schedule on the host (costs: one key tile = 1, a fixed cost per block, an
// extra cost when a partial result has to be parked, and for a head's last segment the cost of reading back
// every partial it merges; the constants are fitted to per-layer timings of every candidate) and keeping
// the shortest finish:
//   1. one segment length for every head, from a list of candidates;
//   2. starting from that, heads with the same key count try every segment count of their own while the
//      others stay fixed, a few rounds (pools of up to PF_PLAN_HEADS heads).
// Plans are remembered per (key tiles of every head, query tiles, kernel, mode) in a hash table large enough for
// whole rollouts, so a step whose shape has been seen before pays a lookup.
static const int kSegCandidates[] = {16, 24, 32, 48, 56, 64, 72, 80, 96, 112, 128, 144, 160, 176, 192, 224, 256, 320, 384};
constexpr int PF_AUTO_MIN_SEG = 48;                 // shortest planned segment: bounds the partial-result workspace
// head_dim 64: a launch that has no more than this many blocks even so may cut down to 16, 24 or 32 tiles.  Four workgroups fit
// a compute unit there and the first ones gain the most: with 5 heads x 4680 queries x 74 tiles, 370 blocks take 78 us, 555
// 63 us, 740 70 us; 6 heads x 600 queries x up to 150 tiles 47 us in 80 blocks, 39 us in 180; 12 heads x 1200 queries x up to
// 132 tiles 59 us in 300 or 570 blocks, 69 us in 870.  The limit also bounds what such plans need of the workspace (22 MB).
constexpr int PF_SHORT_SEG_BLOCKS = 640;
static const int kShortSegs[] = {16, 24, 32};
struct PlanCosts {
  double block, split, merge;                       // per block; per parked partial; per partial read back by the merging block
};
static const PlanCosts kCostsDirect = {8.0, 2.0, 2.0};
static const PlanCosts kCostsQueue = {4.0, 1.0, 2.0};
// Charged 2 and 3, as before partial results were parked in the order the threads hold them and read back without emptying an L2, heads
// were cut too coarsely (12 heads x 1560 queries x up to 514 tiles, six layers: 245 blocks a layer, 1018 us; now up to 343, 958; 91
// random launches that are cut otherwise take 0.990 of their time on average, 0.67 to 1.05).
// 1 and 1 or 2 and 1 cut too finely (8 heads x 1560 queries, 45 frames: 419 -> 431 us; with 1 and 2 419).  The former
// charges still say which launches are cut at all.
static const PlanCosts kCostsQueueCut = {4.0, 2.0, 3.0};
static const PlanCosts kCostsD64 = {2.0, 0.7, 0.7};  // a tile takes four times as long where four workgroups share a compute unit
// A thin block (32 query rows, pf_attn_thin.h): its share of a full block's time per key tile, its fixed cost, and what parking a
// partial result adds to it.  A full block's time shared by its eight groups of 32 rows would be 0.125, but a thin block streams all
// its keys for 32 rows alone: where many of them run at once that costs 0.30 (16 heads x 1038 queries x up to 503 tiles: 180 us as
// 1056 thin blocks, 124 us as full ones; 5 heads x 1560 queries x up to 537 tiles 138 us against 108), and they pay where full
// blocks leave most of the chip idle (5 heads x 666 queries x up to 58 tiles: 25 us against 57).  The fixed cost is the one of a
// launch whose blocks are mostly taken over by other dies (12 heads x 1560 queries x 25 tiles: 55 us as thin blocks, 45 us as full
// ones).  Parking was charged 0.25 to 1 at first: launches of split thin blocks took 5 to 20 tiles longer than replayed, 4 per
// block (7 heads x 1380 queries x up to 54 tiles: 65 us as 704 thin blocks in halves, 55 us as full ones).  All of this was fitted when
// merges and border steps cost both forms more than now.  Looked at since over 220 random launches whose replays lie within 0.6 to 1
// of each other: the choice takes 0.705 of the full form's time on average and more than 1.02 of it 7 times (up to 1.16: 35 heads x
// 204 queries x 5 tiles, frames of 31 tokens, 18.4 us against 15.8; 27 x 82 x 662, 150 against 130), and in 16 of the 31 that it
// leaves to the full form thin items would take at least 5 % less.
static const double kThinTile = 0.30, kThinBlock = 5.5, kThinPark = 4.0;
// ... must finish this much earlier than full ones by the replay, which is good to about a tenth; and what kCostsQueue.merge, fitted to
// launches of two to four segments a head, charges too much for one with many: at 3 per partial, 20 segments were replayed at 122
// tiles and took 86 (2 heads x 1192 queries x 1118 tiles), 10 at 81 and took 61, 5 at 66 and took 61.
static const double kThinGain = 0.9, kMergeOver = 1.0;
constexpr int PF_PLAN_ROUNDS = 3;
constexpr int PF_PLAN_MAX_NSEG = 16;                // segment counts tried per head in step 2
constexpr double PF_PLAN_MIN_GAIN = 0.01;           // step 2 must beat step 1 by this much to be used
constexpr size_t PF_PLAN_CACHE = 16384;            // remembered plans (about 300 bytes each)

// Blocks of a launch: n_qt query tiles per (head, segment).
struct LaunchShape {
  int n_qt, slots_per_die, min_seg;
  bool thin, queue, d64, cut;                        // cut: replayed only to see which launches are cut
};
static LaunchShape launch_shape(int variant, int head_dim, int q_tokens, bool queue) {
  LaunchShape S;
  const int bq = pf_variant_bq(variant);
  S.n_qt = pf_ceil_div(q_tokens, bq);
  S.slots_per_die = 32 * (variant != 0 ? 1 : head_dim == 64 ? 4 : 2);   // workgroups resident per die
  S.thin = variant == PF_THIN_VARIANT;
  S.queue = queue;
  S.d64 = head_dim == 64;
  S.cut = false;
  S.min_seg = PF_AUTO_MIN_SEG;
  return S;
}

// A worker of the replay as one number, by which the heap gives the one who is free first (equal times: the lower die): times are not
// negative, so their bits are ordered as they are.  A worker who takes a block is given back with a later time: the hole at the top sinks
// along the earlier children and he rises from the bottom, where most stay.  Taken out and put in again as two steps, and with memory of
// its own for every replay, a plan took 2.8 ms on average over 400 random launches at head_dim 128 (up to 39), now 0.7 (up to 10).
typedef unsigned __int128 Worker;
static Worker worker(double free_at, int home) {
  unsigned long long bits;
  memcpy(&bits, &free_at, sizeof(bits));
  return (Worker)bits << 8 | (unsigned)home;
}
static double free_at(Worker w) {
  const unsigned long long bits = (unsigned long long)(w >> 8);
  double t;
  memcpy(&t, &bits, sizeof(t));
  return t;
}
static void replace_top(std::vector<Worker> &heap, Worker w) {
  Worker *const a = heap.data();
  const size_t n = heap.size();
  size_t at = 0, c = 1;
  for (; c + 1 < n; c = 2 * at + 1) {
    c += a[c + 1] < a[c];
    a[at] = a[c];
    at = c;
  }
  if (c < n) {
    a[at] = a[c];
    at = c;
  }
  for (; at > 0 && w < a[(at - 1) / 2]; at = (at - 1) / 2) a[at] = a[(at - 1) / 2];
  a[at] = w;
}
struct ReplayMemory {                                // kept over the replays of one plan
  std::vector<int> order, nsegs, len;
  std::vector<double> teams[PF_NUM_XCD];             // per die: the cost of each team (n_qt equal blocks), in launch order
  std::vector<Worker> workers;
};

// Finish time of the launch in which head h has key tiles n_kvt[h] cut into segments of at most seg[h] tiles; of one that takes at
// least `bound`, maybe only that much of it is known.
static double model_finish(const std::vector<int> &n_kvt, const std::vector<int> &seg, const LaunchShape &S, double bound, ReplayMemory &M) {
  const PlanCosts &C = S.d64 ? kCostsD64 : !S.queue ? kCostsDirect : S.cut ? kCostsQueueCut : kCostsQueue;
  const int H = (int)n_kvt.size();
  // heads by descending segment length (ties: head id), as the index kernel ranks them
  M.order.resize(H), M.nsegs.resize(H), M.len.resize(H);
  for (int h = 0; h < H; ++h) {
    M.order[h] = h;
    M.nsegs[h] = pf_max(1, pf_ceil_div(n_kvt[h], seg[h]));
    M.len[h] = pf_ceil_div(n_kvt[h], M.nsegs[h]);
  }
  std::sort(M.order.begin(), M.order.end(), [&](int a, int b) { return M.len[a] != M.len[b] ? M.len[a] > M.len[b] : a < b; });
  for (int x = 0; x < PF_NUM_XCD; ++x) M.teams[x].clear();
  int k = 0;                                         // team rank, as in the index kernel
  for (int o = 0; o < H; ++o) {
    const int nk = n_kvt[M.order[o]], nseg = M.nsegs[M.order[o]];
    for (int sgi = 0; sgi < nseg; ++sgi, ++k) {
      const int row = k / PF_NUM_XCD, col = k % PF_NUM_XCD;
      const int xcd = (row & 1) ? PF_NUM_XCD - 1 - col : col;
      const int tiles = pf_seg_begin(nk, nseg, sgi + 1) - pf_seg_begin(nk, nseg, sgi);
      // the merge falls to whichever segment arrives last; the replay charges it to the last one launched
      const double park = (nseg > 1 ? C.split : 0.0) + (nseg > 1 && sgi == nseg - 1 ? C.merge * nseg : 0.0);
      M.teams[xcd].push_back(S.thin ? kThinTile * tiles + kThinBlock + (nseg > 1 ? kThinPark : 0.0) : tiles + C.block + park);
    }
  }
  // No schedule ends before its work spread evenly would (over a die where dies keep to their lists, over the chip otherwise), and none
  // gets shorter again: most cuts are seen to lose without a whole replay.
  double even = 0.0;
  for (int x = 0; x < PF_NUM_XCD; ++x) {
    double die = 0.0;
    for (double t : M.teams[x]) die += t * S.n_qt;
    even = S.queue ? even + die / PF_NUM_XCD : die > even ? die : even;
  }
  even /= S.slots_per_die;
  if (even * (1.0 - 1e-9) >= bound) return even;
  double finish = 0.0;
  if (!S.queue) {
    for (int x = 0; x < PF_NUM_XCD; ++x) {
      M.workers.assign(S.slots_per_die, worker(0.0, 0));
      for (double t : M.teams[x])
        for (int i = 0; i < S.n_qt; ++i) {
          const double e = free_at(M.workers[0]) + t;
          replace_top(M.workers, worker(e, 0));
          finish = e > finish ? e : finish;
          if (finish >= bound) return finish;
        }
    }
    return finish;
  }
  // work queue: the worker that frees up first takes the next block of its die's list, else of the next die's
  M.workers.resize(PF_NUM_XCD * S.slots_per_die);
  for (size_t w = 0; w < M.workers.size(); ++w) M.workers[w] = worker(0.0, (int)w / S.slots_per_die);   // in order, so a heap
  size_t next[PF_NUM_XCD] = {}, left = 0;            // the team that a die hands out, and blocks of it that are gone
  int gone[PF_NUM_XCD] = {};
  for (int x = 0; x < PF_NUM_XCD; ++x) left += M.teams[x].size() * (size_t)S.n_qt;
  for (; left > 0; --left) {
    const int home = (int)(M.workers[0] & 255);
    int x = home;
    while (next[x] == M.teams[x].size()) x = (x + 1) % PF_NUM_XCD;
    const double e = free_at(M.workers[0]) + M.teams[x][next[x]];
    if (++gone[x] == S.n_qt) gone[x] = 0, ++next[x];
    replace_top(M.workers, worker(e, home));
    finish = e > finish ? e : finish;
    if (finish >= bound) return finish;
  }
  return finish;
}

namespace {
// Remembered plans: key = key tiles of every head, then query tiles, then kernel / launch form / planning depth.
// Sized for whole rollouts (30 layers x a few hundred history lengths each have their own key); emptied when full.
struct KeyHash {
  size_t operator()(const std::vector<int> &k) const {
    unsigned long long h = 1469598103934665603ull;
    for (size_t i = 0; i < k.size(); ++i) h = (h ^ (unsigned)k[i]) * 1099511628211ull;
    return (size_t)h;
  }
};
std::mutex g_plan_mutex;
struct Remembered {
  PfSegPlan plan;
  int variant;
};
std::unordered_map<std::vector<int>, Remembered, KeyHash> g_plan_cache;

// Segment lengths for one kernel; returns the replayed finish time.
double plan_segments(const std::vector<int> &n_kvt, const LaunchShape &S, bool uniform_only, PfSegPlan *plan, ReplayMemory &M) {
  const int H = (int)n_kvt.size();
  // Many candidate lengths cut the heads into the same segment counts: the replay runs once per distinct cut.
  std::unordered_map<std::vector<int>, double, KeyHash> seen;
  std::vector<int> cut(H);
  // a bound is never larger than an earlier one, so what was found too late once stays so
  auto finish_of = [&](const std::vector<int> &seg, double bound) {
    for (int h = 0; h < H; ++h) cut[h] = pf_max(1, pf_ceil_div(n_kvt[h], seg[h]));
    auto f = seen.find(cut);
    if (f != seen.end()) return f->second;
    const double t = model_finish(n_kvt, seg, S, bound, M);
    seen.emplace(cut, t);
    return t;
  };

  // step 1: one length for all
  std::vector<int> seg(H);
  double best_t = 0.0;
  for (size_t ci = 0; ci < sizeof(kSegCandidates) / sizeof(kSegCandidates[0]); ++ci) {
    if (kSegCandidates[ci] < S.min_seg) continue;
    std::fill(seg.begin(), seg.end(), kSegCandidates[ci]);
    const double t = finish_of(seg, best_t == 0.0 ? INFINITY : best_t);
    if (best_t == 0.0 || t < best_t * 0.995) {       // a longer segment must win clearly: it costs fewer partials
      best_t = best_t == 0.0 ? t : (t < best_t ? t : best_t);
      plan->uniform = kSegCandidates[ci];
    }
  }
  std::fill(seg.begin(), seg.end(), plan->uniform);
  const double uniform_t = best_t;
  if (uniform_only) return uniform_t;

  // step 2: per key count, the segment count of its own
  std::vector<int> distinct(n_kvt);
  std::sort(distinct.begin(), distinct.end());
  distinct.erase(std::unique(distinct.begin(), distinct.end()), distinct.end());
  double cur_t = uniform_t;
  for (int round = 0; round < PF_PLAN_ROUNDS; ++round) {
    bool changed = false;
    for (size_t d = 0; d < distinct.size(); ++d) {
      const int nk = distinct[d];
      int cur_seg = 0;
      for (int h = 0; h < H; ++h)
        if (n_kvt[h] == nk) cur_seg = seg[h];
      int best_seg = cur_seg;
      for (int n = 1; n <= PF_PLAN_MAX_NSEG; ++n) {
        const int cand = pf_ceil_div(nk, n);
        if (cand < S.min_seg && n > 1) break;
        if (cand == cur_seg) continue;
        for (int h = 0; h < H; ++h)
          if (n_kvt[h] == nk) seg[h] = pf_max(cand, S.min_seg);
        const double t = finish_of(seg, cur_t * 0.998);
        if (t < cur_t * 0.998) {
          cur_t = t;
          best_seg = pf_max(cand, S.min_seg);
        }
      }
      for (int h = 0; h < H; ++h)
        if (n_kvt[h] == nk) seg[h] = best_seg;
      changed = changed || best_seg != cur_seg;
    }
    if (!changed) break;
  }
  if (cur_t >= uniform_t * (1.0 - PF_PLAN_MIN_GAIN)) return uniform_t;
  plan->per_head = 1;
  for (int h = 0; h < H; ++h) plan->seg[h] = (uint16_t)pf_min(seg[h], 65535);
  return cur_t;
}

// Partial results of a launch with n_qt query tiles per head.
size_t plan_partials(const std::vector<int> &n_kvt, const PfSegPlan &plan, int n_qt) {
  size_t n = 0;
  for (size_t h = 0; h < n_kvt.size(); ++h)
    if (n_kvt[h] > plan.of((int)h)) n += (size_t)pf_ceil_div(n_kvt[h], plan.of((int)h)) * n_qt;
  return n;
}
bool plan_splits(const std::vector<int> &n_kvt, const PfSegPlan &plan) { return plan_partials(n_kvt, plan, 1) > 0; }
}  // namespace

int pf_auto_plan(const pf_pool *pool, int T, int q_tokens, PfSegPlan *plan) {
  const int H = pool->n_heads;
  const int variant = pf_resolve_variant(pool->head_dim);
  const bool queue = pf_attn_queue_mode(variant);
  const LaunchShape S = launch_shape(variant, pool->head_dim, q_tokens, queue);
  memset(plan, 0, sizeof(*plan));
  plan->uniform = PF_DEFAULT_SEG_TILES;
  std::vector<int> key(H + 2);
  long long total = 0, tiles = 0;
  for (int h = 0; h < H; ++h) {
    const int nsel = pf_sel_count_impl(pool->policy_host[h], T);
    key[h] = pf_ceil_div(nsel * pool->tokens_per_frame + q_tokens, PF_BK);
    total += pf_ceil_div(key[h], PF_AUTO_MIN_SEG);
    tiles += key[h];
  }
  if (total * S.n_qt > 50000) return variant;                     // keep the replay cheap on huge launches
  const bool uniform_only = H > PF_PLAN_HEADS || tuning().plan_uniform != 0;
  const bool may_thin = tuning().attn_variant < 0 && pool->head_dim == 128 && queue;
  key[H] = q_tokens;
  key[H + 1] = (variant * 256 + pool->head_dim) * 8 + (may_thin ? 4 : 0) + (queue ? 2 : 0) + (uniform_only ? 1 : 0);
  {
    std::lock_guard<std::mutex> lock(g_plan_mutex);
    auto hit = g_plan_cache.find(key);
    if (hit != g_plan_cache.end()) {
      *plan = hit->second.plan;
      return hit->second.variant;
    }
  }
  const std::vector<int> n_kvt(key.begin(), key.begin() + H);
  Remembered R;
  R.variant = variant;
  ReplayMemory M;
  double finish = plan_segments(n_kvt, S, uniform_only, plan, M);
  // A launch whose heads fit one segment each needs no workspace, and callers may rely on that: the forms below are not
  // allowed to bring partial results into it.
  bool splits = plan_splits(n_kvt, *plan);
  if (splits && (S.d64 || queue)) {
    // Callers may also rely on which launches do without scratch memory, or with the library's own array.  That is decided by a
    // replay with kCostsQueueCut, at head_dim 64 with the rates of two workgroups per compute unit: what it leaves whole stays whole,
    // and what it fits into the array stays in it, although more, shorter segments would often finish earlier (head_dim 64, 40
    // heads x 4680 queries x up to 1463 key tiles: 1480 blocks without partial results, or 16280 with 550 MB of them).
    LaunchShape before = S;
    before.cut = true;
    before.d64 = false;
    if (S.d64) before.slots_per_die = 64;
    const size_t slot = pf_partial_bytes(pf_variant_bq(variant), pool->head_dim);
    const bool over = plan_partials(n_kvt, *plan, S.n_qt) * slot > PF_STATIC_SCRATCH_BYTES;
    PfSegPlan base;
    memset(&base, 0, sizeof(base));
    double base_finish = plan_segments(n_kvt, before, true, &base, M);
    // step 2 only betters step 1: it leaves a launch cut that step 1 cuts, unless whole heads finish earlier
    const bool cut_anyway = plan_splits(n_kvt, base) && model_finish(n_kvt, n_kvt, before, INFINITY, M) >= base_finish;
    if (!uniform_only && (over || !cut_anyway)) {
      memset(&base, 0, sizeof(base));
      base_finish = plan_segments(n_kvt, before, false, &base, M);
    }
    splits = plan_splits(n_kvt, base);
    if (!splits || (over && plan_partials(n_kvt, base, S.n_qt) * slot <= PF_STATIC_SCRATCH_BYTES)) {
      *plan = base;
      if (!S.d64) finish = base_finish;
    }
  }
  if (splits && S.d64) {
    LaunchShape fine = S;
    for (int seg : kShortSegs) {
      long long teams = 0;
      for (int h = 0; h < H; ++h) teams += pf_ceil_div(n_kvt[h], seg);
      if (teams * S.n_qt > PF_SHORT_SEG_BLOCKS) continue;
      fine.min_seg = seg;
      break;
    }
    PfSegPlan fp;
    memset(&fp, 0, sizeof(fp));
    if (fine.min_seg < S.min_seg && plan_segments(n_kvt, fine, uniform_only, &fp, M) < finish) *plan = fp;
  }
  // Small launches: with 32 query rows per block there are eight times the blocks, at 2.4 times the time per row; which side wins is
  // left to the replay.  Looked at only where it could: its work spread evenly over the chip would finish earlier.
  if (may_thin) {
    int most = 1;
    for (int h = 0; h < H; ++h) most = pf_max(most, pf_ceil_div(n_kvt[h], plan->of(h)));
    const double full = finish - (most > 1 ? kMergeOver * most : 0.0);
    const LaunchShape thin = launch_shape(PF_THIN_VARIANT, pool->head_dim, q_tokens, queue);
    const double even = thin.n_qt * (kThinTile * tiles + kThinBlock * H) / (PF_NUM_XCD * thin.slots_per_die);
    if (even < full && total * thin.n_qt <= PF_THIN_MAX_BLOCKS) {
      PfSegPlan tp;
      memset(&tp, 0, sizeof(tp));
      if (plan_segments(n_kvt, thin, true, &tp, M) < kThinGain * full && (splits || !plan_splits(n_kvt, tp))) {
        *plan = tp;
        R.variant = PF_THIN_VARIANT;
      }
    }
  }
  R.plan = *plan;
  std::lock_guard<std::mutex> lock(g_plan_mutex);
  if (g_plan_cache.size() >= PF_PLAN_CACHE) g_plan_cache.clear();
  g_plan_cache.emplace(key, R);
  return R.variant;
}

bool pf_attn_queue_mode(int variant) { return variant >= 1 && tuning().attn_queue != 0; }

int pf_resolve_variant(int head_dim) {
  int v = tuning().attn_variant;
  if (v < 0 || v >= PF_NUM_VARIANTS) v = PF_DEFAULT_VARIANT;
  return head_dim == 128 ? v : 0;                   // the pipelined kernels exist for head_dim 128 only
}

void pf_host_plan(const pf_pool *pool, int T, int q_tokens, int variant, const PfSegPlan &plan,
                  int *n_teams, int *n_blocks, int *n_partials, int *max_sel_needed) {
  const int n_qt = pf_ceil_div(q_tokens, pf_variant_bq(variant));
  long long teams = 0, parts = 0;
  int max_sel = 0;
  for (int h = 0; h < pool->n_heads; ++h) {
    const int nsel = pf_sel_count_impl(pool->policy_host[h], T);
    max_sel = pf_max(max_sel, nsel);
    const PfHeadPlan hp = pf_plan_head(nsel * pool->tokens_per_frame + q_tokens, plan.of(h));
    teams += hp.nseg;
    if (hp.nseg > 1) parts += (long long)hp.nseg * n_qt;
  }
  *n_teams = (int)teams;
  *n_blocks = (int)(pf_ceil_div((int)teams, PF_NUM_XCD) * PF_NUM_XCD * (long long)n_qt);
  *n_partials = (int)parts;
  *max_sel_needed = max_sel;
}

// Worst case over every T the slot capacities allow: a head never selects more frames than it has slots.
static void worst_case(const pf_pool *pool, int q_tokens, int seg_tiles, int variant, long long *max_blocks,
                       long long *max_partials, int *n_qt_out) {
  const int n_qt = pf_ceil_div(q_tokens, pf_variant_bq(variant));
  long long teams = 0, parts = 0;
  for (int h = 0; h < pool->n_heads; ++h) {
    const long long lkv = (long long)pool->policy_host[h].slots * pool->tokens_per_frame + q_tokens;
    const PfHeadPlan hp = pf_plan_head((int)lkv, seg_tiles);
    teams += hp.nseg;
    if (hp.nseg > 1) parts += (long long)hp.nseg * n_qt;
  }
  *max_blocks = (teams + PF_NUM_XCD - 1) / PF_NUM_XCD * PF_NUM_XCD * n_qt;
  *max_partials = parts;
  *n_qt_out = n_qt;
}

extern "C" size_t pf_index_work_bytes(const pf_pool *pool, int q_tokens) {
  if (pf_validate_pool(pool) != PF_OK || q_tokens < 1) return 0;
  size_t need = 0;
  for (int v = 0; v < PF_NUM_KERNELS; ++v) {
    long long mb, mp;
    int n_qt;
    worst_case(pool, q_tokens, v == PF_THIN_VARIANT ? PF_AUTO_MIN_SEG : PF_MIN_SEG_TILES, v, &mb, &mp, &n_qt);
    // the planner takes thin blocks only for small launches (padding: see pf_host_plan); then there are no more counters than blocks
    if (v == PF_THIN_VARIANT && mb > PF_THIN_MAX_BLOCKS + (PF_NUM_XCD - 1) * n_qt) {
      mb = PF_THIN_MAX_BLOCKS + (PF_NUM_XCD - 1) * (long long)n_qt;
      n_qt = pf_min(n_qt, PF_THIN_MAX_BLOCKS / pool->n_heads);
    }
    const size_t t = pf_work_layout(pool->n_heads, n_qt, mb).total;
    need = t > need ? t : need;
  }
  return need;
}

extern "C" size_t pf_attn_workspace_bytes(const pf_pool *pool, int q_tokens) {
  if (pf_validate_pool(pool) != PF_OK || q_tokens < 1) return 0;
  // The shortest automatic segment length (or the PF_SEG_TILES override) bounds the partial count unless the
  // caller asks for shorter segments through pf_index.seg_tiles; pf_ragged_attn_fwd checks the actual need
  // against workspace_bytes.
  size_t need = 0;
  for (int v = 0; v < PF_NUM_KERNELS; ++v) {
    long long mb, mp;
    int n_qt;
    worst_case(pool, q_tokens, pf_tuned_seg_tiles() ? pf_resolve_seg_tiles(0) : PF_AUTO_MIN_SEG, v, &mb, &mp, &n_qt);
    if (pool->head_dim == 64 && v == 0 && !pf_tuned_seg_tiles()) {       // small launches may cut finer
      long long mb_short, mp_short;
      worst_case(pool, q_tokens, PF_MIN_SEG_TILES, v, &mb_short, &mp_short, &n_qt);
      mp_short = mp_short < PF_SHORT_SEG_BLOCKS ? mp_short : PF_SHORT_SEG_BLOCKS;
      mp = mp > mp_short ? mp : mp_short;
    }
    const size_t t = (size_t)mp * pf_partial_bytes(pf_variant_bq(v), pool->head_dim);
    need = t > need ? t : need;
  }
  return pf_align_up(need + 256, 256);
}

extern "C" int pf_plan_segments(const pf_pool *pool, int T, int q_tokens, int32_t *seg_tiles, int32_t *n_blocks,
                                int32_t *n_partials) {
  if (pf_validate_pool(pool) != PF_OK || T < 0 || q_tokens < 1 || q_tokens > (1 << 24)) return PF_ERR_INVALID_ARG;
  for (int h = 0; h < pool->n_heads; ++h)
    if (pf_sel_count_impl(pool->policy_host[h], T) > pool->policy_host[h].slots) return PF_ERR_INVALID_ARG;
  int variant = pf_resolve_variant(pool->head_dim);
  PfSegPlan plan;
  if (pf_tuned_seg_tiles()) {
    memset(&plan, 0, sizeof(plan));
    plan.uniform = pf_resolve_seg_tiles(0);
  } else {
    variant = pf_auto_plan(pool, T, q_tokens, &plan);
  }
  int teams, blocks, partials, max_sel;
  pf_host_plan(pool, T, q_tokens, variant, plan, &teams, &blocks, &partials, &max_sel);
  if (seg_tiles)
    for (int h = 0; h < pool->n_heads; ++h) seg_tiles[h] = plan.of(h);
  if (n_blocks) *n_blocks = blocks;
  if (n_partials) *n_partials = partials;
  return PF_OK;
}

extern "C" int pf_selected_count(const pf_head_policy *pol, int T) {
  if (!pol || T < 0 || !policy_ok(*pol)) return PF_ERR_INVALID_ARG;
  return pf_sel_count_impl(*pol, T);
}

extern "C" int pf_retained_count(const pf_head_policy *pol, int T) {
  if (!pol || T < 0 || !policy_ok(*pol)) return PF_ERR_INVALID_ARG;
  return pf_ret_count_impl(*pol, T);
}

extern "C" const char *pf_status_string(int status) {
  switch (status) {
    case PF_OK: return "ok";
    case PF_ERR_INVALID_ARG: return "invalid argument";
    case PF_ERR_CAPACITY: return "capacity exceeded";
    case PF_ERR_UNSUPPORTED: return "unsupported head_dim or dtype";
    case PF_ERR_HIP: return "HIP runtime error";
    default: return "unknown status";
  }
}
