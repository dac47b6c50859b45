// Host side of the HPD library: validation, layout tables and the C ABI.
// The layout follows the paper's problem statement: a shared header per prompt,
// J stacked documents (Section 4.3.5), N attribute branches per document decoded for at
// most K_max steps (Sections 4.3.1, 4.3.4), prompts batched (Section 4.3.6).
#include <algorithm>
#include <cmath>
#include <cstring>
#include <limits>
#include <new>
#include <numeric>
#include <string>

#include "hpd_internal.h"

namespace {

thread_local std::string g_hip_text = "no HIP error recorded";

int hip_fail(hipError_t e) {
  g_hip_text = std::string("HIP error: ") + hipGetErrorString(e);
  return HPD_E_HIP;
}

#define HPD_HIP(expr)                        \
  do {                                       \
    hipError_t e_ = (expr);                  \
    if (e_ != hipSuccess) return hip_fail(e_); \
  } while (0)

inline int64_t round_up(int64_t x, int64_t m) { return (x + m - 1) / m * m; }

size_t elem_bytes(const hpd_config& c) { return c.dtype == HPD_F32 ? 4 : 2; }
bool paper_mode(const hpd_layout* L) { return L->cfg.mask_mode == HPD_MASK_PAPER; }

int validate_config(const hpd_config* c) {
  if (!c) return HPD_E_INVALID;
  if (c->n_q_heads < 1 || c->n_kv_heads < 1 || c->n_q_heads % c->n_kv_heads != 0) return HPD_E_INVALID;
  if (c->head_dim < 2 || (c->head_dim & 1)) return HPD_E_INVALID;
  if (c->max_new < 1) return HPD_E_INVALID;
  if (!(c->rope_base > 1.0) || !std::isfinite(c->rope_base)) return HPD_E_INVALID;
  if (c->dtype != HPD_F32 && c->dtype != HPD_BF16) return HPD_E_UNSUPPORTED;
  if (c->head_dim % 8 != 0 || c->head_dim > 256) return HPD_E_UNSUPPORTED;
  if (c->pos_mode != HPD_POS_CONTIG && c->pos_mode != HPD_POS_PAPER_GAP) return HPD_E_UNSUPPORTED;
  if (c->mask_mode != HPD_MASK_BLOCK && c->mask_mode != HPD_MASK_PAPER) return HPD_E_UNSUPPORTED;
  if (c->mask_mode == HPD_MASK_PAPER && c->pos_mode != HPD_POS_PAPER_GAP) return HPD_E_INVALID;
  if (c->flags & ~HPD_FLAG_HOST_ONLY) return HPD_E_INVALID;
  if (c->out_dtype != HPD_OUT_SAME && c->out_dtype != HPD_OUT_F32) return HPD_E_UNSUPPORTED;
  return HPD_OK;
}

// The steps of the fp32 decode kernel.  A launch of as many row groups for every unit as the unit with the most
// branches needs is mostly empty workgroups where one document has many times the branches of the others, and an
// empty one is not free: 2000 documents of one branch and one of 2000, 16/4 heads x 64, 5854 us, one workgroup per
// row and head in the generic kernel 1020.  From twice the groups that exist on they are therefore listed: 254 us.
// (A list costs one more dependent load, and in a step of a few workgroups every load shows.)
void plan_f32(hpd_layout* L, int32_t n_cus) {
  const int32_t D = L->cfg.head_dim, G = L->cfg.n_q_heads / L->cfg.n_kv_heads;
  if (L->cfg.dtype != HPD_F32 || paper_mode(L) || G > HPD_F32_ROWS || (D != 32 && D != 64 && D != 128)) return;
  L->f32_steps.resize(L->T);
  std::vector<int32_t> list, last;
  for (int32_t t = 0; t < L->T; ++t) {
    hpd_f32_step& s = L->f32_steps[t];
    const int32_t u0 = L->unit_ptr[t], n_units = L->unit_ptr[t + 1] - u0;
    auto desc = [&](int32_t u) { return L->unit_desc.data() + (size_t)(u0 + u) * 8; };
    auto row_groups = [&](int32_t nb) { return (nb + s.per_group - 1) / s.per_group; };
    auto prefix_tiles = [&](int32_t u) { return (int64_t)(desc(u)[1] + 15) / 16 + (desc(u)[3] + 15) / 16; };
    auto tail_tiles = [&](int64_t nb) { return (nb * t + 15) / 16; };
    s.per_group = HPD_F32_ROWS / G;
    int64_t exist = 0, most = 1, all = 0;  // groups; tiles of the longest one and of all of them together
    for (;; s.per_group = (s.per_group + 1) / 2) {
      int64_t prefix = 1;  // tiles of the longest unit
      exist = all = 0;
      for (int32_t u = 0; u < n_units; ++u) {
        exist += row_groups(desc(u)[5]);
        prefix = std::max(prefix, prefix_tiles(u));
        all += row_groups(desc(u)[5]) * prefix_tiles(u) + tail_tiles(desc(u)[5]);
      }
      const int64_t tails = tail_tiles(std::min(s.per_group, L->max_rows[t]));
      most = prefix + tails;
      // Fewer branches per group where their tails are most of a group's keys and CUs are idle: a group
      // streams the prefix once for its branches, but the tails of each (one document of 32 keys, 16 branches of
      // 400 tokens, 4/4 heads x 64: one group per kv head 137 us, one per branch 16, generic kernels 50).
      if (s.per_group == 1 || tails <= prefix || exist * L->cfg.n_kv_heads >= n_cus) break;
    }
    s.rg = row_groups(L->max_rows[t]);
    s.groups = (int64_t)n_units * s.rg;
    if (s.groups > 2 * exist || s.rg > 65535) {  // (the row groups of a unit are the grid's y)
      s.rg = 0;
      s.groups = exist;
      list.clear();
      for (int32_t u = 0; u < n_units; ++u)
        for (int32_t g = 0; g < row_groups(desc(u)[5]); ++g) list.insert(list.end(), {u, g});
      if (list != last) {  // (steps in a row that lose no branch share one)
        L->f32_groups.insert(L->f32_groups.end(), list.begin(), list.end());
        last = list;
      }
      s.list = L->f32_groups.size() / 2 - (size_t)exist;
    }
    // A wave per tile of an average group: the waves that a shorter group has no tile for hold LDS and registers
    // that workgroups in the queue need (3000 documents of 20 keys and one of 3000, three branches each, 8/8 heads x
    // 32: 674 us with a wave per tile of the longest group, 260 so, 302 in the generic kernels; measured before the
    // tiles went through LDS).  But not so few that the longest group is still at work when the others are done: a CU
    // does about 8 tiles side by side.
    const int64_t work = std::max<int64_t>(1, all * L->cfg.n_kv_heads), wgs = exist * L->cfg.n_kv_heads;
    const int64_t waves = std::max((all + exist - 1) / std::max<int64_t>(1, exist), 8 * most * n_cus / work);
    // One more for the newest tokens, but for workgroups of one or two tiles that queue up, where the last wave takes them
    // with its tile (4000 documents of 3 keys, 8/8 heads x 32, 70 us with it, 60 without).
    const bool newest_wave = wgs <= n_cus || all > 2 * exist;
    // 128 channels, groups with one row in use of 16 (one branch per document, one query head per kv head) and few keys:
    // the matrix work for the other rows, and the registers (two waves per SIMD), cost more than the generic kernel's
    // loads as soon as workgroups queue up.  This / generic, 8/8 heads, documents of 3, 20, 60, 150 keys, us: 64 of
    // them 7 / 10, 8 / 14, 15 / 26, 24 / 53; 128 of them 9 / 12, 19 / 18, 38 / 36, 45 / 72; 4000 of them 267 / 228, 502 /
    // 452, 1073 / 960, 1297 / 2085.  (64 channels: 4000 of them 122 / 136, 186 / 275, 467 / 526, 806 / 1102.)  Two rows in
    // use: slower with a tile each of document and tail.
    int64_t rows = 0;  // (row, tile) pairs in use over G
    for (int32_t u = 0; u < n_units; ++u) rows += desc(u)[5] * (prefix_tiles(u) + tail_tiles(1));
    s.generic = D == 128 && ((2 * rows * G < 3 * all && all < 10 * exist && wgs > 3 * (int64_t)n_cus) ||
                             (2 * rows * G < 5 * all && all <= 2 * exist && wgs > 8 * (int64_t)n_cus));
    // The smallest steps, of one or two branches with 12 or more query heads and a tile or two, stay with the generic
    // kernels, whose bits they have always had, at a price: 8.5 .. 12.3 us in two launches, 7.1 .. 8.0 in this kernel (16/1, 14/1,
    // 12/1 and 32/2 heads, 3 .. 20 keys).
    const int64_t calls = (int64_t)(L->live_ptr[t + 1] - L->live_ptr[t]) * L->cfg.n_q_heads;
    s.generic |= D == 128 && std::min(s.per_group, L->max_rows[t]) * G >= 12 && most <= 2 && calls <= 32;
    int64_t n_waves = std::max<int64_t>(1, std::min<int64_t>({hpd_f32_max_waves(D), most + newest_wave, waves + newest_wave}));
    // Workgroups that are at work at once: by registers (24, 16 and 8 waves on a CU), by LDS.
    auto at_once = [&](int64_t w) -> int64_t {
      const int64_t by_waves = std::max<int64_t>(1, (D == 32 ? 24 : D == 64 ? 16 : 8) / w);
      return (int64_t)n_cus * std::min<int64_t>(by_waves, 163840 / ((w * 32 + HPD_F32_ROWS) * D * (int64_t)sizeof(float)));
    };
    // Where they have room, three or four waves also for one or two tiles: they share the rotation of the query and the
    // merge (498 documents of up to 5 keys, 8/2 heads x 32, 15.1 us with one wave, 12.1 with two, 10.3 with four; but 682
    // workgroups with 128 channels, three of which fit a CU with two waves, 15.9 with two, 21.2 with three).  Where short
    // workgroups queue up, two or three tiles a wave: 3739 documents of up to 54 keys, 10/2 heads x 64, 91.8 us with five
    // waves, 58.6 with four, 49.2 with two.  Over 2000 batches 1.04 times the speed without these two rules in the mean,
    // 11 slower by more than 3 %, none by more than 7 %.
    if (n_waves < 4) {
      while (n_waves < 4 && 4 * wgs <= 3 * at_once(n_waves + 1)) ++n_waves;
    } else if (wgs > 2 * at_once(n_waves) && all <= 6 * exist && most * exist <= 2 * all && waves * exist < all + exist) {
      n_waves = std::max<int64_t>(2, (2 * all + 5 * exist - 1) / (5 * exist));
    }
    s.waves = (int32_t)n_waves;
  }
}

// The steps that run attn_dense_kernel (hpd_attn_dense.hip).  Against the kernel with loader waves it has the faster
// loop for many rows (four waves that load and compute, two or three workgroups per CU), and the start and end of a workgroup under
// another's work; but it reads the prefix once per 128 rows, keeps fewer bytes in flight, and a wave without rows idles where
// the other kernel gives it a share of the keys.  Which one is faster depends on how the units' rows divide, on their
// lengths and on how many workgroups there are, so both are estimated from the units: the time of a workgroup (start, blocks
// of the prefix, tail tiles), all of them over the places that the CUs have for them, and half of the longest for the end of
// the launch.
// The constants are microseconds of an MI355X, fitted to 3200 random batches that ran both kernels, and rounded; in the ratio
// of the two the estimate is off by 17 % (one sigma), so this kernel runs where it promises more.  A tenth is enough where
// four of five waves have rows and, under the literal mask, there is more than a workgroup per CU and few branches have ended
// (their tiles are masked key by key).  Elsewhere it has to promise a bit more than half of the time, under the literal mask
// three quarters: with the tenth there, about 300 more of the 3200 batches would run it under the block mask, 1.37 times as
// fast in the mean, but one in ten of them slower, down to 0.70.  And a launch estimated at 20 us or less is latency in either kernel.
// Measured over 2800 other batches for which the rule takes it (4 .. 400 branches, 1 .. 6 documents of up to 4000 tokens, 1 ..
// 160 prompts, even, ragged and with branches that end, up to 256 steps, contiguous and paged tails, either mask; two workgroups
// per CU in every launch, as for the fit: what the third adds from 512 workgroups on is left as margin): 1.41 times
// the speed in the mean, up to 3.28; 26 of them slower, 14 by more than 3 %, the slowest 63 us instead of 52.
void plan_dense(hpd_layout* L, int32_t n_cus) {
  const int32_t Hkv = L->cfg.n_kv_heads, Gr = L->cfg.n_q_heads / Hkv;
  if (L->cfg.dtype != HPD_BF16 || L->cfg.head_dim != 128 || Gr > 8) return;
  const int32_t G = Gr <= 2 ? Gr : Gr <= 4 ? 4 : 8, BPB = 32 / G;  // rows per branch, branches per row block
  const bool paper = paper_mode(L);
  L->dense_steps.assign(L->T, 0);
  L->dense_workgroups.assign(L->T, 0);
  auto ceil_div = [](int32_t a, int32_t b) { return (a + b - 1) / b; };
  for (int32_t t = 0; t < L->T; ++t) {
    const int32_t u0 = paper ? L->punit_ptr[t] : L->unit_ptr[t], n_units = (paper ? L->punit_ptr[t + 1] : L->unit_ptr[t + 1]) - u0;
    const int32_t most = ceil_div((paper ? L->pmax_rows[t] : L->max_rows[t]) * G, 32);  // row blocks
    // (up to three row blocks are one workgroup of the other kernel's narrow shape)
    if (n_units == 0 || most < 4) continue;
    const int32_t chunks = (t >> 3) + 1, newest = (t & 7) + 1, fmt = newest <= 1 ? 0 : newest <= 2 ? 1 : newest <= 4 ? 2 : 3;
    const int32_t lg_new = std::max(fmt, G == 8 ? 3 : G == 4 ? 2 : G == 2 ? 1 : 0);  // positions of a wave's own tiles in the newest chunk
    const int32_t rg_wide = ceil_div(most, 6), rg_dense = ceil_div(most, 4);
    const bool narrow = (int64_t)n_units * Hkv * rg_wide >= 2 * (int64_t)n_cus && most <= 6;
    const int32_t rg_old = narrow ? ceil_div(most, 3) : rg_wide;
    double sum_old = 0, sum = 0, longest_old = 0, longest = 0;  // us
    double bytes = 0;  // that the launch cannot do without
    int64_t blocks = 0, wgs = 0;  // row blocks, workgroups (of 4 waves for them)
    int64_t seen = 0, rows = 0;   // branches whose tails are seen, live ones
    for (int32_t u = u0; u < u0 + n_units; ++u) {
      const int32_t* d = paper ? L->punit_desc.data() + (size_t)u * 16 : L->unit_desc.data() + (size_t)u * 8;
      const int32_t nb = d[5], nblk = ceil_div(nb * G, 32), keys = paper ? d[8] : nb;  // keys: branches whose tails are seen
      const int32_t prefix = ceil_div(d[1], 32) + (paper ? d[3] : ceil_div(d[3], 32));
      seen += keys;
      rows += nb;
      bytes += 512. * Hkv * (32. * prefix + (double)keys * (t + 1));
      // literal mask: branches that the rows up to row block `last` see
      auto branches_seen = [&](int32_t last) { return (int32_t)std::ceil(keys * std::min(1.0, (double)last / nblk)); };
      // the kernel with loader waves; 0.7 us for each of the workgroups that the unit has no rows for: they are counted,
      // not walked (one document of 200 000 branches and 20 000 of one: 0.55 s of a build of 0.6)
      const int32_t per_old = ceil_div(nblk, rg_old), n_old = ceil_div(nblk, per_old);
      sum_old += 0.7 * Hkv * (rg_old - n_old);
      for (int32_t r = 0; r < n_old; ++r) {
        const int32_t h = std::min(per_old, nblk - r * per_old);
        const int32_t kg = narrow ? (h == 1 ? 3 : 1) : h == 1 ? 4 : h <= 3 ? 2 : 1;  // key groups
        double tiles, x = 9 + prefix * (h > (narrow ? 1 : 4) ? 0.77 : 0.55);
        if (paper) {
          tiles = ceil_div(branches_seen(r * per_old + h), 4) * chunks;
          x += 1.23 * tiles / kg;
        } else {
          const int32_t n = std::min(nb - r * per_old * BPB, h * BPB);
          tiles = ceil_div(n, 4) * (chunks - 1) + ceil_div(n, 32 >> fmt);
          x += 2.9 * tiles / (h * kg);
        }
        if (narrow) x += 0.45 * tiles;
        longest_old = std::max(longest_old, x);
        sum_old += x * Hkv;
      }
      const int32_t n_rg = ceil_div(nblk, 4), per = ceil_div(nblk, n_rg), n_used = ceil_div(nblk, per);
      for (int32_t r = 0; r < n_used; ++r) {
        double tail;
        if (paper) {
          const int32_t n = branches_seen(std::min(r * per + per, nblk));
          tail = 1.6 * (fmt < 3 ? ceil_div(n, 4) * (chunks - 1) + ceil_div(n, 32 >> fmt) : ceil_div(n, 4) * chunks);
        } else {
          tail = 2.2 * (ceil_div(std::min(BPB, nb), 4) * (chunks - 1) + ceil_div(BPB, 32 >> lg_new));
        }
        const double x = (paper ? 15 : 10) + 0.77 * prefix + tail;
        longest = std::max(longest, x);
        sum += x * Hkv;
      }
      wgs += (int64_t)Hkv * n_used;
      blocks += (int64_t)Hkv * nblk;
      sum += 0.5 * Hkv * (rg_dense - n_rg);
    }
    const int32_t slots = narrow ? 2 * n_cus : n_cus;
    const double old_us = sum_old > longest_old * slots ? sum_old / slots + 0.5 * longest_old : longest_old;
    const double us = std::max(0.255e-6 * bytes,  // 3.9 TB/s is all that it streams
                               wgs <= n_cus ? 0.75 * longest : wgs <= 2 * n_cus ? longest : sum / (2 * n_cus) + 0.5 * longest);
    const bool close = 5 * blocks >= 4 * (4 * wgs) && (!paper || (5 * seen <= 6 * rows && wgs > n_cus));
    L->dense_workgroups[t] = (int32_t)std::min<int64_t>(wgs, std::numeric_limits<int32_t>::max());
    L->dense_steps[t] = old_us > 20 && us < (close ? 0.9 : paper ? 0.72 : 0.55) * old_us;
  }
}

// Row groups of attn_prefill_kernel, one record of 8 words each: the unit's descriptor with the row group's first token
// in its last word.  The later a row group lies in its segment, the more keys it has.
//  * Few row groups (up to 16 per CU; 2 or 3 run at a time): the longest of all first.  Times the speed of a grid of (unit, row
//    groups of the longest segment), unit after unit / longest first, geometric means of random batches with that many row
//    groups: 512-1000 1.25 / 1.33, 1000-2000 1.21 / 1.30, 2000-4000 1.24 / 1.26.
//  * Up to two per CU: all start at once, the second half where the first one's workgroups are, in their order.  The shortest
//    join each other - the longest of them the shortest -, and the longest have a CU to themselves: longest first 1.05-1.17, so
//    1.14-1.22 (280 row groups of one prompt of 115 + 345 tokens, literal mask: 17.4 us, so 16.2).  No lanes (below): dealt to
//    them, the row groups of a few units load some XCDs twice as much as others, and the records that fill up start in front of row
//    groups.  Against the same grid, up to 256 | 256-512 row groups, in lanes -> so: 1 kv head 1.06 -> 1.07 | 1.21 -> 1.35, 2: 1.07
//    -> 1.07 | 1.22 -> 1.26, 3: 1.08 -> 1.09 | 1.18 -> 1.22, 4: 1.09 -> 1.09 | 1.25 -> 1.24, 5 to 7: 1.09 -> 1.11 | 1.26 -> 1.29, 12:
//    1.14 -> 1.15 | 1.32 -> 1.35; 84 documents of 59 tokens, 12/3 heads, 12.6 -> 8.9 us (grid 9.6).
//  * More than 16: unit after unit, so that the row groups that run at a time read the same keys out of the L2 (all of 28000 row
//    groups longest first: 3349 us, unit after unit 2078); the heaviest unit first, in each the longest row group first.
// Workgroup b runs on XCD b % 8, and takes kv head b % Hkv of record b / Hkv: with more than two row groups per CU and a number of kv
// heads that is no multiple of 8 the records are dealt to 8 / gcd(8, Hkv) lanes in turn, and the row groups of a unit stay in one
// lane, hence those of a (unit, kv head) on one XCD.
// More than 16 row groups per CU are written straight to their places; collected and copied twice, they made building slower by up to a
// third.  What is left is one pass over the memory (ms of hpd_build_layout, without the list -> collected -> so: 256 x 2 x 4000
// tokens, 64/8 heads 3.97 -> 4.52 -> 4.18; 1000 x 4 x 500, 32/8 heads 1.20 -> 1.57 -> 1.24; that one has the sorting of the documents
// once instead of once per step in its favour).
void list_prefill_groups(hpd_layout* L, int32_t n_cus) {
  const int32_t Gr = L->cfg.n_q_heads / L->cfg.n_kv_heads, Hkv = L->cfg.n_kv_heads;
  if (L->cfg.dtype != HPD_BF16 || L->cfg.head_dim != 128 || Gr > 8) return;
  const int32_t per = HPD_PREFILL_ROWS / (Gr <= 2 ? Gr : Gr <= 4 ? 4 : 8);  // tokens per row group
  const bool list = L->cfg.mask_mode == HPD_MASK_PAPER;
  const size_t n_units = L->funit_desc.size() / 8;
  auto ceil_div = [](int32_t a, int32_t b) { return (a + b - 1) / b; };
  auto unit = [&](size_t u) { return L->funit_desc.data() + u * 8; };
  auto groups = [&](size_t u) { return ceil_div(unit(u)[5], per); };
  auto seen_in_full = [&](size_t u) { return list ? unit(u)[1] : ceil_div(unit(u)[1], HPD_KEY_BLOCK); };  // blocks
  int64_t all = 0;
  for (size_t u = 0; u < n_units; ++u) all += groups(u);
  L->prefill_groups = all * Hkv;
  struct Lane { int64_t load = 0, n = 0; };
  std::vector<Lane> lanes(L->prefill_groups <= 2 * (int64_t)n_cus ? 1 : 8 / std::gcd(8, Hkv));
  std::vector<uint8_t> lane_of(lanes.size() > 1 ? n_units : 0);
  for (size_t u = 0; u < n_units; ++u) {
    size_t to = 0;
    if (!lane_of.empty()) {
      for (size_t i = 1; i < lanes.size(); ++i)
        if (lanes[i].load < lanes[to].load) to = i;
      lane_of[u] = (uint8_t)to;
      // the blocks of all row groups; a row group's start and end take as long as about 6
      const int64_t m = groups(u) - 1;  // full ones: 1, 1, 2, 2 .. own blocks with 16 tokens each, else multiples of per / 32
      lanes[to].load += (m + 1) * (seen_in_full(u) + 6) + ceil_div(unit(u)[5], HPD_KEY_BLOCK) +
                        (per < HPD_KEY_BLOCK ? (m + 1) * (m + 1) / 4 : per / HPD_KEY_BLOCK * (m * (m + 1) / 2));
    }
    lanes[to].n += groups(u);
  }
  int64_t most = 0;
  for (const Lane& l : lanes) most = std::max(most, l.n);
  L->fgroup_desc.resize(most * lanes.size() * 8);
  auto put = [&](size_t lane, size_t k, size_t u, int32_t tok) {
    int32_t* o = L->fgroup_desc.data() + (k * lanes.size() + lane) * 8;
    std::copy_n(unit(u), 7, o);
    o[7] = tok;
  };
  auto lane = [&](size_t u) -> size_t { return lane_of.empty() ? 0 : lane_of[u]; };
  if (L->prefill_groups > 16 * (int64_t)n_cus) {  // many: every record straight to its place
    std::vector<int32_t*> next(lanes.size());
    for (size_t i = 0; i < lanes.size(); ++i) next[i] = L->fgroup_desc.data() + i * 8;
    for (size_t u = 0; u < n_units; ++u) {
      int32_t d[8], *o = next[lane(u)];
      std::copy_n(unit(u), 8, d);
      for (d[7] = (groups(u) - 1) * per; d[7] >= 0; d[7] -= per, o += lanes.size() * 8) std::memcpy(o, d, sizeof(d));
      next[lane(u)] = o;
    }
    return;
  }
  struct Item { int32_t blocks, unit, tok; };
  std::vector<Item> items;
  for (size_t i = 0; i < lanes.size(); ++i) {
    items.clear();
    for (size_t u = 0; u < n_units; ++u)
      for (int32_t t = (groups(u) - 1) * per; t >= 0 && lane(u) == i; t -= per)
        items.push_back({seen_in_full(u) + ceil_div(std::min(t + per, unit(u)[5]), HPD_KEY_BLOCK), (int32_t)u, t});
    std::stable_sort(items.begin(), items.end(), [](const Item& x, const Item& y) { return x.blocks > y.blocks; });
    const size_t row = (size_t)n_cus / lanes.size() / Hkv, n = items.size();  // records of a lane for one workgroup on every CU
    if (n > row && n <= 2 * row) {
      std::reverse(items.begin() + row, items.end());
      std::rotate(items.begin(), items.begin() + (2 * row - n), items.begin() + row);
    }
    for (size_t k = 0; k < n; ++k) put(i, k, items[k].unit, items[k].tok);
  }
}

// Copies a host vector into the device int arena and returns its device address.
struct IntArena {
  std::vector<int32_t> host;
  std::vector<size_t> offs;
  size_t add(const std::vector<int32_t>& v) {
    size_t o = host.size();
    host.insert(host.end(), v.begin(), v.end());
    // keep every table 16-byte aligned
    while (host.size() % 4) host.push_back(0);
    if (v.empty()) { host.insert(host.end(), 4, 0); }
    return o;
  }
};

}  // namespace

// Three workgroups per CU where all of them run at a time that two per CU would leave to a second round, and from more than
// four per CU on; between them the third would only leave a longer last round.  Time with two per CU over time with three,
// geometric means of 3220 random batches, block mask | literal mask: up to 256 workgroups 0.89 | 0.88, 256-512 0.97 | 0.96, 512-768
// 1.12 | 1.19, 768-1024 0.97 | 0.99, 1024-1600 1.05 | 1.07, 1600-3000 1.07 | 1.09, more 1.11 | 1.10.  In the first of these ranges the
// grid has to have few workgroups without rows, which upset where the others go: the figures are for up to 1.25 times as many in
// the grid; with more 1.04 | 1.03, in a quarter of them below 0.97, down to 0.84.
hpd_dense_launch hpd_plan_dense_launch(const hpd_layout* L, int32_t step) {
  const bool paper = paper_mode(L);
  const int32_t Hkv = L->cfg.n_kv_heads, Gr = L->cfg.n_q_heads / Hkv, G = Gr <= 2 ? Gr : Gr <= 4 ? 4 : 8;
  const int32_t n_units = paper ? L->punit_ptr[step + 1] - L->punit_ptr[step] : L->unit_ptr[step + 1] - L->unit_ptr[step];
  hpd_dense_launch d;
  d.n_groups = n_units * Hkv;
  d.row_groups = ((paper ? L->pmax_rows[step] : L->max_rows[step]) * G + HPD_DENSE_ROWS - 1) / HPD_DENSE_ROWS;
  d.grid = ((int64_t)d.n_groups + 7) / 8 * 8 * d.row_groups;
  const int64_t cu = L->n_cus, workgroups = L->dense_workgroups[step];
  d.per_cu = (workgroups > 2 * cu && workgroups <= 3 * cu && 4 * d.grid <= 5 * workgroups) || workgroups > 4 * cu ? 3 : 2;
  d.at_once = workgroups <= 3 * cu;
  return d;
}

extern "C" {

const char* hpd_status_string(int status) {
  switch (status) {
    case HPD_OK: return "ok";
    case HPD_E_INVALID: return "invalid argument";
    case HPD_E_OVERFLOW: return "integer overflow in positions or offsets";
    case HPD_E_UNSUPPORTED: return "unsupported dtype, head_dim or mode";
    case HPD_E_HIP: return g_hip_text.c_str();
    case HPD_E_NOMEM: return "out of host memory";
    case HPD_E_CAPACITY: return "the layout exceeds the fixed scratch memory of the allocation-free call";
    default: return "unknown status";
  }
}

int hpd_build_layout(const hpd_config* cfg, int32_t n_prompts, const int32_t* header_len,
                     const int32_t* doc_ptr, const int32_t* doc_len, const int32_t* branch_ptr,
                     const int32_t* branch_len, const int32_t* attr_len, void* stream,
                     hpd_layout** out) {
  if (!out) return HPD_E_INVALID;
  int rc = validate_config(cfg);
  if (rc != HPD_OK) return rc;
  if (n_prompts < 1 || !header_len || !doc_ptr || !doc_len || !branch_ptr) return HPD_E_INVALID;
  if (cfg->pos_mode == HPD_POS_PAPER_GAP && !attr_len) return HPD_E_INVALID;
  const int32_t P = n_prompts;
  const int32_t T = cfg->max_new;
  if (doc_ptr[0] != 0) return HPD_E_INVALID;
  for (int32_t p = 0; p < P; ++p) {
    if (header_len[p] < 0) return HPD_E_INVALID;
    if (doc_ptr[p + 1] < doc_ptr[p]) return HPD_E_INVALID;
  }
  const int32_t n_docs = doc_ptr[P];
  if (branch_ptr[0] != 0) return HPD_E_INVALID;
  for (int32_t d = 0; d < n_docs; ++d) {
    if (doc_len[d] < 1) return HPD_E_INVALID;
    if (branch_ptr[d + 1] < branch_ptr[d]) return HPD_E_INVALID;
  }
  const int32_t B = branch_ptr[n_docs];
  for (int32_t b = 0; b < B; ++b) {
    if (branch_len && (branch_len[b] < 1 || branch_len[b] > T)) return HPD_E_INVALID;
    if (cfg->pos_mode == HPD_POS_PAPER_GAP && attr_len[b] < 1) return HPD_E_INVALID;
  }
  if ((int64_t)B * T > (int64_t)1 << 40) return HPD_E_OVERFLOW;

  hpd_layout* L = new (std::nothrow) hpd_layout();
  if (!L) return HPD_E_NOMEM;
  try {
    L->cfg = *cfg;
    const bool paper = cfg->mask_mode == HPD_MASK_PAPER;
    // (under the literal mask every prompt has a third kind of segment: its attribute names)
    L->P = P; L->n_docs = n_docs; L->B = B; L->T = T; L->n_seg = P + n_docs + (paper ? P : 0);
    const int32_t n_seg = L->n_seg;
    L->seg_off.assign(n_seg, 0); L->seg_len.assign(n_seg, 0); L->seg_pos0.assign(n_seg, 0);
    L->seg_raw_off.assign(n_seg + 1, 0); L->raw_seg.assign(n_seg, 0);
    L->doc_prompt.assign(n_docs, 0);
    L->branch_doc.assign(B, 0); L->branch_base_pos.assign(B, 0); L->branch_len.assign(B, T);
    if (branch_len) std::copy(branch_len, branch_len + B, L->branch_len.begin());
    if (paper) { L->skel_cum.assign(B, 0); L->skel_seg_off.assign(P, 0); }
    L->prompt_doc_ptr.assign(doc_ptr, doc_ptr + P + 1);
    L->doc_branch_ptr.assign(branch_ptr, branch_ptr + n_docs + 1);
    for (int32_t d = 0; d < n_docs; ++d)
      L->max_doc_branches = std::max(L->max_doc_branches, branch_ptr[d + 1] - branch_ptr[d]);
    L->prompt_branch_ptr.resize(P + 1);
    for (int32_t p = 0; p <= P; ++p) L->prompt_branch_ptr[p] = branch_ptr[doc_ptr[p]];

    // ---- segments: pool slots (each segment starts on a HPD_KEY_BLOCK boundary), raw
    //      token order [header | doc_0 | doc_1 ...] per prompt, position of first token
    int64_t slot = 0, raw = 0, max_pos = 0;
    int32_t ri = 0;
    for (int32_t p = 0; p < P; ++p) {
      const int64_t H = header_len[p];
      L->seg_off[p] = (int32_t)slot; L->seg_len[p] = (int32_t)H; L->seg_pos0[p] = 0;
      L->seg_raw_off[ri] = (int32_t)raw; L->raw_seg[ri] = p; ++ri;
      slot += round_up(H, HPD_KEY_BLOCK); raw += H;
      int64_t run_pos = H;  // paper-gap mode: ordinary increasing positions across documents
      for (int32_t d = doc_ptr[p]; d < doc_ptr[p + 1]; ++d) {
        const int64_t Ld = doc_len[d];
        const int32_t sid = P + d;
        L->doc_prompt[d] = p;
        L->seg_off[sid] = (int32_t)slot; L->seg_len[sid] = (int32_t)Ld;
        const int64_t pos0 = (cfg->pos_mode == HPD_POS_CONTIG) ? H : run_pos;
        L->seg_pos0[sid] = (int32_t)pos0;
        L->seg_raw_off[ri] = (int32_t)raw; L->raw_seg[ri] = sid; ++ri;
        slot += round_up(Ld, HPD_KEY_BLOCK); raw += Ld; run_pos += Ld;
        max_pos = std::max(max_pos, pos0 + Ld - 1);
        if (slot > std::numeric_limits<int32_t>::max() - 4096 || run_pos > (1 << 30)) {
          delete L; return HPD_E_OVERFLOW;
        }
      }
      // ---- branches of this prompt: base position = position of the token they continue from
      if (cfg->pos_mode == HPD_POS_CONTIG) {
        for (int32_t d = doc_ptr[p]; d < doc_ptr[p + 1]; ++d)
          for (int32_t b = branch_ptr[d]; b < branch_ptr[d + 1]; ++b) {
            L->branch_doc[b] = d;
            L->branch_base_pos[b] = (int32_t)(H + doc_len[d] - 1);
          }
      } else {
        // Algorithm 2 over s = cat(prompt, a_1..a_N): attribute n keeps its ordinary
        // position plus n*K_max; a branch continues from its attribute's last token.
        int64_t idx = run_pos;  // index in s of the next skeleton token
        int64_t offset = 0;
        int32_t cum = 0;
        if (paper) L->skel_off.push_back((int32_t)L->skel_pos.size());
        for (int32_t d = doc_ptr[p]; d < doc_ptr[p + 1]; ++d)
          for (int32_t b = branch_ptr[d]; b < branch_ptr[d + 1]; ++b) {
            L->branch_doc[b] = d;
            const int64_t end = idx + attr_len[b] - 1;
            const int64_t bp = end + offset;
            if (bp + T > (1 << 30)) { delete L; return HPD_E_OVERFLOW; }
            L->branch_base_pos[b] = (int32_t)bp;
            if (paper) {
              for (int64_t i = idx; i <= end; ++i) L->skel_pos.push_back((int32_t)(i + offset));
              cum += attr_len[b];
              L->skel_cum[b] = cum;
            }
            idx = end + 1;
            offset += T;
          }
        if (paper) {
          // the skeleton segment of the prompt: after its documents in the input order
          const int32_t sid = P + n_docs + p;
          L->seg_off[sid] = (int32_t)slot; L->seg_len[sid] = cum; L->seg_pos0[sid] = -1;
          L->skel_seg_off[p] = (int32_t)slot;
          L->seg_raw_off[ri] = (int32_t)raw; L->raw_seg[ri] = sid; ++ri;
          slot += round_up(cum, HPD_KEY_BLOCK); raw += cum;
          if (slot > std::numeric_limits<int32_t>::max() - 4096) { delete L; return HPD_E_OVERFLOW; }
        }
      }
    }
    if (paper) L->skel_off.push_back((int32_t)L->skel_pos.size());
    L->seg_raw_off[n_seg] = (int32_t)raw;
    L->n_prefix_tokens = raw;
    // slack of 128 slots so that a kernel tile that starts inside the last segment never
    // leaves the pool
    L->NP = round_up(slot, HPD_KEY_BLOCK) + 128;
    // the RoPE table covers the whole step budget of every branch, not only the steps branch_len
    // announces: the device-side pruning calls ignore branch_len and keep a branch alive until
    // its flag comes, at most up to step T - 1 (position base + T)
    for (int32_t b = 0; b < B; ++b)
      max_pos = std::max<int64_t>(max_pos, (int64_t)L->branch_base_pos[b] + T);
    if (max_pos > (1 << 30)) { delete L; return HPD_E_OVERFLOW; }
    L->max_pos = (int32_t)max_pos;

    // ---- per-step live lists (Section 4.3.4: a finished value is no longer fed)
    L->live_ptr.assign(T + 1, 0);
    for (int32_t t = 0; t < T; ++t) {
      int32_t n = 0;
      for (int32_t b = 0; b < B; ++b) n += L->branch_len[b] > t;
      L->live_ptr[t + 1] = L->live_ptr[t] + n;
    }
    L->total_live = L->live_ptr[T];
    L->live_branch.assign((size_t)L->total_live, 0);
    L->doc_live_ptr.assign((size_t)T * (n_docs + 1), 0);
    L->unit_ptr.assign(T + 1, 0);
    L->max_rows.assign(T, 0);
    // heaviest documents first: cost ~ keys streamed
    std::vector<int64_t> doc_keys(n_docs);
    for (int32_t d = 0; d < n_docs; ++d) doc_keys[d] = (int64_t)header_len[L->doc_prompt[d]] + doc_len[d];
    std::vector<int32_t> heaviest(n_docs);
    std::iota(heaviest.begin(), heaviest.end(), 0);
    std::stable_sort(heaviest.begin(), heaviest.end(), [&](int32_t a, int32_t b) { return doc_keys[a] > doc_keys[b]; });
    for (int32_t t = 0; t < T; ++t) {
      int32_t w = L->live_ptr[t];
      int32_t* dlp = &L->doc_live_ptr[(size_t)t * (n_docs + 1)];
      for (int32_t d = 0; d < n_docs; ++d) {
        dlp[d] = w - L->live_ptr[t];
        for (int32_t b = branch_ptr[d]; b < branch_ptr[d + 1]; ++b)
          if (L->branch_len[b] > t) L->live_branch[w++] = b;
        const int32_t nb = w - L->live_ptr[t] - dlp[d];
        L->max_rows[t] = std::max(L->max_rows[t], nb);
      }
      dlp[n_docs] = w - L->live_ptr[t];
      for (int32_t d : heaviest) {
        if (dlp[d + 1] == dlp[d]) continue;
        L->unit_doc.push_back(d);
        const int32_t p = L->doc_prompt[d];
        // all live branches of a document share one position in the contiguous mode
        int32_t pos = -1;
        if (cfg->pos_mode == HPD_POS_CONTIG) pos = L->seg_len[p] + L->seg_len[P + d] + t;
        // first branch id if the document's live branches are consecutive ids (no finished
        // branch in between): the kernels then need no lookup in the live list
        const int32_t nbl = dlp[d + 1] - dlp[d];
        const int32_t bf = L->live_branch[L->live_ptr[t] + dlp[d]];
        const int32_t bl = L->live_branch[L->live_ptr[t] + dlp[d + 1] - 1];
        const int32_t b_first = (bl - bf == nbl - 1) ? bf : -1;
        const int32_t desc[8] = {L->seg_off[p], L->seg_len[p], L->seg_off[P + d], L->seg_len[P + d],
                                 dlp[d], nbl, pos, b_first};
        L->unit_desc.insert(L->unit_desc.end(), desc, desc + 8);
      }
      L->unit_ptr[t + 1] = (int32_t)L->unit_doc.size();
    }
    L->total_units = (int64_t)L->unit_doc.size();
    int device = 0, n_cus = L->n_cus;
    if (!(cfg->flags & HPD_FLAG_HOST_ONLY) && hipGetDevice(&device) == hipSuccess)
      (void)hipDeviceGetAttribute(&n_cus, hipDeviceAttributeMultiprocessorCount, device);
    plan_f32(L, n_cus);

    // ---- paper-literal mask: the work unit is the prompt (its rows see every document and the
    //      tails of all earlier branches).  Document blocks of a prompt in stream order; per
    //      step the prompts with live branches, heaviest first.
    if (cfg->mask_mode == HPD_MASK_PAPER) {
      L->pblk_ptr.assign(P + 1, 0);
      for (int32_t p = 0; p < P; ++p) {
        for (int32_t d = doc_ptr[p]; d < doc_ptr[p + 1]; ++d)
          for (int32_t i = 0; i < doc_len[d]; i += HPD_KEY_BLOCK) {
            L->pblk.push_back(L->seg_off[P + d] + i);
            L->pblk.push_back(std::min<int32_t>(HPD_KEY_BLOCK, doc_len[d] - i));
          }
        L->pblk_docs.push_back((int32_t)(L->pblk.size() / 2) - L->pblk_ptr[p]);
        // then the blocks of the attribute names: a row keeps the names up to its own branch's,
        // so the second entry is 1000 + the index of the block's first name token
        for (int32_t i = 0; i < L->seg_len[P + n_docs + p]; i += HPD_KEY_BLOCK) {
          L->pblk.push_back(L->skel_seg_off[p] + i);
          L->pblk.push_back(1000 + i);
        }
        L->pblk_ptr[p + 1] = (int32_t)(L->pblk.size() / 2);
        L->max_prompt_branches = std::max(L->max_prompt_branches,
                                          L->prompt_branch_ptr[p + 1] - L->prompt_branch_ptr[p]);
      }
      L->punit_ptr.assign(T + 1, 0);
      L->pmax_rows.assign(T, 0);
      for (int32_t t = 0; t < T; ++t) {
        const int32_t* dlp = &L->doc_live_ptr[(size_t)t * (n_docs + 1)];
        std::vector<int32_t> units;
        for (int32_t p = 0; p < P; ++p)
          if (dlp[doc_ptr[p + 1]] > dlp[doc_ptr[p]]) units.push_back(p);
        std::stable_sort(units.begin(), units.end(), [&](int32_t x, int32_t y) {
          return L->pblk_ptr[x + 1] - L->pblk_ptr[x] > L->pblk_ptr[y + 1] - L->pblk_ptr[y];
        });
        for (int32_t p : units) {
          const int32_t r0 = dlp[doc_ptr[p]], nbl = dlp[doc_ptr[p + 1]] - r0;
          const int32_t bf = L->live_branch[L->live_ptr[t] + r0];
          const int32_t bl = L->live_branch[L->live_ptr[t] + r0 + nbl - 1];
          const int32_t pb0 = L->prompt_branch_ptr[p];
          const int32_t desc[16] = {L->seg_off[p], L->seg_len[p], L->pblk_ptr[p],
                                    L->pblk_ptr[p + 1] - L->pblk_ptr[p], r0, nbl, pb0,
                                    (bl - bf == nbl - 1) ? bf : -1, bl - pb0 + 1, L->pblk_docs[p], 0, 0, 0, 0, 0, 0};
          L->punit_desc.insert(L->punit_desc.end(), desc, desc + 16);
          L->pmax_rows[t] = std::max(L->pmax_rows[t], nbl);
        }
        L->punit_ptr[t + 1] = L->punit_ptr[t] + (int32_t)units.size();
      }
    }

    plan_dense(L, n_cus);

    // ---- attention of the prefix tokens (first inference step, block mask): a unit per
    //      non-empty header and per document, the most expensive (tokens x keys) first
    if (cfg->mask_mode == HPD_MASK_BLOCK) {
      std::vector<int32_t> segs;
      for (int32_t sid = 0; sid < n_seg; ++sid)
        if (L->seg_len[sid] > 0) segs.push_back(sid);
      std::vector<int32_t> raw_of(n_seg);
      for (int32_t i = 0; i < n_seg; ++i) raw_of[L->raw_seg[i]] = L->seg_raw_off[i];
      auto cost = [&](int32_t sid) -> int64_t {
        const int64_t hl = sid < P ? 0 : L->seg_len[L->doc_prompt[sid - P]];
        return (int64_t)L->seg_len[sid] * (hl + L->seg_len[sid]);
      };
      std::stable_sort(segs.begin(), segs.end(), [&](int32_t x, int32_t y) { return cost(x) > cost(y); });
      for (int32_t sid : segs) {
        const int32_t p = sid < P ? sid : L->doc_prompt[sid - P];
        const int32_t desc[8] = {L->seg_off[p], sid < P ? 0 : L->seg_len[p], L->seg_off[sid], L->seg_len[sid],
                                 raw_of[sid], L->seg_len[sid], L->seg_pos0[sid], 0};
        L->funit_desc.insert(L->funit_desc.end(), desc, desc + 8);
        L->fmax_rows = std::max(L->fmax_rows, L->seg_len[sid]);
      }
    }

    // ---- the same under the literal mask: header, documents and attribute names of a prompt
    //      are one causal sequence.  A segment sees the earlier segments of its prompt in full -
    //      a list of their 32-key blocks (first pool slot, keys), of which every segment takes
    //      a prefix - and itself up to the query.  A unit per non-empty segment:
    //      {first list entry of the prompt, list blocks the segment sees, first slot, tokens,
    //       first token in q / out order, tokens, position ID of the first token or
    //       -(1 + first entry in skel_pos) for the names, 0}
    if (cfg->mask_mode == HPD_MASK_PAPER) {
      std::vector<int32_t> raw_of(n_seg), before(n_seg, 0), list0(n_seg, 0);
      for (int32_t i = 0; i < n_seg; ++i) raw_of[L->raw_seg[i]] = L->seg_raw_off[i];
      for (int32_t p = 0; p < P; ++p) {
        const int32_t base = (int32_t)(L->fblk.size() / 2);
        auto add = [&](int32_t sid, bool keys) {
          list0[sid] = base;
          before[sid] = (int32_t)(L->fblk.size() / 2) - base;
          for (int32_t i = 0; keys && i < L->seg_len[sid]; i += HPD_KEY_BLOCK) {
            L->fblk.push_back(L->seg_off[sid] + i);
            L->fblk.push_back(std::min<int32_t>(HPD_KEY_BLOCK, L->seg_len[sid] - i));
          }
        };
        add(p, true);
        for (int32_t d = doc_ptr[p]; d < doc_ptr[p + 1]; ++d) add(P + d, true);
        add(P + n_docs + p, false);  // nothing comes after the names
      }
      std::vector<int32_t> segs;
      for (int32_t sid = 0; sid < n_seg; ++sid)
        if (L->seg_len[sid] > 0) segs.push_back(sid);
      auto cost = [&](int32_t sid) -> int64_t {
        return (int64_t)L->seg_len[sid] * ((int64_t)before[sid] * HPD_KEY_BLOCK + L->seg_len[sid]);
      };
      std::stable_sort(segs.begin(), segs.end(), [&](int32_t x, int32_t y) { return cost(x) > cost(y); });
      for (int32_t sid : segs) {
        const bool names = sid >= P + n_docs;
        const int32_t desc[8] = {list0[sid], before[sid], L->seg_off[sid], L->seg_len[sid], raw_of[sid],
                                 L->seg_len[sid], names ? -(1 + L->skel_off[sid - P - n_docs]) : L->seg_pos0[sid], 0};
        L->funit_desc.insert(L->funit_desc.end(), desc, desc + 8);
        L->fmax_rows = std::max(L->fmax_rows, L->seg_len[sid]);
        L->fmax_list_blocks = std::max(L->fmax_list_blocks, before[sid]);
      }
    }

    list_prefill_groups(L, n_cus);

    // ---- for hpd_prefix_fill: which segment owns a 32-slot block of the pools, and where its
    //      first token sits in the input order
    {
      std::vector<int32_t> raw_of(n_seg);
      for (int32_t i = 0; i < n_seg; ++i) raw_of[L->raw_seg[i]] = L->seg_raw_off[i];
      L->fill_blk.assign((size_t)(L->NP / HPD_KEY_BLOCK) * 2, -1);
      for (int32_t sid = 0; sid < n_seg; ++sid)
        for (int32_t i = 0; i < L->seg_len[sid]; i += HPD_KEY_BLOCK) {
          const size_t b = (size_t)(L->seg_off[sid] + i) / HPD_KEY_BLOCK;
          L->fill_blk[2 * b] = sid;
          L->fill_blk[2 * b + 1] = raw_of[sid] + i;
        }
    }

    // ---- device-side pruning: what never changes, one record of 8 words per unit (document, or
    //      prompt under the literal mask), the units with the most keys first.  Documents:
    //      {hoff, Hlen, doff, Llen, first branch, end of branches, position of step 0 | -1, 0};
    //      prompts: {hoff, Hlen, first entry of the block list, its blocks, first branch, end of
    //      branches, document blocks of the list, 0}
    {
      const size_t nU = paper ? (size_t)P : (size_t)n_docs;
      std::vector<int32_t> order(nU);
      std::iota(order.begin(), order.end(), 0);
      std::stable_sort(order.begin(), order.end(), [&](int32_t x, int32_t y) {
        if (paper) return L->pblk_ptr[x + 1] - L->pblk_ptr[x] > L->pblk_ptr[y + 1] - L->pblk_ptr[y];
        return (int64_t)L->seg_len[L->doc_prompt[x]] + L->seg_len[L->P + x] >
               (int64_t)L->seg_len[L->doc_prompt[y]] + L->seg_len[L->P + y];
      });
      L->dyn_fixed.assign(nU * 8, 0);
      for (size_t u = 0; u < nU; ++u) {
        int32_t* o = L->dyn_fixed.data() + u * 8;
        if (paper) {
          const int32_t p = order[u];
          o[0] = L->seg_off[p]; o[1] = L->seg_len[p]; o[2] = L->pblk_ptr[p]; o[3] = L->pblk_ptr[p + 1] - L->pblk_ptr[p];
          o[4] = L->prompt_branch_ptr[p]; o[5] = L->prompt_branch_ptr[p + 1]; o[6] = L->pblk_docs[p];
        } else {
          const int32_t d = order[u], p = L->doc_prompt[d];
          o[0] = L->seg_off[p]; o[1] = L->seg_len[p]; o[2] = L->seg_off[L->P + d]; o[3] = L->seg_len[L->P + d];
          o[4] = L->doc_branch_ptr[d]; o[5] = L->doc_branch_ptr[d + 1];
          o[6] = L->cfg.pos_mode == HPD_POS_CONTIG ? L->seg_len[p] + L->seg_len[L->P + d] : -1;
        }
      }
    }

    // ---- RoPE table: angles in double, stored as float (cos, sin)
    const int32_t half = cfg->head_dim / 2;
    L->rope.resize((size_t)(L->max_pos + 1) * half * 2);
    std::vector<double> theta(half);
    for (int32_t i = 0; i < half; ++i)
      theta[i] = std::pow(cfg->rope_base, -2.0 * (double)i / (double)cfg->head_dim);
    for (int64_t pos = 0; pos <= L->max_pos; ++pos)
      for (int32_t i = 0; i < half; ++i) {
        const double a = (double)pos * theta[i];
        L->rope[((size_t)pos * half + i) * 2 + 0] = (float)std::cos(a);
        L->rope[((size_t)pos * half + i) * 2 + 1] = (float)std::sin(a);
      }
  } catch (const std::bad_alloc&) {
    delete L;
    return HPD_E_NOMEM;
  }

  if (!(cfg->flags & HPD_FLAG_HOST_ONLY)) {
    // ---- upload
    IntArena A;
    const size_t o_seg_off = A.add(L->seg_off), o_seg_len = A.add(L->seg_len),
                 o_seg_pos0 = A.add(L->seg_pos0), o_raw_off = A.add(L->seg_raw_off),
                 o_raw_seg = A.add(L->raw_seg), o_doc_prompt = A.add(L->doc_prompt),
                 o_branch_doc = A.add(L->branch_doc), o_base = A.add(L->branch_base_pos),
                 o_live_ptr = A.add(L->live_ptr), o_live_branch = A.add(L->live_branch),
                 o_dlp = A.add(L->doc_live_ptr), o_unit_ptr = A.add(L->unit_ptr),
                 o_unit_doc = A.add(L->unit_doc), o_unit_desc = A.add(L->unit_desc),
                 o_pdp = A.add(L->prompt_doc_ptr), o_pbp = A.add(L->prompt_branch_ptr),
                 o_blen = A.add(L->branch_len), o_pblk = A.add(L->pblk), o_pdesc = A.add(L->punit_desc),
                 o_fdesc = A.add(L->funit_desc), o_spos = A.add(L->skel_pos), o_soff = A.add(L->skel_off),
                 o_sseg = A.add(L->skel_seg_off), o_scum = A.add(L->skel_cum), o_fblk = A.add(L->fblk),
                 o_fill = A.add(L->fill_blk), o_dynfix = A.add(L->dyn_fixed), o_f32 = A.add(L->f32_groups);
    // (a long list goes behind the others as it is: a second transfer is 10 us, one more copy of it on the host more than that)
    const size_t n_fgrp = L->fgroup_desc.size() > 1 << 16 ? L->fgroup_desc.size() : 0;
    const size_t o_fgrp = n_fgrp ? A.host.size() : A.add(L->fgroup_desc);
    hipStream_t s = (hipStream_t)stream;
    hipError_t e = hipGetDevice(&L->device);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&L->n_cus, hipDeviceAttributeMultiprocessorCount, L->device);
    if (e == hipSuccess) e = hipMalloc(&L->d_ints, (A.host.size() + n_fgrp) * sizeof(int32_t));
    if (e == hipSuccess) e = hipMalloc(&L->d_rope, L->rope.size() * sizeof(float));
    if (e == hipSuccess)
      e = hipMemcpyAsync(L->d_ints, A.host.data(), A.host.size() * sizeof(int32_t),
                         hipMemcpyHostToDevice, s);
    if (e == hipSuccess && n_fgrp)
      e = hipMemcpyAsync((int32_t*)L->d_ints + o_fgrp, L->fgroup_desc.data(), n_fgrp * sizeof(int32_t),
                         hipMemcpyHostToDevice, s);
    if (e == hipSuccess)
      e = hipMemcpyAsync(L->d_rope, L->rope.data(), L->rope.size() * sizeof(float),
                         hipMemcpyHostToDevice, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) {
      if (L->d_ints) (void)hipFree(L->d_ints);
      if (L->d_rope) (void)hipFree(L->d_rope);
      delete L;
      return hip_fail(e);
    }
    const int32_t* base = (const int32_t*)L->d_ints;
    L->dev.seg_off = base + o_seg_off; L->dev.seg_len = base + o_seg_len;
    L->dev.seg_pos0 = base + o_seg_pos0; L->dev.seg_raw_off = base + o_raw_off;
    L->dev.raw_seg = base + o_raw_seg; L->dev.doc_prompt = base + o_doc_prompt;
    L->dev.branch_doc = base + o_branch_doc; L->dev.branch_base_pos = base + o_base;
    L->dev.live_ptr = base + o_live_ptr; L->dev.live_branch = base + o_live_branch;
    L->dev.doc_live_ptr = base + o_dlp; L->dev.unit_ptr = base + o_unit_ptr;
    L->dev.unit_doc = base + o_unit_doc; L->dev.unit_desc = base + o_unit_desc;
    L->dev.prompt_doc_ptr = base + o_pdp; L->dev.prompt_branch_ptr = base + o_pbp;
    L->dev.branch_len = base + o_blen; L->dev.pblk = base + o_pblk; L->dev.punit_desc = base + o_pdesc;
    L->dev.funit_desc = base + o_fdesc; L->dev.fblk = base + o_fblk;
    L->dev.fgroup_desc = base + o_fgrp;
    L->dev.fill_blk = base + o_fill; L->dev.f32_groups = base + o_f32;
    L->dyn_fixed_dev = const_cast<int32_t*>(base) + o_dynfix;
    L->dev.skel_pos = paper_mode(L) ? base + o_spos : nullptr; L->dev.skel_off = base + o_soff;
    L->dev.skel_seg_off = base + o_sseg; L->dev.skel_cum = base + o_scum;
    L->dev.rope = (const float2*)L->d_rope;
    L->on_device = true;
  }
  *out = L;
  return HPD_OK;
}

void hpd_layout_free(hpd_layout* L) {
  if (!L) return;
  if (L->d_dyn) (void)hipFree(L->d_dyn);
  if (L->d_ints) (void)hipFree(L->d_ints);
  if (L->d_rope) (void)hipFree(L->d_rope);
  delete L;
}

int hpd_layout_query(const hpd_layout* L, int32_t what, void* host_out, size_t bytes) {
  if (!L || !host_out) return HPD_E_INVALID;
  auto copy32 = [&](const std::vector<int32_t>& v, size_t n) -> int {
    if (bytes < n * sizeof(int32_t)) return HPD_E_INVALID;
    if (n) std::memcpy(host_out, v.data(), n * sizeof(int32_t));
    return HPD_OK;
  };
  const size_t eb = elem_bytes(L->cfg);
  switch (what) {
    case HPD_Q_COUNTS: {
      if (bytes < HPD_N_COUNTS * sizeof(int64_t)) return HPD_E_INVALID;
      int64_t c[HPD_N_COUNTS];
      c[HPD_C_N_PROMPTS] = L->P; c[HPD_C_N_DOCS] = L->n_docs; c[HPD_C_N_BRANCHES] = L->B;
      c[HPD_C_N_PREFIX_TOKENS] = L->n_prefix_tokens; c[HPD_C_N_PREFIX_SLOTS] = L->NP;
      c[HPD_C_N_TAIL_SLOTS] = (int64_t)L->B * L->T; c[HPD_C_MAX_POS] = L->max_pos;
      c[HPD_C_TOTAL_LIVE] = L->total_live;
      std::memcpy(host_out, c, sizeof(c));
      return HPD_OK;
    }
    case HPD_Q_POOL_BYTES: {
      if (bytes < 4 * sizeof(int64_t)) return HPD_E_INVALID;
      const int64_t per_slot = (int64_t)L->cfg.n_kv_heads * L->cfg.head_dim * (int64_t)eb;
      const int64_t tail_slots = L->dev.tail_pages ? ((int64_t)L->dev.n_pages << L->dev.page_shift)
                                                   : (int64_t)L->B * L->T;
      int64_t c[4] = {L->NP * per_slot, L->NP * per_slot, tail_slots * per_slot, tail_slots * per_slot};
      std::memcpy(host_out, c, sizeof(c));
      return HPD_OK;
    }
    case HPD_Q_N_LIVE: {
      if (bytes < (size_t)L->T * sizeof(int32_t)) return HPD_E_INVALID;
      int32_t* o = (int32_t*)host_out;
      for (int32_t t = 0; t < L->T; ++t) o[t] = L->live_ptr[t + 1] - L->live_ptr[t];
      return HPD_OK;
    }
    case HPD_Q_N_UNITS: {
      if (bytes < (size_t)L->T * sizeof(int32_t)) return HPD_E_INVALID;
      int32_t* o = (int32_t*)host_out;
      const std::vector<int32_t>& up = L->cfg.mask_mode == HPD_MASK_PAPER ? L->punit_ptr : L->unit_ptr;
      for (int32_t t = 0; t < L->T; ++t) o[t] = up[t + 1] - up[t];
      return HPD_OK;
    }
    case HPD_Q_LIVE_BRANCH: return copy32(L->live_branch, (size_t)L->total_live);
    case HPD_Q_BRANCH_BASE_POS: return copy32(L->branch_base_pos, (size_t)L->B);
    case HPD_Q_BRANCH_DOC: return copy32(L->branch_doc, (size_t)L->B);
    case HPD_Q_SEG_OFF: return copy32(L->seg_off, (size_t)L->n_seg);
    case HPD_Q_SEG_LEN: return copy32(L->seg_len, (size_t)L->n_seg);
    case HPD_Q_SEG_POS0: return copy32(L->seg_pos0, (size_t)L->n_seg);
    case HPD_Q_SEG_RAW_OFF: {
      if (bytes < (size_t)L->n_seg * sizeof(int32_t)) return HPD_E_INVALID;
      int32_t* o = (int32_t*)host_out;
      for (int32_t i = 0; i < L->n_seg; ++i) o[L->raw_seg[i]] = L->seg_raw_off[i];
      return HPD_OK;
    }
    default: return HPD_E_INVALID;
  }
}

int hpd_set_kernel_mode(hpd_layout* L, int32_t mode) {
  if (!L || mode < 0 || mode > 4) return HPD_E_INVALID;
  if (mode >= 2 && !hpd_stream_supported(L)) return HPD_E_UNSUPPORTED;
  L->kernel_mode = mode;
  return HPD_OK;
}

static int check_step(const hpd_layout* L, int32_t step) {
  if (!L) return HPD_E_INVALID;
  if (!L->on_device) return HPD_E_INVALID;
  if (step < 0 || step >= L->T) return HPD_E_INVALID;
  return HPD_OK;
}

int hpd_prefix_fill(const hpd_layout* L, const void* k_raw, const void* v_raw, void* k_prefix,
                    void* v_prefix, void* stream) {
  if (!L || !L->on_device || !k_prefix || !v_prefix) return HPD_E_INVALID;
  if (L->n_prefix_tokens == 0) return HPD_OK;
  if (!k_raw || !v_raw) return HPD_E_INVALID;
  HPD_HIP(hpd_launch_prefix_fill(L, k_raw, v_raw, k_prefix, v_prefix, (hipStream_t)stream));
  return HPD_OK;
}

int hpd_rope_positions(const hpd_layout* L, int32_t step, int32_t* pos_out, int32_t* n_live_out,
                       void* stream) {
  int rc = check_step(L, step);
  if (rc != HPD_OK) return rc;
  const int32_t n_live = L->live_ptr[step + 1] - L->live_ptr[step];
  if (n_live > 0 && !pos_out) return HPD_E_INVALID;
  if (n_live > 0) HPD_HIP(hpd_launch_positions(L, step, pos_out, (hipStream_t)stream));
  if (n_live_out) *n_live_out = n_live;
  return HPD_OK;
}

int hpd_kv_append(const hpd_layout* L, int32_t step, const void* k_new, const void* v_new,
                  void* k_tail, void* v_tail, int64_t* slot_out, void* stream) {
  int rc = check_step(L, step);
  if (rc != HPD_OK) return rc;
  const int32_t n_live = L->live_ptr[step + 1] - L->live_ptr[step];
  if (n_live == 0) return HPD_OK;
  if (!k_new || !v_new || !k_tail || !v_tail) return HPD_E_INVALID;
  HPD_HIP(hpd_launch_append(L, step, k_new, v_new, k_tail, v_tail, slot_out, (hipStream_t)stream));
  return HPD_OK;
}

// The generic kernel keeps one score per key in LDS.  The fp32 kernel does not, but it shares the
// limit: whether a call is taken must not hang on the pools' alignment or on the kernel mode.
static bool too_many_keys(const hpd_layout* L, int32_t step) { return hpd_generic_max_keys(L, step) > 15000; }

int hpd_decode_attention(const hpd_layout* L, int32_t step, const void* q, const void* k_prefix,
                         const void* v_prefix, const void* k_tail, const void* v_tail, void* out,
                         void* stream) {
  int rc = check_step(L, step);
  if (rc != HPD_OK) return rc;
  const int32_t n_live = L->live_ptr[step + 1] - L->live_ptr[step];
  if (n_live == 0) return HPD_OK;
  if (!q || !k_prefix || !v_prefix || !k_tail || !v_tail || !out) return HPD_E_INVALID;
  const bool use_stream = L->kernel_mode >= 2 || (L->kernel_mode == 0 && hpd_stream_supported(L));
  if (use_stream) {
    HPD_HIP(hpd_launch_attention_stream(L, step, q, k_prefix, v_prefix, const_cast<void*>(k_tail),
                                        const_cast<void*>(v_tail), nullptr, nullptr, out,
                                        (hipStream_t)stream));
  } else {
    if (too_many_keys(L, step)) return HPD_E_UNSUPPORTED;
    if (hpd_use_attention_f32(L, step, k_prefix, v_prefix, k_tail)) {
      HPD_HIP(hpd_launch_attention_f32(L, step, q, k_prefix, v_prefix, const_cast<void*>(k_tail),
                                       const_cast<void*>(v_tail), nullptr, nullptr, out, (hipStream_t)stream));
      return HPD_OK;
    }
    HPD_HIP(hpd_launch_attention_generic(L, step, q, k_prefix, v_prefix, k_tail, v_tail, out,
                                         (hipStream_t)stream));
  }
  return HPD_OK;
}

int hpd_prefill_attention(const hpd_layout* L, const void* q, const void* k_prefix, const void* v_prefix,
                          void* out, void* stream) {
  if (!L || !L->on_device) return HPD_E_INVALID;
  if (L->n_prefix_tokens == 0) return HPD_OK;
  if (!q || !k_prefix || !v_prefix || !out) return HPD_E_INVALID;
  const bool paper = L->cfg.mask_mode == HPD_MASK_PAPER;
  // (the streaming kernel keeps the key counts of a unit's block list in LDS: 512 entries)
  if ((L->kernel_mode >= 2 || (L->kernel_mode == 0 && hpd_stream_supported(L))) &&
      (!paper || L->fmax_list_blocks <= 512)) {
    HPD_HIP(hpd_launch_prefill_stream(L, q, k_prefix, v_prefix, out, (hipStream_t)stream));
    return HPD_OK;
  }
  // the generic kernel keeps one score per key in LDS
  int64_t max_keys = 0;
  for (int32_t d = 0; d < L->n_docs; ++d)
    max_keys = std::max<int64_t>(max_keys, (int64_t)L->seg_len[L->doc_prompt[d]] + L->seg_len[L->P + d]);
  for (int32_t p = 0; p < L->P; ++p) max_keys = std::max<int64_t>(max_keys, L->seg_len[p]);
  if (paper)  // a prompt's last name token sees the whole prefix of the prompt
    for (int32_t p = 0; p < L->P; ++p) {
      int64_t keys = (int64_t)L->seg_len[p] + L->seg_len[L->P + L->n_docs + p];
      for (int32_t d = L->prompt_doc_ptr[p]; d < L->prompt_doc_ptr[p + 1]; ++d) keys += L->seg_len[L->P + d];
      max_keys = std::max(max_keys, keys);
    }
  if (max_keys > 15000) return HPD_E_UNSUPPORTED;
  HPD_HIP(hpd_launch_prefill_generic(L, q, k_prefix, v_prefix, out, (hipStream_t)stream));
  return HPD_OK;
}

int hpd_decode_step(const hpd_layout* L, int32_t step, const void* q, const void* k_new,
                    const void* v_new, const void* k_prefix, const void* v_prefix, void* k_tail,
                    void* v_tail, void* out, void* stream) {
  int rc = check_step(L, step);
  if (rc != HPD_OK) return rc;
  const int32_t n_live = L->live_ptr[step + 1] - L->live_ptr[step];
  if (n_live == 0) return HPD_OK;
  if (!q || !k_new || !v_new || !k_prefix || !v_prefix || !k_tail || !v_tail || !out)
    return HPD_E_INVALID;
  if (L->kernel_mode >= 2 || (L->kernel_mode == 0 && hpd_stream_supported(L))) {
    // one launch: the attention kernel rotates, stores and uses the new keys itself
    HPD_HIP(hpd_launch_attention_stream(L, step, q, k_prefix, v_prefix, k_tail, v_tail, k_new, v_new,
                                        out, (hipStream_t)stream));
    return HPD_OK;
  }
  if (too_many_keys(L, step)) return HPD_E_UNSUPPORTED;  // before anything is appended
  if (hpd_use_attention_f32(L, step, k_prefix, v_prefix, k_tail)) {
    HPD_HIP(hpd_launch_attention_f32(L, step, q, k_prefix, v_prefix, k_tail, v_tail, k_new, v_new, out,
                                     (hipStream_t)stream));
    return HPD_OK;
  }
  HPD_HIP(hpd_launch_append(L, step, k_new, v_new, k_tail, v_tail, nullptr, (hipStream_t)stream));
  HPD_HIP(hpd_launch_attention_generic(L, step, q, k_prefix, v_prefix, k_tail, v_tail, out, (hipStream_t)stream));
  return HPD_OK;
}

int hpd_expand_mask(const hpd_layout* L, int32_t prompt, int32_t step_hi, uint8_t* mask_out,
                    int32_t* s_out, void* stream) {
  if (!L || !L->on_device || !s_out) return HPD_E_INVALID;
  if (prompt < 0 || prompt >= L->P || step_hi < -1 || step_hi >= L->T) return HPD_E_INVALID;
  // token descriptors in memory order: (kind, document, branch, step | position for the
  // paper-literal mask);  kind 0 header, 1 document, 2 branch token
  const bool paper = L->cfg.mask_mode == HPD_MASK_PAPER;
  std::vector<int32_t> desc;
  const int32_t H = L->seg_len[prompt];
  for (int32_t i = 0; i < H; ++i) { desc.insert(desc.end(), {0, -1, -1, paper ? i : -1}); }
  int32_t d0 = -1, d1 = -1;
  for (int32_t d = 0; d < L->n_docs; ++d)
    if (L->doc_prompt[d] == prompt) { if (d0 < 0) d0 = d; d1 = d + 1; }
  for (int32_t d = d0; d >= 0 && d < d1; ++d)
    for (int32_t i = 0; i < L->seg_len[L->P + d]; ++i)
      desc.insert(desc.end(), {1, d, -1, paper ? L->seg_pos0[L->P + d] + i : -1});
  if (paper)  // the attribute names, fed with the prompt (kind 3)
    for (int32_t i = L->skel_off[prompt]; i < L->skel_off[prompt + 1]; ++i)
      desc.insert(desc.end(), {3, -1, -1, L->skel_pos[i]});
  for (int32_t t = 0; t <= step_hi; ++t)
    for (int32_t r = L->live_ptr[t]; r < L->live_ptr[t + 1]; ++r) {
      const int32_t b = L->live_branch[r];
      const int32_t d = L->branch_doc[b];
      if (L->doc_prompt[d] == prompt)
        desc.insert(desc.end(), {2, d, b, paper ? L->branch_base_pos[b] + 1 + t : t});
    }
  const int64_t S = (int64_t)desc.size() / 4;
  if (S > 46000) return HPD_E_OVERFLOW;
  *s_out = (int32_t)S;
  if (!mask_out || S == 0) return HPD_OK;
  int32_t* d_desc = nullptr;
  hipStream_t s = (hipStream_t)stream;
  HPD_HIP(hipMalloc((void**)&d_desc, desc.size() * sizeof(int32_t)));
  hipError_t e = hipMemcpyAsync(d_desc, desc.data(), desc.size() * sizeof(int32_t),
                                hipMemcpyHostToDevice, s);
  if (e == hipSuccess) e = hpd_launch_expand_mask(d_desc, (int32_t)S, paper ? 1 : 0, mask_out, s);
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  (void)hipFree(d_desc);
  if (e != hipSuccess) return hip_fail(e);
  return HPD_OK;
}

static int dynamic_supported(const hpd_layout* L) {
  if (!L || !L->on_device) return HPD_E_INVALID;
  if (!hpd_stream_supported(L) || L->kernel_mode == 1 || L->B > 65536) return HPD_E_UNSUPPORTED;
  return HPD_OK;
}

// words of device-side pruning state a layout needs: desc [units * 8 | 16] (read and written 16
// bytes at a time), n_live [4], live [B], and for the literal mask len [B]; units = documents, or
// prompts under the literal mask
static size_t dynamic_state_words(const hpd_layout* L) {
  const bool paper = L->cfg.mask_mode == HPD_MASK_PAPER;
  const size_t nB = (size_t)L->B, nU = paper ? (size_t)L->P : (size_t)L->n_docs, dw = paper ? 16 : 8;
  return nU * dw + 4 + nB + (paper ? nB : 0) + 16;
}

// points the layout's state at `mem` (dynamic_state_words(L) words, 16-byte aligned)
static void dynamic_state_bind(hpd_layout* L, void* mem) {
  const bool paper = L->cfg.mask_mode == HPD_MASK_PAPER;
  const size_t nB = (size_t)L->B, nU = paper ? (size_t)L->P : (size_t)L->n_docs, dw = paper ? 16 : 8;
  int32_t* w = (int32_t*)mem;
  L->dyn_desc = w; w += nU * dw;
  L->dyn_n_live = w; w += 4;
  L->dyn_live = w; w += nB;
  L->dyn_len = paper ? w : nullptr;
}

int hpd_dynamic_begin(hpd_layout* L, void* stream) {
  int rc = dynamic_supported(L);
  if (rc != HPD_OK) return rc;
  hipStream_t s = (hipStream_t)stream;
  if (!L->d_dyn) HPD_HIP(hipMalloc(&L->d_dyn, dynamic_state_words(L) * sizeof(int32_t)));
  dynamic_state_bind(L, L->d_dyn);
  L->dyn_next_step = 0;
  HPD_HIP(hpd_launch_dynamic_prune(L, 0, nullptr, s));
  return HPD_OK;
}

int hpd_dynamic_begin_static(hpd_layout* L, void* stream) {
  int rc = dynamic_supported(L);
  if (rc != HPD_OK) return rc;
  if (dynamic_state_words(L) * sizeof(int32_t) > (size_t)HPD_DYNAMIC_STATIC_MAX_BYTES) return HPD_E_CAPACITY;
  void* mem = nullptr;
  size_t bytes = 0;
  HPD_HIP(hpd_dynamic_scratch(L->device, &mem, &bytes));
  if (dynamic_state_words(L) * sizeof(int32_t) > bytes) return HPD_E_CAPACITY;
  dynamic_state_bind(L, mem);
  L->dyn_next_step = 0;
  HPD_HIP(hpd_launch_dynamic_prune(L, 0, nullptr, (hipStream_t)stream));
  return HPD_OK;
}

int hpd_dynamic_prune(hpd_layout* L, const uint8_t* finished, void* stream) {
  int rc = dynamic_supported(L);
  if (rc != HPD_OK) return rc;
  if (!L->dyn_live || !finished) return HPD_E_INVALID;
  if (L->dyn_next_step + 1 >= L->T) return HPD_E_INVALID;  // no step left to prune for
  L->dyn_next_step += 1;
  HPD_HIP(hpd_launch_dynamic_prune(L, L->dyn_next_step, finished, (hipStream_t)stream));
  return HPD_OK;
}

int hpd_dynamic_step(const hpd_layout* L, int32_t step, const void* q, const void* k_new,
                     const void* v_new, const void* k_prefix, const void* v_prefix, void* k_tail,
                     void* v_tail, void* out, void* stream) {
  int rc = dynamic_supported(L);
  if (rc != HPD_OK) return rc;
  if (!L->dyn_live || step != L->dyn_next_step) return HPD_E_INVALID;  // the state describes another step
  if (!q || !k_new || !v_new || !k_prefix || !v_prefix || !k_tail || !v_tail || !out) return HPD_E_INVALID;
  if (L->n_docs == 0) return HPD_OK;
  HPD_HIP(hpd_launch_attention_stream(L, step, q, k_prefix, v_prefix, k_tail, v_tail, k_new, v_new, out,
                                      (hipStream_t)stream, true));
  return HPD_OK;
}

int hpd_dynamic_state(const hpd_layout* L, const int32_t** live_branch, const int32_t** n_live) {
  if (!L || !L->dyn_live) return HPD_E_INVALID;
  if (live_branch) *live_branch = L->dyn_live;
  if (n_live) *n_live = L->dyn_n_live;
  return HPD_OK;
}

int hpd_dynamic_read(const hpd_layout* L, int32_t* live_host, int32_t capacity, int32_t* n_live_host,
                     void* stream) {
  if (!L || !L->dyn_live || !n_live_host || capacity < 0 || (capacity > 0 && !live_host)) return HPD_E_INVALID;
  hipStream_t s = (hipStream_t)stream;
  HPD_HIP(hipMemcpyAsync(n_live_host, L->dyn_n_live, sizeof(int32_t), hipMemcpyDeviceToHost, s));
  HPD_HIP(hipStreamSynchronize(s));
  const int32_t n = std::min(*n_live_host, capacity);
  if (n > 0) {
    HPD_HIP(hipMemcpyAsync(live_host, L->dyn_live, (size_t)n * sizeof(int32_t), hipMemcpyDeviceToHost, s));
    HPD_HIP(hipStreamSynchronize(s));
  }
  return HPD_OK;
}

int hpd_set_tail_pages(hpd_layout* L, int32_t page_size, int32_t n_pages, const int32_t* page_table) {
  if (!L || !L->on_device) return HPD_E_INVALID;
  if (page_size == 0) {
    L->dev.tail_pages = nullptr;
    L->dev.page_shift = L->dev.pages_per_branch = L->dev.n_pages = 0;
    return HPD_OK;
  }
  if (page_size < 8 || (page_size & (page_size - 1)) != 0 || n_pages < 1 || !page_table) return HPD_E_INVALID;
  if ((int64_t)n_pages * page_size > ((int64_t)1 << 40)) return HPD_E_OVERFLOW;
  int32_t shift = 0;
  while ((1 << shift) < page_size) ++shift;
  L->dev.tail_pages = page_table;
  L->dev.page_shift = shift;
  L->dev.pages_per_branch = (L->T + page_size - 1) / page_size;
  L->dev.n_pages = n_pages;
  return HPD_OK;
}

int hpd_finetune_mask(int32_t prompt_len, int32_t n_attr, const int32_t* attr_len,
                      const int32_t* value_len, int32_t k_max, int32_t* pos_out, uint8_t* mask_out,
                      int64_t* s_out, void* stream) {
  if (!s_out || prompt_len < 0 || n_attr < 0 || k_max < 1) return HPD_E_INVALID;
  if (n_attr > 0 && (!attr_len || !value_len)) return HPD_E_INVALID;
  int64_t S = prompt_len;
  for (int32_t n = 0; n < n_attr; ++n) {
    if (attr_len[n] < 1 || value_len[n] < 0 || value_len[n] > k_max) return HPD_E_INVALID;
    S += (int64_t)attr_len[n] + value_len[n];
    if (S > 46000) return HPD_E_OVERFLOW;
  }
  if (S > 46000 || S + (int64_t)n_attr * k_max > ((int64_t)1 << 30)) return HPD_E_OVERFLOW;
  *s_out = S;
  if (S == 0 || (!pos_out && !mask_out)) return HPD_OK;
  // where every attribute's name and value tokens start in the regular order, and the name tokens in
  // front of it
  hipStream_t s = (hipStream_t)stream;
  try {
    std::vector<int32_t> table(3 + 3 * (size_t)n_attr);
    table[0] = prompt_len; table[1] = n_attr; table[2] = k_max;
    int32_t *first_name = table.data() + 3, *first_value = first_name + n_attr, *before = first_value + n_attr;
    int32_t at = prompt_len, names = 0;
    for (int32_t n = 0; n < n_attr; ++n) {
      first_name[n] = at;
      first_value[n] = at + attr_len[n];
      before[n] = names;
      at += attr_len[n] + value_len[n];
      names += attr_len[n];
    }
    HPD_HIP(hpd_launch_finetune_mask(table.data(), (int32_t)S, pos_out, mask_out, s));
  } catch (const std::bad_alloc&) {
    return HPD_E_NOMEM;
  }
  HPD_HIP(hipStreamSynchronize(s));
  return HPD_OK;
}

}  // extern "C"
