// Decode attention of launches with many rows per unit (gfx950, bf16, head_dim 128): the loop of the prefill kernel
// (attn_prefill_kernel in hpd_attn_stream.hip: four waves of 32 rows that load and compute) with the units, the append and
// the tails of attn_stream_kernel.  Which steps run it is plan_dense's.
//
// What bounds such a launch is the compute waves.  attn_stream_kernel has six of them on a CU's four SIMDs beside two
// loaders: a block of 32 keys took 184 ns per row block and CU (70B-like, in-kernel timestamps), 129 ns here, and its one
// workgroup per CU leaves the CU idle while it starts and ends (18 of 93 us), where here the others work.
//  * Two or three workgroups per CU (WGS; the rule is hpd_plan_dense_launch's), as in the prefill: rounds of two blocks and a ring of four, or
//    rounds of one block, a ring of three, 168 registers.  For those what only the tails need of a lane is formed behind the prefix
//    (again()), a row's branch waits in LDS, a tile's values are read 16 keys at a time, and the start value of the scores is
//    two registers (MinusPoint).  No register may be left over for scratch memory: the compiler does not see the loads that are
//    written out, so at a reload the wave waits for all of them.  One to eight registers there, four in the loop over a wave's own
//    tiles (16/8 heads) and one in the loop over the tiles of the literal mask, cost 1.6 % in the mean of 1131 random batches, 16/8
//    heads 4 %.
//  * Launches that run all at a time: a wave lowers its priority as it goes.  With equal ones the oldest workgroup of a CU is always
//    served first and the last is left alone for the last fifth of the launch (16 x 2 documents below: 145.7 -> 131.4 us from
//    the first wave to the last); where workgroups follow each other the same costs 3 %.
//  * Block mask: a tail belongs to one wave's rows, so behind the shared blocks every wave fetches and works on the tiles
//    of its own branches, through pieces of the ring that are its own: no barrier.  16 KB of them, and the keys of a tile are
//    requested as soon as the scores of the one before are settled, its values when those have been read; with three workgroups
//    per CU 12 KB, where the second half of a tile's values follows its keys.  The first tile's keys come during the last round
//    of the prefix.  Positions in the newest chunk follow its length, as there.
//  * Literal mask: the tiles are shared blocks like the prefix (a wave skips those behind its last branch), with as few
//    positions in the newest chunk as it holds.  A row group's last tiles are only its own, so the last row group of a
//    prompt, which has the most, is started first.  Both blocks of a round of tiles at a time, as in the prefix: the
//    compiler spills 55 registers, 440 us instead of 317.
//  * Paged tails: the page table's entries for a tile come by DMA ahead of it.
// Measured (us per hpd_decode_step, the other kernel -> two workgroups per CU -> this): 16 prompts x 2 documents of 2048 tokens,
// 48 branches, 64/8 heads, step 17, 160 -> 142 -> 135 (768 workgroups); literal mask, 64 prompts x 4 documents of 384 tokens, 96
// branches, 32/8 heads, step 7, 369 -> 315 -> 305.  Outputs differ from the other kernel's by rounding (relative 7e-4 in bf16);
// error against 64 bits 1.7e-3 for both.
#include <algorithm>
#include <type_traits>

#include "hpd_attn_bf16.h"

namespace {

constexpr int DENSE_WAVES = HPD_DENSE_ROWS / 32;  // row blocks per workgroup

// Minus the reference point of a row, 16 times in the start value of its scores.  With two workgroups per CU the 16
// registers are kept, and the first matrix instruction of a chain reads them as its addend; with three they are two, and
// eight moves of 64 bits.
template <int WGS>
struct MinusPoint {
  floatx16 m = {};
  __device__ __forceinline__ float get() const { return m[0]; }
  __device__ __forceinline__ void set(float x) {
#pragma unroll
    for (int i = 0; i < 16; ++i) m[i] = x;
  }
  __device__ __forceinline__ floatx16 all() const { return m; }
};
template <>
struct MinusPoint<3> {
  typedef double doublex8 __attribute__((ext_vector_type(8)));
  double two = 0.0;
  __device__ __forceinline__ float get() const { return __builtin_bit_cast(floatx2, two)[0]; }
  __device__ __forceinline__ void set(float x) {
    two = __builtin_bit_cast(double, floatx2{x, x});
    asm volatile("" : "+v"(two));  // (one 64-bit value: taken apart it is moved 32 bits at a time)
  }
  __device__ __forceinline__ floatx16 all() const {
    double d[8];
    // (the moves written out, as the compiler takes 32 bits at a time; it does not know that the matrix instruction behind them
    // may read a register two instructions after a vector instruction wrote it)
    asm volatile(
        "v_mov_b64 %0, %8\n\tv_mov_b64 %1, %8\n\tv_mov_b64 %2, %8\n\tv_mov_b64 %3, %8\n\t"
        "v_mov_b64 %4, %8\n\tv_mov_b64 %5, %8\n\tv_mov_b64 %6, %8\n\tv_mov_b64 %7, %8\n\ts_nop 1"
        : "=&v"(d[0]), "=&v"(d[1]), "=&v"(d[2]), "=&v"(d[3]), "=&v"(d[4]), "=&v"(d[5]), "=&v"(d[6]), "=&v"(d[7])
        : "v"(two));
    return __builtin_bit_cast(floatx16, doublex8{d[0], d[1], d[2], d[3], d[4], d[5], d[6], d[7]});
  }
};

template <int G, bool PAPER, bool PAGED, int WGS>
__global__ void __launch_bounds__(DENSE_WAVES * 64, WGS)
attn_dense_kernel(const int32_t* __restrict__ descs, int32_t n_groups, int32_t row_groups, int32_t kv_heads, StreamArgs a,
                  const uint16_t* __restrict__ q, const uint16_t* __restrict__ k_prefix,
                  const uint16_t* __restrict__ v_prefix, uint16_t* __restrict__ k_tail, uint16_t* __restrict__ v_tail,
                  const uint16_t* __restrict__ k_new, const uint16_t* __restrict__ v_new, void* __restrict__ out) {
  constexpr int BPB = 32 / G;  // branches per row block (wave)
  constexpr int LG_G = G == 1 ? 0 : G == 2 ? 1 : G == 4 ? 2 : 3;
  constexpr uint32_t BLK = 16384;           // bytes of a block (8 KB of K, 8 KB of V)
  constexpr int SB = WGS == 2 ? 2 : 1;      // blocks per round
  constexpr int SLOTS = WGS == 2 ? 4 : 3;   // blocks in the ring
  constexpr uint32_t RING = SLOTS * BLK;
  // Two workgroups per CU, block mask: what most rounds of the prefix do lies in one piece, the rest behind the loop.  A branch that is
  // taken costs a round 2 % where a SIMD has one wave (the loop had one more than with two per CU alone: up to 256 workgroups 0.987
  // of its speed, so 1.002).  Three per CU: paged tails 0.5 % slower so; literal mask: registers spill.
  constexpr bool STRAIGHT = !PAPER && WGS == 2;
  __shared__ uint4 ring[SLOTS * SLOT_U4];
  constexpr int MAX_KEY_BRANCHES = 256;
  __shared__ int32_t klen[PAPER ? MAX_KEY_BRANCHES : 1];  // tokens in memory of every key branch
  __shared__ int32_t row_sees[PAPER ? DENSE_WAVES * 64 : 1];  // per wave: the branch of its 32 rows, the names they see
  // ids of the row group's branches where they are no run: a lookup in memory waits for the loads in front of it
  __shared__ int32_t ids[PAPER ? 1 : DENSE_WAVES * BPB];
  // paged tails: what the page table says for the branches of the tiles that a wave loads next (of its next round or own
  // tile, by the parity of that).  They come by DMA in front of the tile before: looked up when a tile is requested,
  // every lookup waited for all loads of the wave in flight, as its address is needed (16 branches of 125 tokens, a
  // document of 141: 380 us, the other kernel 152).
  __shared__ int32_t page_of[PAGED ? DENSE_WAVES : 1][2][64];

  const int tid = threadIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lane = tid & 63;
  const int n = lane & 31, g2 = lane >> 5, r4 = lane >> 4, c16 = lane & 15;
  // (unit, kv head) and row group of this workgroup, and the unit's descriptor: as in attn_stream_kernel
  if (WGS == 3 && a.at_once) __builtin_amdgcn_s_setprio(3);
  const int32_t rg = row_groups - 1 - (blockIdx.x >> 3) % row_groups;
  const int32_t grp = ((blockIdx.x >> 3) / row_groups) * 8 + (blockIdx.x & 7);
  if (grp >= n_groups) return;
  const int32_t hk = grp % kv_heads, u = grp / kv_heads;
  const int32_t* desc = descs + (int64_t)u * (PAPER ? 16 : 8);
  const int32_t hoff = desc[0], Hlen = desc[1], doff = desc[2], Llen = desc[3];
  const int32_t row0 = desc[4], nb = desc[5], upos = PAPER ? -1 : desc[6], ub0 = desc[7];
  const int32_t pb0 = PAPER ? desc[6] : 0;
  const int32_t n_doc_blk = PAPER ? desc[9] : 0;
  // the unit's row blocks, shared out evenly over the row groups that it needs
  const int32_t nblk = (nb * G + 31) >> 5, n_rg = (nblk + DENSE_WAVES - 1) / DENSE_WAVES;
  if (rg >= n_rg) return;  // uniform over the workgroup
  const int32_t per_group = (nblk + n_rg - 1) / n_rg, first_blk = rg * per_group;
  const int32_t nblk_here = min(per_group, nblk - first_blk);
  if (nblk_here <= 0) return;
  const int32_t br0 = first_blk * BPB, nbr_here = min(nb - br0, nblk_here * BPB);
  const bool active = wave < nblk_here;  // the wave has rows
  // global id of the unit's li-th live branch
  auto unit_branch = [&](int32_t li) -> int32_t { return ub0 >= 0 ? ub0 + li : a.tb.live_branch[a.live_base + row0 + li]; };
  const int32_t kb_end = PAPER ? __builtin_amdgcn_readfirstlane(unit_branch(br0 + nbr_here - 1)) - pb0 + 1 : 0;

  // ---- what all rows share: NB prefix blocks, at least one, as a document has a token; literal mask: then the tail tiles of the prompt's branches 0 .. kb_end-1
  const int32_t NBh = (Hlen + 31) >> 5, NBd = PAPER ? Llen : (Llen + 31) >> 5, NB = NBh + NBd;
  const int32_t NC = (a.step >> 3) + 1, newest = (a.step & 7) + 1;
  const int32_t fmt_lg = newest <= 1 ? 0 : newest <= 2 ? 1 : newest <= 4 ? 2 : 3;
  const int32_t NQ = PAPER ? (kb_end + 3) >> 2 : 0;
  const int32_t n_full = PAPER ? (fmt_lg < 3 ? NQ * (NC - 1) : NQ * NC) : 0;
  const int32_t NS = NB + (PAPER ? n_full + (fmt_lg < 3 ? (kb_end + (32 >> fmt_lg) - 1) >> (5 - fmt_lg) : 0) : 0);
  const int32_t NR = (NS + SB - 1) / SB;  // rounds
  const const_i32* const list = (const const_i32*)(uintptr_t)(a.tb.pblk + 2 * (int64_t)(PAPER ? doff : 0));

  // What only the tails need of the lane is formed where they need it: kept through the loops it costs registers.  (The literal mask
  // with two workgroups per CU has them: forming it again there, and looking for non-finite values 16 keys at a time, cost 1 to 2 %.)
  auto again = [](int lane) -> int { asm volatile("" : "+v"(lane)); return lane; };
  // ---- loads: quarter `wave` of a block (K rows 0..15, K rows 16..31, V d-blocks 0..1, 2..3; tail tiles: V rows 0..15,
  //      16..31)
  const bool is_v = wave >= 2;
  uint32_t vo[4];
#pragma unroll
  for (int f = 0; f < 4; ++f) {
    const uint32_t k_off = (uint32_t)(r4 * 256 + ((c16 ^ r4 ^ (4 * f)) << 4));  // + f * 1024
    const uint32_t v_off = (uint32_t)(((g2 * 128 + n) << 4) + 2048 + (f & 1) * 4096 + (f >> 1) * 512 - f * 1024);
    vo[f] = is_v ? v_off : k_off;
  }
  const char* const src = (is_v ? reinterpret_cast<const char*>(v_prefix) + (wave & 1) * 1024 - 2048
                                : reinterpret_cast<const char*>(k_prefix) + (wave & 1) * 4096) +
                          (int64_t)hk * a.NP * (D * 2);
  const uint32_t ring_lds = (uint32_t)reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) char*)ring);
  auto issue_prefix = [&](int32_t slot0, uint32_t at) {
    const char* const s = uniform(src + (int64_t)slot0 * (D * 2));
    const uint32_t dst = __builtin_amdgcn_readfirstlane(ring_lds + at + (uint32_t)wave * 4096);
    uint32_t keep;  // M0 is the compiler's: put back what it held
    asm volatile(
        "s_mov_b32 %0, m0\n\ts_mov_b32 m0, %5\n\ts_nop 0\n\t"
        "global_load_lds_dwordx4 %1, %6\n\t"
        "global_load_lds_dwordx4 %2, %6 offset:1024\n\t"
        "global_load_lds_dwordx4 %3, %6 offset:2048\n\t"
        "global_load_lds_dwordx4 %4, %6 offset:3072\n\t"
        "s_mov_b32 m0, %0"
        : "=&s"(keep)
        : "v"(vo[0]), "v"(vo[1]), "v"(vo[2]), "v"(vo[3]), "s"(dst), "s"(s)
        : "memory");
  };
  // four rows-of-four: rows rw[0..3] of a pool, chunk ch[f] of each, to LDS bytes at .. at + 4095; streaming hint
  auto issue_rows = [&](const uint16_t* pool, const uint32_t (&rw)[4], const uint32_t (&ch)[4], uint32_t at) {
    const char* p[4];
#pragma unroll
    for (int f = 0; f < 4; ++f) p[f] = reinterpret_cast<const char*>(pool) + ((uint64_t)rw[f] * (D * 2) + ch[f]) - f * 1024;
    const uint32_t dst = __builtin_amdgcn_readfirstlane(ring_lds + at);
    uint32_t keep;
    asm volatile(
        "s_mov_b32 %0, m0\n\ts_mov_b32 m0, %5\n\ts_nop 0\n\t"
        "global_load_lds_dwordx4 %1, off nt\n\t"
        "global_load_lds_dwordx4 %2, off offset:1024 nt\n\t"
        "global_load_lds_dwordx4 %3, off offset:2048 nt\n\t"
        "global_load_lds_dwordx4 %4, off offset:3072 nt\n\t"
        "s_mov_b32 m0, %0"
        : "=&s"(keep)
        : "v"(p[0]), "v"(p[1]), "v"(p[2]), "v"(p[3]), "s"(dst)
        : "memory");
  };
  // row (32 bits hold the rows of any pool that fits the memory) of token t of branch b
  auto tail_row = [&](int32_t b, int32_t t) -> uint32_t {
    if (PAGED) return (uint32_t)hpd_tail_row(a.tb, b, hk, a.Hkv, a.Tcap, t);
    return ((uint32_t)b * (uint32_t)a.Hkv + (uint32_t)hk) * (uint32_t)a.Tcap + (uint32_t)t;
  };
  // paged: the page table's entry for the page of token t of branch b, one per lane, to page_of[wave][half]
  auto request_pages = [&](int32_t half, int32_t b, int32_t t) __attribute__((always_inline)) {
    const int32_t* const p = a.tb.tail_pages + (int64_t)b * a.tb.pages_per_branch + (t >> a.tb.page_shift);
    const uint32_t dst = __builtin_amdgcn_readfirstlane((uint32_t)reinterpret_cast<uintptr_t>(
        (__attribute__((address_space(3))) int32_t*)page_of[wave][half]));
    uint32_t keep;
    asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dword %1, off\n\ts_mov_b32 m0, %0"
                 : "=&s"(keep) : "v"(p), "s"(dst) : "memory");
  };
  // ... and the row of token t (as in hpd_tail_row) of the branch that lane l asked for
  auto paged_row = [&](int32_t half, int32_t l, int32_t t) -> uint32_t {
    const uint32_t pg = (uint32_t)min(max(page_of[wave][half][l], 0), a.tb.n_pages - 1);
    return ((pg * (uint32_t)a.Hkv + (uint32_t)hk) << a.tb.page_shift) + (uint32_t)(t & ((1 << a.tb.page_shift) - 1));
  };
  // literal mask, tail tile tt: key k is position c * 8 + k % 2^lg of branch tb0 + k / 2^lg
  struct TileAt { int32_t c, tb0, lg; };
  auto tile_at = [&](int32_t tt) -> TileAt {
    if (tt < n_full) {
      const int32_t c = tt / max(NQ, 1);
      return {c, (tt - c * NQ) * 4, 3};
    }
    return {NC - 1, (tt - n_full) << (5 - fmt_lg), fmt_lg};
  };
  // (a branch's positions in a tile are those of one chunk of 8, or its last token: they lie in one page)
  auto round_pages = [&](int32_t r) __attribute__((always_inline)) {  // of the tiles of round r
    if (r >= NR || SB * r + SB - 1 < NB) return;
    const TileAt x = tile_at(max(SB * r - NB, 0)), y = tile_at(min(SB * r + SB - 1, NS - 1) - NB);
    const int32_t c = g2 ? y.c : x.c, j = min((g2 ? y.tb0 : x.tb0) + n, kb_end - 1);
    request_pages(r & 1, pb0 + j, max(min(c * 8, klen[j] - 1), 0));
  };
  auto issue_tile = [&](int32_t gb, uint32_t at) {
    const TileAt x = tile_at(gb - NB);
    const int lane_t = WGS == 3 ? again(lane) : lane, r4 = lane_t >> 4, c16 = lane_t & 15;
    uint32_t rw[4], ch[4];
#pragma unroll
    for (int f = 0; f < 4; ++f) {
      const int32_t k = (wave & 1) * 16 + f * 4 + r4;
      const int32_t j = min(x.tb0 + (k >> x.lg), kb_end - 1);
      const int32_t pos = max(min(x.c * 8 + (k & ((1 << x.lg) - 1)), klen[j] - 1), 0);
      rw[f] = PAGED ? paged_row((SB == 2 ? gb >> 1 : gb) & 1, (SB == 2 ? (gb & 1) * 32 : 0) + (k >> x.lg), pos) : tail_row(pb0 + j, pos);
      ch[f] = (uint32_t)(is_v ? (c16 ^ (2 * r4)) << 4 : (c16 ^ r4 ^ (4 * f)) << 4);
    }
    issue_rows(is_v ? v_tail : k_tail, rw, ch, at + (uint32_t)wave * 4096);
  };
  auto slot_of = [&](int32_t gb) -> int32_t {  // first pool slot of a prefix block
    if (gb < NBh) return hoff + gb * 32;
    return PAPER ? list[2 * (gb - NBh)] : doff + (gb - NBh) * 32;
  };
  auto issue = [&](int32_t gb, int32_t slot, uint32_t at) {
    if (!PAPER || gb < NB) issue_prefix(slot, at);
    else issue_tile(gb, at);
  };
  // blocks SB * r .. of round r, whose prefix blocks lie at sA, sB, to ring bytes at.. (a block past the last one re-loads the
  // last one, never read)
  auto issue_round = [&](int32_t r, int32_t sA, int32_t sB, uint32_t at) {
    issue(SB * r, sA, at);
    if (SB == 2) issue(min(2 * r + 1, NS - 1), sB, at + BLK);
  };
  auto slot_clamped = [&](int32_t gb) -> int32_t { return slot_of(min(gb, NB - 1)); };

  // ---- fused mode: append the newest tokens (the arithmetic of hpd_kv_append), 8 lanes per branch.  Literal mask:
  //      all live branches up to the row group's last (the same bytes from every writer).
  auto append = [&]() {
    const int32_t ap_c = (tid & 7) * 8;
    for (int32_t li = (PAPER ? 0 : br0) + (tid >> 3); li < br0 + nbr_here; li += DENSE_WAVES * 8) {
      const int64_t noff = ((int64_t)(row0 + li) * a.Hkv + hk) * D;
      const uint4 klo = *reinterpret_cast<const uint4*>(k_new + noff + ap_c);
      const uint4 khi = *reinterpret_cast<const uint4*>(k_new + noff + 64 + ap_c);
      const uint4 vlo = *reinterpret_cast<const uint4*>(v_new + noff + ap_c);
      const uint4 vhi = *reinterpret_cast<const uint4*>(v_new + noff + 64 + ap_c);
      const int32_t b = unit_branch(li);
      const int32_t pos = upos >= 0 ? upos : a.tb.branch_base_pos[b] + 1 + a.step;
      float rl[8], rh[8];
      rotate16(klo, khi, a.tb.rope + (int64_t)pos * (D / 2), ap_c, rl, rh);
      const int64_t trow = (int64_t)tail_row(b, a.step) * D;
      *reinterpret_cast<uint4*>(k_tail + trow + ap_c) = pack8_key(rl);
      *reinterpret_cast<uint4*>(k_tail + trow + 64 + ap_c) = pack8_key(rh);
      *reinterpret_cast<uint4*>(v_tail + trow + ap_c) = cache8(vlo);
      *reinterpret_cast<uint4*>(v_tail + trow + 64 + ap_c) = cache8(vhi);
    }
  };
  if constexpr (PAPER) {
    for (int32_t i = tid; i < kb_end; i += DENSE_WAVES * 64) klen[i] = min(a.step + 1, a.tb.branch_len[pb0 + i]);
  }
  if (!PAPER && ub0 < 0) {
    for (int32_t i = tid; i < nbr_here; i += DENSE_WAVES * 64) ids[i] = unit_branch(br0 + i);
  }
  // rounds 0 and 1 are requested in front of the first barrier: with tail tiles among them the append comes before
  const bool append_first = a.fused && PAPER && NB < 4;
  if (PAPER && NB < 4) {
    if (append_first) append();
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __syncthreads();
    if (PAGED) {
      round_pages(0);
      round_pages(1);
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
  }

  // ---- block mask: the tails of the wave's own branches, tile by tile, through pieces of 4 KB of the ring that are the wave's:
  //      two in the slots that the last round does not use, and one (three workgroups per CU) or two in the last round's
  const uint32_t last_at = (uint32_t)((NR - 1) % (SLOTS / SB)) * (SB * BLK);  // where the last round lies
  auto ring_wrap = [&](uint32_t at) -> uint32_t { return at >= RING ? at - RING : at; };
  const uint32_t my_free = ring_wrap(last_at + SB * BLK + (uint32_t)wave * 8192), my_last = last_at + (uint32_t)wave * (SB * 4096);
  const int32_t wb0 = wave * BPB, wnb = min(BPB, nbr_here - wb0);  // the wave's branches
  const int32_t lg_new = max(fmt_lg, LG_G);
  const int32_t n_quad = (wnb + 3) >> 2;
  const int32_t n_own = PAPER ? 0 : n_quad * (NC - 1) + ((wnb + (32 >> lg_new) - 1) >> (5 - lg_new));
  auto own_tile = [&](int32_t t) -> TileAt {
    const int32_t nf = n_quad * (NC - 1);
    if (t < nf) {
      const int32_t c = n_quad == 1 ? t : t / n_quad;
      return {c, wb0 + (t - c * n_quad) * 4, 3};
    }
    return {NC - 1, wb0 + ((t - nf) << (5 - lg_new)), lg_new};
  };
  auto own_pages = [&](int32_t t) __attribute__((always_inline)) {
    const TileAt x = own_tile(t);
    const int32_t j = min(x.tb0 + n, nbr_here - 1);
    request_pages(t & 1, t < 2 ? unit_branch(br0 + j) : ub0 >= 0 ? ub0 + br0 + j : ids[j], x.c * 8);
  };
  if (PAGED && !PAPER && active) {
    own_pages(0);
    if (n_own > 1) own_pages(1);
  }

  // ---- the query rows of the wave, straight into operand layout, and their position
  const int32_t lb_row = wave * BPB + n / G;                       // this row's branch, counted in the row group
  const int32_t my_lb = br0 + min(lb_row, nbr_here - 1);           // ... in the unit; rows behind the last repeat it
  uint4 qraw[8];
  {
    const uint16_t* qp = q + ((int64_t)(row0 + my_lb) * a.Hq + hk * a.Gr + min(n % G, a.Gr - 1)) * D + g2 * 8;
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) qraw[kk] = *reinterpret_cast<const uint4*>(qp + kk * 16);
  }
  const int32_t my_branch = unit_branch(my_lb);
  const int32_t pos = upos >= 0 ? upos : a.tb.branch_base_pos[my_branch] + 1 + a.step;
  issue_round(0, slot_clamped(0), slot_clamped(1), 0);
  if (NR > 1) issue_round(1, slot_clamped(SB), slot_clamped(3), SB * BLK);
  if (PAPER && PAGED && SB == 1) {  // of tiles among blocks 2 and 3
    round_pages(2);
    round_pages(3);
  }
  f16x8 Qf[8];
  {
    const float4* cs_row = reinterpret_cast<const float4*>(a.tb.rope + (int64_t)pos * (D / 2));
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      float lo[8], hi[8], rl[8], rh[8];
      unpack8(qraw[kk], lo);
      unpack8(qraw[kk + 4], hi);
#pragma unroll
      for (int e2 = 0; e2 < 4; ++e2) {
        const float4 cs = cs_row[kk * 8 + g2 * 4 + e2];
        hpd::rope_pair(lo[2 * e2], hi[2 * e2], cs.x, cs.y, rl[2 * e2], rh[2 * e2]);
        hpd::rope_pair(lo[2 * e2 + 1], hi[2 * e2 + 1], cs.z, cs.w, rl[2 * e2 + 1], rh[2 * e2 + 1]);
      }
#pragma unroll
      for (int e = 0; e < 8; ++e) { rl[e] *= a.scale_log2; rh[e] *= a.scale_log2; }
      Qf[kk] = pack8_half(rl);
      Qf[kk + 4] = pack8_half(rh);
    }
  }
  if (a.fused && !append_first) append();

  float l_lane = 0.f;
  MinusPoint<WGS> minus_m;
  float slack = -INFINITY;
  floatx16 acc[4];
#pragma unroll
  for (int blk = 0; blk < 4; ++blk)
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[blk][i] = 0.f;

  const char* const rc = reinterpret_cast<const char*>(ring);
  auto k_of = [](int lane) -> uint32_t {  // fragment kk of the lane lies at k_of ^ (kk << 5)
    const int n = lane & 31, krow = ((n >> 4) << 4) | (((n >> 2) & 1) << 3) | (((n >> 3) & 1) << 2) | (n & 3);
    return (uint32_t)(krow * 256 + (((lane >> 5) ^ (krow & 15)) << 4));
  };
  const uint32_t k_lane = k_of(lane);
  // Scores, softmax and value product as in attn_prefill_kernel.  N blocks whose K halves lie at `at`, `at` + BLK; k_lane: where
  // the lane's row of a block lies.
  auto settle = [&](auto nc, float (&s)[decltype(nc)::value][16], uint32_t k_lane, uint32_t at, bool masked, uint32_t ok0, uint32_t ok1)
      __attribute__((always_inline)) {
    constexpr int N = decltype(nc)::value;
    auto scores = [&]() __attribute__((always_inline)) {
      uint32_t base = k_lane + at;
      if (WGS == 3) asm volatile("" : "+v"(base));  // (eight addresses kept from one block for the next are eight registers)
#pragma unroll
      for (int b = 0; b < N; ++b) {
        floatx16 S = minus_m.all();
#pragma unroll
        for (int kk = 0; kk < 8; ++kk) {
          const f16x8 kf = __builtin_bit_cast(f16x8, *reinterpret_cast<const uint4*>(
              rc + (WGS == 3 ? base ^ (kk << 5) : at + (k_lane ^ (kk << 5))) + b * BLK));
          S = __builtin_amdgcn_mfma_f32_32x32x16_f16(kf, Qf[kk], S, 0, 0, 0);
        }
#pragma unroll
        for (int i = 0; i < 16; ++i) s[b][i] = S[i];
      }
      if (STRAIGHT ? __builtin_expect(masked, 0) : masked) {
#pragma unroll
        for (int b = 0; b < N; ++b)
#pragma unroll
          for (int i = 0; i < 16; ++i) s[b][i] = ((b ? ok1 : ok0) >> i) & 1 ? s[b][i] : -INFINITY;
      }
    };
    scores();
    float bm = NEG_BIG;
#pragma unroll
    for (int b = 0; b < N; ++b)
#pragma unroll
      for (int i = 0; i < 16; ++i) bm = fmaxf(bm, s[b][i]);
    if (STRAIGHT ? __builtin_expect(__any(bm > slack), 0) : __any(bm > slack)) {
      bm = fmaxf(bm, __shfl_xor(bm, 32));
      // (a row that has seen no key yet keeps its empty state)
      const bool none = bm <= NEG_BIG, first = slack < 0.f;
      const float d = none ? 0.f : first ? bm : fmaxf(bm, 0.f);
      const float alpha = first ? 0.f : fast_exp2(-d);
      slack = none && first ? slack : WGS == 3 && N == 1 && first ? 0.f : MAX_SLACK;  // (the second block moves a first one's point)
      const float m_old = minus_m.get(), m_new = m_old - d;
      const bool again = __any(fabsf(m_old) > fmaxf(128.f, fabsf(m_new)));
      minus_m.set(m_new);
      const float shift = again ? 0.f : d;
      if (STRAIGHT ? __builtin_expect(again, 0) : again) scores();
#pragma unroll
      for (int b = 0; b < N; ++b)
#pragma unroll
        for (int i = 0; i < 16; ++i) s[b][i] -= shift;
      l_lane *= alpha;
#pragma unroll
      for (int blk = 0; blk < 4; ++blk)
#pragma unroll
        for (int i = 0; i < 16; ++i) acc[blk][i] *= alpha;
    }
  };
  // the weights, rounded to halves, and their sum
  auto weights = [&](float (&s)[16], f16x8& P0, f16x8& P1) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 16; ++i) s[i] = fast_exp2(s[i]);
    P0 = pack8_half(s);
    P1 = pack8_half(s + 8);
    const uint4 w0 = __builtin_bit_cast(uint4, P0), w1 = __builtin_bit_cast(uint4, P1);
    float la = sum_half_pair(w0.x, l_lane), lb = sum_half_pair(w1.x, 0.f);
    la = sum_half_pair(w0.y, la); lb = sum_half_pair(w1.y, lb);
    la = sum_half_pair(w0.z, la); lb = sum_half_pair(w1.z, lb);
    la = sum_half_pair(w0.w, la); lb = sum_half_pair(w1.w, lb);
    l_lane = la + lb;
  };
  auto value_product = [&](const f16x8& P0, const f16x8& P1, const uint4 (&vf)[8]) __attribute__((always_inline)) {
#pragma unroll
    for (int blk = 0; blk < 4; ++blk) {
      acc[blk] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, vf[blk * 2]), P0, acc[blk], 0, 0, 0);
      acc[blk] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, vf[blk * 2 + 1]), P1, acc[blk], 0, 0, 0);
    }
  };
  auto read_values = [&](uint32_t at, uint4 (&vf)[8]) __attribute__((always_inline)) {  // of a prefix block's V half
#pragma unroll
    for (int f = 0; f < 8; ++f) vf[f] = *reinterpret_cast<const uint4*>(rc + at + lane * 16 + f * 1024);
  };
  // the fragments of 16 keys of a tail tile, whose rows lie at `at`; as in attn_stream_kernel
  auto read_tail_half = [&](int lane, uint32_t at, uint4 (&vf)[4]) __attribute__((always_inline)) {
    const int g2 = lane >> 5;
    const int tj = (lane >> 2) & 3, tr = lane & 3;
    const int tx = ((lane >> 4) & 1) * 2 + (tr >> 1);
    const char* vlane = rc + at + (g2 * 8 + tj) * 256 + (tr & 1) * 8;
#pragma unroll
    for (int blk = 0; blk < 4; ++blk) {
      const char* p = vlane + ((blk * 4 + tx) ^ (2 * tj)) * 16;
      const uint2 k03 = hpd::lds_read_tr16(p), k47 = hpd::lds_read_tr16(p + 4 * 256);
      vf[blk] = make_uint4(k03.x, k03.y, k47.x, k47.y);
    }
  };
  auto read_tail_values = [&](int lane, uint32_t at, uint4 (&vf)[8]) __attribute__((always_inline)) {
    uint4 half[2][4];
    read_tail_half(lane, at, half[0]);
    read_tail_half(lane, at + 4096, half[1]);
#pragma unroll
    for (int f = 0; f < 8; ++f) vf[f] = half[f & 1][f >> 1];
  };
  auto half_product = [&](const f16x8& P, const uint4 (&vf)[4]) __attribute__((always_inline)) {
#pragma unroll
    for (int blk = 0; blk < 4; ++blk)
      acc[blk] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, vf[blk]), P, acc[blk], 0, 0, 0);
  };
  // literal mask: the branch of this row and of the row block's last one, counted from the prompt's first, and the
  // names they see; a row's own wait in LDS until the prefix is done
  int32_t kb_row = 0, kb_row_min = 0, kb_row_max = 0, names_row = 0, names_max = 0;
  if constexpr (PAPER) {
    kb_row_min = __builtin_amdgcn_readfirstlane(my_branch) - pb0;
    kb_row_max = __builtin_amdgcn_readfirstlane(unit_branch(br0 + min(wave * BPB + BPB - 1, nbr_here - 1))) - pb0;
    names_max = __builtin_amdgcn_readfirstlane(a.tb.skel_cum[pb0 + kb_row_max]);
    row_sees[tid] = g2 ? a.tb.skel_cum[my_branch] : my_branch - pb0;
  }
  // Literal mask: an infinite or NaN value of a branch must not reach the rows of earlier ones as 0 * value.  Where a tile
  // with branches that not all rows see has one, the product takes zeros in its place, and the rows that see it add it.  (A
  // token's value before it is weighted: what matters is that it is not finite.)
  auto non_finite = [](uint32_t half) -> bool { return (half & 0x7c00u) == 0x7c00u; };
  // vf: N fragments, of keys k0 .. k0 + 4 * N - 1.
  auto take_out_non_finite = [&](auto nc, int32_t tile, uint32_t at, int32_t k0, uint4 (&vf)[decltype(nc)::value])
      __attribute__((always_inline)) {
    constexpr int N = decltype(nc)::value;
    const f16x2 zero = {(_Float16)0, (_Float16)0};
    f16x2 z[4] = {zero, zero, zero, zero};
#pragma unroll
    for (int f = 0; f < N; ++f) {  // (a finite value times zero is zero)
      z[0] = __builtin_elementwise_fma(__builtin_bit_cast(f16x2, vf[f].x), zero, z[0]);
      z[1] = __builtin_elementwise_fma(__builtin_bit_cast(f16x2, vf[f].y), zero, z[1]);
      z[2] = __builtin_elementwise_fma(__builtin_bit_cast(f16x2, vf[f].z), zero, z[2]);
      z[3] = __builtin_elementwise_fma(__builtin_bit_cast(f16x2, vf[f].w), zero, z[3]);
    }
    const f16x2 sum = (z[0] + z[1]) + (z[2] + z[3]);
    if (!__any(!((float)sum[0] + (float)sum[1] == 0.f))) return;
    auto finite_pair = [&](uint32_t w) -> uint32_t {
      return w & ((non_finite(w) ? 0u : 0xffffu) | (non_finite(w >> 16) ? 0u : 0xffff0000u));
    };
#pragma unroll
    for (int f = 0; f < N; ++f) vf[f] = make_uint4(finite_pair(vf[f].x), finite_pair(vf[f].y), finite_pair(vf[f].z), finite_pair(vf[f].w));
    const TileAt x = tile_at(tile);
    const int g2 = (WGS == 3 ? again(lane) : lane) >> 5;
#pragma nounroll
    for (int32_t k = k0; k < k0 + 4 * N; ++k) {
      const int32_t j = x.tb0 + (k >> x.lg);
      const bool sees = j <= kb_row && (k & ((1 << x.lg) - 1)) < klen[min(j, kb_end - 1)] - x.c * 8;
#pragma unroll
      for (int blk = 0; blk < 4; ++blk)
#pragma unroll
        for (int cc = 0; cc < 4; ++cc) {  // channels blk * 32 + cc * 8 + g2 * 4 + 0 .. 3 of key k
          const uint2 v = *reinterpret_cast<const uint2*>(rc + at + k * 256 + (((blk * 4 + cc) ^ (2 * (k & 3))) << 4) + g2 * 8);
          const uint32_t h4[4] = {v.x & 0xffffu, v.x >> 16, v.y & 0xffffu, v.y >> 16};
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (sees && non_finite(h4[e])) acc[blk][cc * 4 + e] += hpd::cache_bits_to_float(h4[e]);
        }
    }
  };
  // N blocks from `at` on; tile >= 0: a tail tile of the literal mask (N = 1); later: with branches that a row does not see
  auto compute = [&](auto nc, uint32_t at, bool masked, uint32_t ok0, uint32_t ok1, int32_t tile,
                     bool later) __attribute__((always_inline)) {
    constexpr int N = decltype(nc)::value;
    float s[N][16];
    settle(nc, s, k_lane, at, masked, ok0, ok1);
    if constexpr (PAPER && N == 1 && WGS == 3) {
      f16x8 P[2];
      weights(s[0], P[0], P[1]);
      const int lane_t = again(lane);
#pragma unroll
      for (int h = 0; h < 2; ++h) {  // 16 keys at a time
        uint4 vf[4];
        if (tile >= 0) {
          read_tail_half(lane_t, at + 8192 + h * 4096, vf);
        } else {
#pragma unroll
          for (int blk = 0; blk < 4; ++blk)
            vf[blk] = *reinterpret_cast<const uint4*>(rc + at + lane_t * 16 + 8192 + (2 * blk + h) * 1024);
        }
        if (later) take_out_non_finite(std::integral_constant<int, 4>{}, tile, at + 8192, 16 * h, vf);
        half_product(P[h], vf);
      }
      return;
    }
#pragma unroll
    for (int b = 0; b < N; ++b) {
      uint4 vf[8];
      if (PAPER && tile >= 0) read_tail_values(lane, at + b * BLK + 8192, vf);
      else read_values(at + b * BLK + 8192, vf);
      f16x8 P0, P1;
      weights(s[b], P0, P1);
      if (PAPER && N == 1 && later) take_out_non_finite(std::integral_constant<int, 8>{}, tile, at + 8192, 0, vf);
      value_product(P0, P1, vf);
    }
  };
  auto first_bits = [](int32_t cnt) -> uint32_t { return (1u << min(max(cnt, 0), 8)) - 1u; };
  auto ok_bits = [&](int32_t valid) -> uint32_t {
    return first_bits(valid - g2 * 8) | (first_bits(valid - 16 - g2 * 8) << 8);
  };

  const int32_t h_part = (Hlen & 31) ? NBh - 1 : -1, d_part = !PAPER && (Llen & 31) ? NB - 1 : -1;
  auto keys_of = [&](int32_t b) -> int32_t {  // of a prefix block
    if (b == h_part) return Hlen & 31;
    if (PAPER) return b < NBh ? 32 : list[2 * (b - NBh) + 1];
    return b == d_part ? Llen & 31 : 32;
  };
  // where the prefix blocks of the round that is requested next lie
  int32_t nA = slot_clamped(2 * SB), nB = slot_clamped(5);
  const int32_t prio_at[3] = {a.at_once ? NR >> 1 : -1, a.at_once ? NR - (NR >> 2) : -1, a.at_once ? NR - (NR >> 3) : -1};
  // at: where round r lies in the ring
  auto open_round = [&](int32_t r, uint32_t at) __attribute__((always_inline)) {
    if (WGS == 3 && r == prio_at[0]) __builtin_amdgcn_s_setprio(2);
    if (WGS == 3 && r == prio_at[1]) __builtin_amdgcn_s_setprio(1);
    if (WGS == 3 && r == prio_at[2]) __builtin_amdgcn_s_setprio(0);
    // (rounds 0 and 1 were requested in front of the loop, a round is 4 * SB loads of the wave; so was the append, which is
    // complete at barrier 1, and the page entries of rounds 2 and 3)
    const bool newer = SB == 2 ? r == 0 && NR > 1 : r + 1 < NR && !(PAPER && PAGED && r == 0);
    if (newer) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(4 * SB) : "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): LDS reads of the previous round are done
    __builtin_amdgcn_s_barrier();        // the round is in LDS; the slots of the round before are free
    if constexpr (SB == 2) {
      if (r >= 1 && r + 1 < NR) {
        issue_round(r + 1, nA, nB, at ^ (2 * BLK));
        nA = slot_clamped(2 * r + 4);
        nB = slot_clamped(2 * r + 5);
      }
      if (PAPER && PAGED) round_pages(r + 2);
    } else {
      if (r + 2 < NR) {
        issue_round(r + 2, nA, 0, at == 0 ? 2 * BLK : at - BLK);
        nA = slot_clamped(r + 3);
      }
      // (two rounds before they are used: the wait of the round between leaves the four newest loads in flight, and round
      // r + 3's are newer)
      if (PAPER && PAGED) round_pages(r + 4);
    }
  };
  auto behind = [&](uint32_t at) -> uint32_t { return at == RING - SB * BLK ? 0u : at + SB * BLK; };

  const int32_t r_plain = (PAPER ? NBh + n_doc_blk : NB) / SB;  // rounds of blocks that all rows see alike
  // rows 16 h .. 16 h + 15 of the K or V half of own tile t, which is x: row k is position c * 8 + k % 2^lg of branch tb0 + k / 2^lg; what
  // lies behind the last branch or position repeats the last one
  auto issue_own = [&](const uint16_t* pool, bool v, int h, uint32_t at, int32_t t, const TileAt& x) __attribute__((always_inline)) {
    const int lane_t = again(lane), r4 = lane_t >> 4, c16 = lane_t & 15;
    uint32_t rw[4], ch[4];
    int32_t j[4], pos[4];
#pragma unroll
    for (int f = 0; f < 4; ++f) {
      const int32_t k = (4 * h + f) * 4 + r4;
      j[f] = PAGED ? k >> x.lg : min(x.tb0 + (k >> x.lg), nbr_here - 1);
      pos[f] = min(x.c * 8 + (k & ((1 << x.lg) - 1)), a.step);
      ch[f] = (uint32_t)(v ? (c16 ^ (2 * r4)) << 4 : (c16 ^ r4 ^ (4 * f)) << 4);
    }
    if constexpr (PAGED) {
#pragma unroll
      for (int f = 0; f < 4; ++f) rw[f] = paged_row(t & 1, j[f], pos[f]);
    } else if (ub0 >= 0) {
#pragma unroll
      for (int f = 0; f < 4; ++f) rw[f] = tail_row(ub0 + br0 + j[f], pos[f]);
    } else {  // (the four looked up together: one wait)
#pragma unroll
      for (int f = 0; f < 4; ++f) rw[f] = tail_row(ids[j[f]], pos[f]);
    }
    issue_rows(pool, rw, ch, at);
  };
  auto issue_own_keys = [&](uint32_t at0, uint32_t at1, int32_t t, const TileAt& x) __attribute__((always_inline)) {
    issue_own(k_tail, false, 0, at0, t, x);
    issue_own(k_tail, false, 1, at1, t, x);
  };

  // Rounds of one block: the first two at once where all rows see both and blocks 2 and 3 are of the prefix, too, so that the reference
  // point is that of 64 keys without being moved.  Against moving it with the second block: 1.008x (block mask, contiguous) and 1.005x
  // (literal) in the mean of 543 random batches, paged tails as before; 16 x 2 documents of 2048 tokens 134.3 -> 133.1 us.
  const bool pair = WGS == 3 && r_plain >= 2 && NB >= 4;
  auto open_pair = [&]() __attribute__((always_inline)) {
    issue_round(2, nA, 0, 2 * BLK);
    asm volatile("s_waitcnt vmcnt(4)" ::: "memory");  // blocks 0 and 1; the append
    __builtin_amdgcn_s_waitcnt(0xc07f);
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    if (PAPER && PAGED) round_pages(4);
  };
  auto close_pair = [&]() __attribute__((always_inline)) {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();  // their slots are free
    issue_round(3, slot_clamped(3), 0, 0);
    nA = slot_clamped(4);
    if (PAPER && PAGED) round_pages(5);
  };
  uint32_t at = 0;
  int32_t r = 0;
  if (!active) {  // a wave without rows loads
    if (pair) {
      open_pair();
      close_pair();
      r = 2;
      at = 2 * BLK;
    }
    for (; r < NR; ++r) {
      open_round(r, at);
      at = behind(at);
    }
    __builtin_amdgcn_s_waitcnt(0xc07f);
    __builtin_amdgcn_s_barrier();
    return;
  }
  if (pair) {
    open_pair();
    const int32_t vA = keys_of(0), vB = keys_of(1);
    const bool masked = (vA & vB) != 32;
    uint32_t ok0 = 0, ok1 = 0;
    if (masked) { ok0 = ok_bits(vA); ok1 = ok_bits(vB); }
    compute(std::integral_constant<int, 2>{}, 0, masked, ok0, ok1, -1, false);
    close_pair();
    r = 2;
    at = 2 * BLK;
  }
  for (; r < r_plain; ++r) {
    open_round(r, at);
    if (!PAPER && (STRAIGHT ? __builtin_expect(r == NR - 1, 0) : r == NR - 1)) issue_own_keys(my_free, my_free + 4096, 0, own_tile(0));
    const int32_t vA = keys_of(SB * r), vB = SB == 2 ? keys_of(2 * r + 1) : 32;
    const bool masked = (vA & vB) != 32;
    uint32_t ok0 = 0, ok1 = 0;
    if (STRAIGHT ? __builtin_expect(masked, 0) : masked) { ok0 = ok_bits(vA); ok1 = ok_bits(vB); }
    compute(std::integral_constant<int, SB>{}, at, masked, ok0, ok1, -1, false);
    at = behind(at);
  }
  if constexpr (PAPER) {
    kb_row = row_sees[wave * 64 + (again(lane) & 31)];
    names_row = row_sees[wave * 64 + 32 + (again(lane) & 31)];
  }
  for (; r < NR; ++r) {
    open_round(r, at);
    if (!PAPER && r == NR - 1) issue_own_keys(my_free, my_free + 4096, 0, own_tile(0));
#pragma nounroll
    for (int32_t b = SB * r; b < min(SB * r + SB, NS); ++b) {
      // what the rows see of the block: all of it, or what their bits say
      uint32_t ok = 0;
      bool masked = true, later = false;
      const bool tail = PAPER && b >= NB;
      if (!tail) {
        int32_t valid = keys_of(b);
        masked = valid < 32;
        if (PAPER && valid >= 1000) {  // a block of attribute names: the row keeps those up to its own branch's
          const int32_t k0 = valid - 1000;
          if (k0 >= names_max) continue;
          masked = true;
          valid = names_row - k0;
        }
        ok = ok_bits(valid);
      } else {
        const TileAt x = tile_at(b - NB);
        if (x.tb0 > kb_row_max) continue;
        later = x.tb0 + (31 >> x.lg) > kb_row_min;
        // a row keeps the tokens in memory of the branches up to its own
        const int lane_t = WGS == 3 ? again(lane) : lane, g2 = lane_t >> 5;
        const int32_t j_lane = x.tb0 + ((lane_t & 31) >> x.lg);
        masked = !__all(j_lane <= kb_row_min && klen[min(j_lane, kb_end - 1)] - x.c * 8 >= 1 << x.lg);
        if (masked) {
#pragma nounroll
          for (int32_t e = 0; e < 16; e += 1 << x.lg) {
            const int32_t j = x.tb0 + (((e >> 3) * 16 + g2 * 8 + (e & 7)) >> x.lg);
            const int32_t cnt = j <= kb_row ? min(klen[min(j, kb_end - 1)] - x.c * 8, 1 << x.lg) : 0;
            ok |= first_bits(cnt) << e;
          }
        }
      }
      compute(std::integral_constant<int, 1>{}, SB == 2 ? (uint32_t)(b & 3) * BLK : at, masked, ok, 0u, tail ? b - NB : -1, later);
    }
    at = behind(at);
  }
  __builtin_amdgcn_s_waitcnt(0xc07f);
  __builtin_amdgcn_s_barrier();  // the ring is the waves' own from here on
  if constexpr (!PAPER) {
    // Two workgroups per CU: a tile's keys lie in the first two pieces, its values in the last two.  Three: the keys in pieces p0,
    // p1, the first half of the values in p2, the second half follows in p0; the next tile's keys go to p1 and p2, its values to
    // p0.
    uint32_t p0 = my_free, p1 = my_free + 4096, p2 = my_last;
    TileAt x = own_tile(0);
    issue_own(v_tail, true, 0, p2, 0, x);
    if (WGS == 2) issue_own(v_tail, true, 1, p2 + 4096, 0, x);
#pragma nounroll
    for (int32_t t = 0; t < n_own; ++t) {
      const TileAt y = own_tile(t + 1);
      const int lane_t = WGS == 3 ? again(lane) : lane, n = lane_t & 31, g2 = lane_t >> 5, lb_row = wave * BPB + n / G;
      const int32_t k0 = (lb_row - x.tb0) << x.lg;  // this row's first key in the tile
      const int32_t lo = k0 - g2 * 8, hi = lo + min(a.step + 1 - x.c * 8, 1 << x.lg);
      const uint32_t ok = (k0 >= 0 && k0 < 32) ? ((first_bits(hi) & ~first_bits(lo)) |
                                                  ((first_bits(hi - 16) & ~first_bits(lo - 16)) << 8)) : 0u;
      const bool more = t + 1 < n_own;
      float s[1][16];
      f16x8 P0, P1;
      if constexpr (WGS == 2) {
        asm volatile("s_waitcnt vmcnt(8)" ::: "memory");  // the keys have landed, the values may be on their way
        settle(std::integral_constant<int, 1>{}, s, k_lane, p0, true, ok, 0u);
        __builtin_amdgcn_s_waitcnt(0xc07f);
        if (more) {
          if (PAGED && t + 2 < n_own) own_pages(t + 2);  // (in front of the keys: they have landed when those have)
          issue_own_keys(p0, p1, t + 1, y);
          asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
        } else {
          asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        }
        uint4 vf[8];
        read_tail_values(lane, p2, vf);
        __builtin_amdgcn_s_waitcnt(0xc07f);
        asm volatile("" ::: "memory");
        if (more) {
          issue_own(v_tail, true, 0, p2, t + 1, y);
          issue_own(v_tail, true, 1, p2 + 4096, t + 1, y);
        }
        weights(s[0], P0, P1);
        value_product(P0, P1, vf);
      } else {
        asm volatile("s_waitcnt vmcnt(4)" ::: "memory");
        settle(std::integral_constant<int, 1>{}, s, k_of(lane_t), n & 16 ? p1 - 4096 : p0, true, ok, 0u);
        __builtin_amdgcn_s_waitcnt(0xc07f);
        issue_own(v_tail, true, 1, p0, t, x);
        weights(s[0], P0, P1);
        uint4 vf[4];
        asm volatile("s_waitcnt vmcnt(4)" ::: "memory");
        read_tail_half(lane_t, p2, vf);
        __builtin_amdgcn_s_waitcnt(0xc07f);
        asm volatile("" ::: "memory");
        if (more) {
          if (PAGED && t + 2 < n_own) own_pages(t + 2);
          issue_own_keys(p1, p2, t + 1, y);
        }
        half_product(P0, vf);
        if (more) asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        read_tail_half(lane_t, p0, vf);
        __builtin_amdgcn_s_waitcnt(0xc07f);
        asm volatile("" ::: "memory");
        if (more) issue_own(v_tail, true, 0, p0, t + 1, y);
        half_product(P1, vf);
        const uint32_t first = p0;
        p0 = p1; p1 = p2; p2 = first;
      }
      x = y;
    }
  }

  // ---- normalise and write: as the waves of attn_stream_kernel that hold whole rows
  // (two workgroups per CU, block mask: the registers are there, 0.4 % faster)
  const int lane_o = WGS == 3 || PAPER ? again(lane) : lane, n_o = lane_o & 31, g2_o = lane_o >> 5;
  const float inv = 1.0f / (l_lane + __shfl_xor(l_lane, 32));
  uint4* const mine = reinterpret_cast<uint4*>(reinterpret_cast<char*>(ring) + my_free);  // 8 KB
  typedef uint32_t u4v __attribute__((ext_vector_type(4)));
  const int32_t rows_here = nbr_here * G;
  if (a.out_f32) {
#pragma nounroll
    for (int half = 0; half < 2; ++half) {  // 16 rows at a time
      if (n_o >> 4 == half) {
        float4* rowp = reinterpret_cast<float4*>(mine) + (n_o & 15) * 32;
#pragma unroll
        for (int blk = 0; blk < 4; ++blk)
#pragma unroll
          for (int cc = 0; cc < 4; ++cc)
            rowp[(blk * 8 + cc * 2 + g2_o) ^ n_o] = make_float4(acc[blk][cc * 4 + 0] * inv, acc[blk][cc * 4 + 1] * inv,
                                                            acc[blk][cc * 4 + 2] * inv, acc[blk][cc * 4 + 3] * inv);
      }
      __builtin_amdgcn_s_waitcnt(0xc07f);
      __builtin_amdgcn_wave_barrier();
#pragma unroll 4
      for (int32_t i = 0; i < 8; ++i) {  // 2 rows per instruction
        const int32_t rr = half * 16 + i * 2 + (lane_o >> 5), chunk = lane_o & 31, lrr = wave * 32 + rr;
        if (lrr < rows_here && lrr % G < a.Gr) {
          const uint4 v = mine[(rr & 15) * 32 + (chunk ^ rr)];
          const int64_t off = ((int64_t)(row0 + br0 + lrr / G) * a.Hq + hk * a.Gr + lrr % G) * D + chunk * 4;
          u4v vv = {v.x, v.y, v.z, v.w};
          __builtin_nontemporal_store(vv, reinterpret_cast<u4v*>(reinterpret_cast<float*>(out) + off));
        }
      }
      __builtin_amdgcn_s_waitcnt(0xc07f);
      __builtin_amdgcn_wave_barrier();
    }
  } else {
    uint2* rowp = reinterpret_cast<uint2*>(mine) + n_o * 32;
#pragma unroll
    for (int blk = 0; blk < 4; ++blk)
#pragma unroll
      for (int cc = 0; cc < 4; ++cc)
        rowp[(((blk * 4 + cc) ^ (n_o & 15)) << 1) | g2_o] =
            make_uint2(cvt_pk_bf16(acc[blk][cc * 4 + 0] * inv, acc[blk][cc * 4 + 1] * inv),
                       cvt_pk_bf16(acc[blk][cc * 4 + 2] * inv, acc[blk][cc * 4 + 3] * inv));
    __builtin_amdgcn_s_waitcnt(0xc07f);
    __builtin_amdgcn_wave_barrier();
#pragma unroll 4
    for (int32_t i = 0; i < 8; ++i) {  // 4 rows per instruction
      const int32_t rr = i * 4 + (lane_o >> 4), chunk = lane_o & 15, lrr = wave * 32 + rr;
      if (lrr < rows_here && lrr % G < a.Gr) {
        const uint4 v = mine[rr * 16 + (chunk ^ (rr & 15))];
        const int64_t off = ((int64_t)(row0 + br0 + lrr / G) * a.Hq + hk * a.Gr + lrr % G) * D + chunk * 8;
        u4v vv = {v.x, v.y, v.z, v.w};
        __builtin_nontemporal_store(vv, reinterpret_cast<u4v*>(reinterpret_cast<uint16_t*>(out) + off));
      }
    }
  }
}

template <int G, bool PAPER, bool PAGED, int WGS>
hipError_t launch_dense(const StreamArgs& a, int64_t items, const void* q, const void* k_prefix, const void* v_prefix, void* k_tail,
                        void* v_tail, const void* k_new, const void* v_new, void* out, hipStream_t s) {
  attn_dense_kernel<G, PAPER, PAGED, WGS><<<dim3((unsigned)items), DENSE_WAVES * 64, 0, s>>>(
      PAPER ? a.tb.punit_desc : a.tb.unit_desc, a.n_groups, a.RG, a.Hkv, a, (const uint16_t*)q, (const uint16_t*)k_prefix,
      (const uint16_t*)v_prefix, (uint16_t*)k_tail, (uint16_t*)v_tail, (const uint16_t*)k_new, (const uint16_t*)v_new, out);
  return hipGetLastError();
}

}  // namespace

hipError_t hpd_launch_attention_dense(const hpd_layout* L, StreamArgs a, int32_t G, bool paper, const void* q, const void* k_prefix,
                                      const void* v_prefix, void* k_tail, void* v_tail, const void* k_new, const void* v_new,
                                      void* out, hipStream_t s) {
  const hpd_dense_launch x = hpd_plan_dense_launch(L, a.step);
  if (x.grid > 0x7fffffff) return hipErrorInvalidValue;
  a.n_groups = x.n_groups;
  a.RG = x.row_groups;
  a.at_once = x.at_once;
#define HPD_DENSE_W(GG, PP, TT, WW) launch_dense<GG, PP, TT, WW>(a, x.grid, q, k_prefix, v_prefix, k_tail, v_tail, k_new, v_new, out, s)
#define HPD_DENSE_M(GG, PP, TT) (x.per_cu == 3 ? HPD_DENSE_W(GG, PP, TT, 3) : HPD_DENSE_W(GG, PP, TT, 2))
#define HPD_DENSE(GG)                                                                   \
  (paper ? a.tb.tail_pages ? HPD_DENSE_M(GG, true, true) : HPD_DENSE_M(GG, true, false) \
         : a.tb.tail_pages ? HPD_DENSE_M(GG, false, true) : HPD_DENSE_M(GG, false, false))
  switch (G) {
    case 1: return HPD_DENSE(1);
    case 2: return HPD_DENSE(2);
    case 4: return HPD_DENSE(4);
    case 8: return HPD_DENSE(8);
    default: return hipErrorInvalidValue;
  }
#undef HPD_DENSE
#undef HPD_DENSE_M
#undef HPD_DENSE_W
}
