// fp32 decode attention on the fp32 matrix instruction (gfx950): hpd_decode_attention and
// hpd_decode_step of fp32 layouts under the block mask, 32, 64 or 128 channels, up to 16 query
// heads per kv head.  Everything else in fp32 runs the generic kernel of hpd_kernels.hip, and so do the
// steps for which the layout's plan (plan_f32 in hpd_host.cpp) finds it faster: few rows and few keys per
// workgroup, and many workgroups.
//
// What bounds it is latency: a decode step of a small fp32 batch moves a few megabytes, and the
// generic kernel (one workgroup per row and query head) spends its time in chains of dependent
// 4-byte loads, one per key and thread.  Here a workgroup takes 16 rows (query heads of
// consecutive live branches of one document) of one kv head, and its waves share out the tiles of 16 keys:
// header, document, then the earlier tokens of the branches, branch by branch.  How many branches and waves a
// workgroup has and which row groups are launched is the plan's, with the reasons and both sides' times there.  A tile is two products with v_mfma_f32_16x16x4_f32,
//     S^T[key,row] = K.Q^T   and   O^T[channel,row] += V^T.P^T,
// exact fp32 multiply-adds in both.  The K operand is one float4 per lane and 16 channels (the
// four channels of a float4 are the lane's operands of four instructions), the scores come out with
// the 4 keys 4*(lane/16) .. +3 of row lane%16 in a lane, which is how the second product takes
// them, and the 8-key interleaved V pool delivers those 4 keys of a channel in one float4.  Every
// wave keeps its own running maximum and sum per row; they meet once, through LDS.
// The chain of latencies is kept short, and with it the number of instructions (a wave alone on its SIMD issues one
// every 5 to 8 cycles):
//  * tiles go from memory to LDS (global_load_lds_dwordx4, 1 KB of whole rows an instruction) and from there into
//    operand layout.  A load straight into operand layout has its 16 rows in 16 consecutive lanes: the memory pipeline
//    takes such an instruction apart lane by lane (82 cycles each were measured, for data in the L2; whole rows 16),
//    and 250 KB of K and V took 10 us;
//  * what the descriptor's lookup takes are the first arguments, in registers when the kernel starts (11.4 -> 11.1 us);
//  * a wave requests its first tile as soon as it has the unit's descriptor, in front of the query, and the
//    next tile as soon as it has read the one it works on;
//  * the query is rotated once, by all waves together, and shared through LDS (in operand layout from memory in every
//    wave: 8 scattered instructions in each of 16 waves, 4 us);
//  * the newest token of a branch is seen by the branch's own rows only: it is no tile but the state that the last wave
//    starts from (weight 1, its value the result).  In the step call it is rotated, shared and stored along with the
//    query: there is no wait for the append in front of the tails;
//  * the waves' shares lie in LDS in rows of D + 4 floats (with D floats the 16 rows of a store share their banks), and a
//    wave merges a row at a time, its 16 lanes working out the weight of each share once;
//  * the row groups of one (unit, kv head), which read the same prefix, run on one XCD, out of one L2.
// Measured (us per hpd_decode_step; generic kernels and append launch -> one launch, loads into operand layout, a
// barrier between the append and the tails -> this): 8 prompts x 12 branches, 16/4 heads x 64, 458 keys a row, 119.2 ->
// 17.6 -> 11.4; 256 documents of 512 keys, 12 branches, 16/4 heads x 64, 4218 -> 247 -> 148, x 128 8400 -> 487 -> 254; 2000
// documents of 12..384 keys, 1..24 branches, 12065 -> 1936 -> 1046; 4 branches, 4/4 heads x 64, 72 keys, the kernel alone,
// 7.0 -> 5.4 (1.0 until the descriptor is there, 1.4 more until the query is shared, 2.1 for the tiles, 0.8 to merge).
// Over 2000 random batches 1.39 times the speed with loads into operand layout in the mean; 21 are slower, down to 0.82: launches
// of thousands of workgroups with 32 channels and one or two tiles, documents of a few keys without a header (526 of up to
// 9 keys, 8/2 heads, 11.5 -> 13.9 us; 476 of one or two keys, 64/8 heads, 116 -> 133).
// Error against 64 bits over 25 batches: 1.4e-7 .. 2.0e-7, before 1.3e-7 .. 2.1e-7 (0.998 of it in the mean), generic kernel 2.1e-7
// .. 3.8e-7.
#include <algorithm>

#include "hpd_internal.h"
#include "hpd_device.h"

namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx4u __attribute__((ext_vector_type(4), aligned(4)));  // four floats of a caller's tensor
constexpr int ROWS = HPD_F32_ROWS;  // rows (branch x query head) per workgroup

// over the four lanes (16 apart) that hold a row; over 16 consecutive lanes
template <typename F>
__device__ __forceinline__ float over_row(float x, F f) {
  auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = f(__uint_as_float(a[0]), __uint_as_float(a[1]));
  a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return f(__uint_as_float(a[0]), __uint_as_float(a[1]));
}
template <typename F>
__device__ __forceinline__ float over_16(float x, F f) {
  x = f(x, __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), 0x128, 0xf, 0xf, false)));  // row_ror:8
  x = f(x, __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), 0x124, 0xf, 0xf, false)));
  x = f(x, __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), 0x122, 0xf, 0xf, false)));
  return f(x, __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(x), 0x121, 0xf, 0xf, false)));
}
__device__ __forceinline__ float add(float a, float b) { return a + b; }
__device__ __forceinline__ float larger(float a, float b) { return fmaxf(a, b); }

// A tile in LDS: 16 keys of D floats, then as many floats of values.
//   keys              row = key, its 16-byte chunk c at position c ^ swizzle(key): the 16 rows of a read differ in their banks
//   values, prefix    as the pool has them, [key / 8][channel][key % 8]: chunk i at position i ^ (i / 16 % 2)
//   values, tails     row = key, the 16 channels j at position j ^ key / 4
// An instruction fills 1 KB from consecutive lanes.  Two of them, LDS bytes `lds` and `lds` + 1024 on: their offset
// moves the address in LDS and the one in memory alike.  (Written out because the compiler makes every LDS read of a
// wave wait for all loads to LDS that the wave has in flight.)
__device__ __forceinline__ void dma2(uint32_t lds, const float* base, uint32_t o0, uint32_t o1) {  // base: one for the wave
  const uint64_t b = reinterpret_cast<uint64_t>(base);
  const uint64_t u = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int32_t)(b >> 32)) << 32 |
                     (uint32_t)__builtin_amdgcn_readfirstlane((int32_t)(uint32_t)b);
  uint32_t keep;  // M0 is the compiler's: put back what it held
  asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %3\n\ts_nop 0\n\t"
               "global_load_lds_dwordx4 %1, %4\n\tglobal_load_lds_dwordx4 %2, %4 offset:1024\n\t"
               "s_mov_b32 m0, %0"
               : "=&s"(keep) : "v"(o0), "v"(o1 - 1024u), "s"(lds), "s"(u) : "memory");
}
__device__ __forceinline__ void dma2(uint32_t lds, const float* p0, const float* p1) {
  uint32_t keep;
  asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %3\n\ts_nop 0\n\t"
               "global_load_lds_dwordx4 %1, off\n\tglobal_load_lds_dwordx4 %2, off offset:1024\n\t"
               "s_mov_b32 m0, %0"
               : "=&s"(keep) : "v"(p0), "v"(p1 - 256), "s"(lds) : "memory");
}
__device__ __forceinline__ void dma_dword(uint32_t lds, const float* p) {  // 256 bytes
  uint32_t keep;
  asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %2\n\ts_nop 0\n\t"
               "global_load_lds_dword %1, off\n\t"
               "s_mov_b32 m0, %0"
               : "=&s"(keep) : "v"(p), "s"(lds) : "memory");
}

template <int D>
__global__ void __launch_bounds__(hpd_f32_max_waves(D) * 64, D == 32 ? 6 : D == 64 ? 4 : 2)
attention_f32_kernel(const int32_t* __restrict__ units, const int2* __restrict__ groups, int32_t group0, int32_t width, int32_t n_groups, int32_t Hkv,
                     int32_t BPG, hpd_dev_tables tb, const int32_t* __restrict__ live, int32_t step, uint32_t step_magic, int32_t Hq,
                     int32_t G, uint32_t g_magic, int32_t Tcap, int64_t NP,
                     const float* __restrict__ q, const float* __restrict__ k_prefix,
                     const float* __restrict__ v_prefix, float* k_tail, float* v_tail,
                     const float* __restrict__ k_new, const float* __restrict__ v_new, float* __restrict__ out) {
  constexpr int NJ = D / 16, half = D / 2, CH = D / 4, PAD = D + HPD_F32_PAD, WAVE_FLOATS = 32 * D;
  extern __shared__ float smem[];
  const int n_waves = blockDim.x >> 6;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int n = lane & 15, kq = lane >> 4;
  // this wave's part of LDS: its tile; at the end its share of the result, ROWS x PAD floats, then maxima and sums
  float* const tile = smem + wave * WAVE_FLOATS;
  constexpr int PART_M = ROWS * PAD, PART_L = PART_M + ROWS;
  static_assert(PART_L + ROWS <= WAVE_FLOATS, "the share fits the place of the tile");

  // BPG branches per row group; unit and row group from the list if the step has one, otherwise from the workgroup's
  // number (it runs on XCD number % 8)
  const int32_t item = (group0 + blockIdx.z) * width + blockIdx.x;
  if (item >= n_groups) return;  // the grid is padded to a multiple of 8 (unit, kv head)
  const int32_t hk = item % Hkv;
  int32_t u = item / Hkv, rg = blockIdx.y;
  if (groups) {
    const int2 g = groups[u];
    u = g.x;
    rg = g.y;
  }
  const int32_t* desc = units + (int64_t)u * 8;
  const int32_t hoff = desc[0], Hlen = desc[1], doff = desc[2], Llen = desc[3], row0 = desc[4], nb = desc[5];
  const int32_t upos = desc[6], ub0 = desc[7];
  const int32_t br0 = rg * BPG;
  if (br0 >= nb) return;  // uniform over the workgroup
  const int32_t nbh = min(BPG, nb - br0);
  auto branch_id = [&](int32_t lb) -> int32_t { return ub0 >= 0 ? ub0 + br0 + lb : live[row0 + br0 + lb]; };
  auto row_branch = [&](int32_t r) -> int32_t { return (int32_t)((uint32_t)r * g_magic >> 8); };  // r / G
  const int32_t lb_row = row_branch(n);  // branch of row n
  // row of token t of a branch of the group in the tail pools (32 bits hold the rows of any pool that fits the memory)
  auto tail_row = [&](int32_t lb, int32_t t) -> uint32_t {
    const uint32_t b = (uint32_t)branch_id(lb);
    uint32_t row = (b * (uint32_t)Hkv + (uint32_t)hk) * (uint32_t)Tcap + (uint32_t)t;
    if (tb.tail_pages) {  // as hpd_tail_row
      int32_t pg = tb.tail_pages[(int64_t)b * tb.pages_per_branch + (t >> tb.page_shift)];
      pg = min(max(pg, 0), tb.n_pages - 1);
      row = (((uint32_t)pg * (uint32_t)Hkv + (uint32_t)hk) << tb.page_shift) + (uint32_t)(t & ((1 << tb.page_shift) - 1));
    }
    return row;
  };

  // ---- tiles: header and document (16 slots each: segments start on multiples of 32 slots and are padded to them;
  //      the padding's values are zero, its keys are masked), then the earlier tokens of the branches, key i being
  //      position i % step of branch i / step
  const int32_t nh = (Hlen + 15) >> 4, nd = (Llen + 15) >> 4, n_tail = nbh * step;
  const int32_t n_tiles = nh + nd + ((n_tail + 15) >> 4);
  auto prefix_slot = [&](int32_t t) -> int64_t { return t < nh ? hoff + 16 * t : doff + 16 * (t - nh); };
  auto tail_branch = [&](int32_t i) -> int32_t { return step == 1 ? i : (int32_t)__umulhi((uint32_t)i, step_magic); };
  const uint32_t k_lds = (uint32_t)reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) char*)tile);
  const uint32_t v_lds = k_lds + 64 * D;
  auto swizzle = [](int32_t key) -> int32_t { return D == 32 ? key >> 1 : key; };
  // instruction f of a tile fills the chunks 64 f + lane: of row 64 f / CH + lane / CH, position lane % CH
  constexpr int RPI = 64 / CH;  // rows per instruction
  uint32_t rows[NJ];  // pool rows of a tail tile's keys f * RPI + lane / CH
  // (a lane's addresses are worked out for every tile: kept, they cost more registers than there are)
  auto request_keys = [&](int32_t t) {
    int32_t x = lane;
    asm volatile("" : "+v"(x));
    const int32_t my_row = x / CH, my_pos = x % CH;
    if (t < nh + nd) {
      const float* kp = k_prefix + ((int64_t)hk * NP + prefix_slot(t)) * D;
#pragma unroll
      for (int f = 0; f < NJ; f += 2) {
        const int32_t r0 = f * RPI + my_row, r1 = r0 + RPI;
        dma2(k_lds + f * 1024, kp, 16 * (r0 * CH + (my_pos ^ swizzle(r0))), 16 * (r1 * CH + (my_pos ^ swizzle(r1))));
      }
      return;
    }
    const int32_t t0 = 16 * (t - nh - nd);
#pragma unroll
    for (int f = 0; f < NJ; ++f) {
      const int32_t i = min(t0 + f * RPI + my_row, n_tail - 1), b = tail_branch(i);
      rows[f] = tail_row(b, i - b * step);
    }
#pragma unroll
    for (int f = 0; f < NJ; f += 2) {
      const int32_t r0 = f * RPI + my_row, r1 = r0 + RPI;
      dma2(k_lds + f * 1024, k_tail + ((uint64_t)rows[f] * D + 4 * (my_pos ^ swizzle(r0))),
           k_tail + ((uint64_t)rows[f + 1] * D + 4 * (my_pos ^ swizzle(r1))));
    }
  };
  auto request_values = [&](int32_t t) {
    int32_t x = lane;
    asm volatile("" : "+v"(x));
    const int32_t my_row = x / CH, my_pos = x % CH;
    if (t < nh + nd) {
      const float* vp = v_prefix + ((int64_t)hk * NP + prefix_slot(t)) * D;
      const uint32_t at = 16 * (x ^ (x >> 4 & 1));
#pragma unroll
      for (int f = 0; f < NJ; f += 2) dma2(v_lds + f * 1024, vp, f * 1024 + at, f * 1024 + 1024 + at);
      return;
    }
    auto channel = [&](int32_t row, int32_t pos) -> int32_t { return pos ^ 16 * (row >> 2 & (NJ - 1)); };
    if (((uintptr_t)v_tail & 15) == 0) {
#pragma unroll
      for (int f = 0; f < NJ; f += 2) {
        const int32_t r0 = f * RPI + my_row, r1 = r0 + RPI;
        dma2(v_lds + f * 1024, v_tail + ((uint64_t)rows[f] * D + channel(r0, 4 * my_pos)),
             v_tail + ((uint64_t)rows[f + 1] * D + channel(r1, 4 * my_pos)));
      }
    } else {  // a float per lane; the lanes that requested a row's keys have its place in the pools
#pragma unroll
      for (int f = 0; f < NJ; ++f) {
#pragma nounroll
        for (int32_t first = f * 256; first < f * 256 + 256; first += 64) {
          const int32_t row = (first + x) / D;
          const uint32_t at = __shfl(rows[f], (row % RPI) * CH);
          dma_dword(v_lds + 4 * first, v_tail + ((uint64_t)at * D + channel(row, (first + x) % D)));
        }
      }
    }
  };
  // wave w takes tiles w, w + waves, ..
  const bool last = wave == n_waves - 1;
  if (wave < n_tiles && !last) {
    request_keys(wave);
    request_values(wave);
  }

  // ---- the rotated query, and the branches' newest tokens: from the caller, rotated and appended (the arithmetic of
  //      hpd_kv_append), or from the pools.  Rows of chunks as those of a tile; the newest tokens lie where the last
  //      wave's tile will.
  float* const rot_q = smem + n_waves * WAVE_FLOATS;  // [ROWS][D]
  float* const new_k = smem + (n_waves - 1) * WAVE_FLOATS;
  float* const new_v = new_k + 16 * D;
  auto place = [&](int32_t row, int32_t c) -> int32_t { return row * D + (4 * (c / 4 ^ swizzle(row)) | c % 4); };
  auto angles = [&](int32_t lb, int32_t c) -> float2 {
    const int32_t pos = upos >= 0 ? upos : tb.branch_base_pos[branch_id(lb)] + 1 + step;
    return tb.rope[(int64_t)pos * half + c];
  };
  // scores in log2 units.  (The product with a key's score is exact inside fma, so the exponents carry one rounding
  // of their own size, and the constant's error is the same for all keys.)
  const float scale = (float)(1.4426950408889634 / sqrt((double)D));
  for (int32_t i = tid; i < ROWS * half; i += n_waves * 64) {
    const int32_t r = i / half, c = i % half, lb = row_branch(r);
    if (lb < nbh) {
      const float* x = q + ((int64_t)(row0 + br0 + lb) * Hq + hk * G + (r - lb * G)) * D + c;
      const float2 cs = angles(lb, c);
      hpd::rope_pair(x[0], x[half], cs.x, cs.y, rot_q[place(r, c)], rot_q[place(r, c + half)]);
    }
  }
  for (int32_t i = tid; i < nbh * half; i += n_waves * 64) {
    const int32_t lb = i / half, c = i % half;
    const int64_t src = ((int64_t)(row0 + br0 + lb) * Hkv + hk) * D + c;
    const uint64_t at = (uint64_t)tail_row(lb, step) * D + c;
    float k1, k2, v1, v2;
    if (k_new) {
      const float2 cs = angles(lb, c);
      v1 = v_new[src];
      v2 = v_new[src + half];
      hpd::rope_pair(k_new[src], k_new[src + half], cs.x, cs.y, k1, k2);
      k_tail[at] = k1;
      k_tail[at + half] = k2;
      v_tail[at] = v1;
      v_tail[at + half] = v2;
    } else {
      k1 = k_tail[at];
      k2 = k_tail[at + half];
      v1 = v_tail[at];
      v2 = v_tail[at + half];
    }
    new_k[place(lb, c)] = k1;
    new_k[place(lb, c + half)] = k2;
    new_v[place(lb, c)] = v1;
    new_v[place(lb, c + half)] = v2;
  }
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // (__syncthreads() would wait for the tiles and the stores, too)
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");

  float m = -INFINITY, l = 0.f;  // of row n over this wave's tiles; l: this lane's keys
  floatx4 O[NJ];              // channels 16 j + 4 kq + 0..3 of row n
  floatx4 Q[NJ];              // channels 16 j + 4 kq + e (instruction 4 j + e of the first product)
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    O[j] = floatx4{0.f, 0.f, 0.f, 0.f};
    Q[j] = lb_row < nbh ? *reinterpret_cast<const floatx4*>(rot_q + place(n, 16 * j + 4 * kq)) : O[j];
  }
  if (last) {
    if (lb_row < nbh) {
      floatx4 c = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const floatx4 K = *reinterpret_cast<const floatx4*>(new_k + place(lb_row, 16 * j + 4 * kq));
        O[j] = *reinterpret_cast<const floatx4*>(new_v + place(lb_row, 16 * j + 4 * kq));
#pragma unroll
        for (int e = 0; e < 4; ++e) c[e] = fmaf(K[e], Q[j][e], c[e]);
      }
      m = over_row((c[0] + c[1]) + (c[2] + c[3]), add) * scale;
      l = kq == 0 ? 1.f : 0.f;
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    if (wave < n_tiles) {
      request_keys(wave);
      request_values(wave);
    }
  }

  auto value_product = [](const floatx4& V, const float (&p)[4], floatx4 o) -> floatx4 {
    o = __builtin_amdgcn_mfma_f32_16x16x4f32(V[0], p[0], o, 0, 0, 0);
    o = __builtin_amdgcn_mfma_f32_16x16x4f32(V[1], p[1], o, 0, 0, 0);
    o = __builtin_amdgcn_mfma_f32_16x16x4f32(V[2], p[2], o, 0, 0, 0);
    return __builtin_amdgcn_mfma_f32_16x16x4f32(V[3], p[3], o, 0, 0, 0);
  };
  for (int32_t t = wave; t < n_tiles; t += n_waves) {
    const int32_t next = t + n_waves;
    const bool tail = t >= nh + nd;
    // ---- scores: value v of a lane belongs to key 4 kq + v, and `ok` says whether row n sees it
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(NJ) : "memory");  // the keys have landed; the values may be on their way
    floatx4 C[NJ];
    {
      floatx4 K[NJ];
#pragma unroll
      for (int j = 0; j < NJ; ++j) K[j] = *reinterpret_cast<const floatx4*>(tile + n * D + 4 * ((4 * j + kq) ^ swizzle(n)));
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // read: their place is free
      // a chain of 4 instructions per 16 channels, added up in pairs: a shorter chain than one over all
      // channels, and less rounding
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
          C[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(K[j][e], Q[j][e], e ? C[j] : floatx4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
    }
    uint32_t ok, owner = 0;  // owner, tails: byte v = the branch of key 4 kq + v, counted in the row group, or 255
    if (!tail) {
      const int32_t mine = (t < nh ? Hlen - 16 * t : Llen - 16 * (t - nh)) - 4 * kq;
      ok = (1u << min(max(mine, 0), 4)) - 1u;
    } else {
      ok = 0;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int32_t i = 16 * (t - nh - nd) + 4 * kq + v, b = i < n_tail ? tail_branch(i) : 255;
        owner |= (uint32_t)b << (8 * v);
        ok |= (uint32_t)(b == lb_row) << v;
      }
    }
    // the values of this tile are read with the addresses of its keys; those of the next one come after
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    floatx4 V[NJ];
    if (!tail) {
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        const int32_t i = kq / 2 * 2 * D + (16 * j + n) * 2 + (kq & 1);
        V[j] = *reinterpret_cast<const floatx4*>(tile + 16 * D + 4 * (i ^ (i >> 4 & 1)));
      }
    } else {
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) V[j][v] = tile[16 * D + (4 * kq + v) * D + 16 * (j ^ (kq & (NJ - 1))) + n];
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    if (next < n_tiles) {
      request_keys(next);
      request_values(next);
    }
#pragma unroll
    for (int w = NJ / 2; w > 0; w /= 2)
#pragma unroll
      for (int j = 0; j < w; ++j) C[j] += C[j + w];
    float p[4], bm = m;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      p[v] = (ok >> v) & 1 ? C[0][v] : -INFINITY;
      bm = fmaxf(bm, p[v] * scale);
    }
    bm = over_row(bm, larger);
    const float ref = bm == -INFINITY ? 0.f : bm;  // (no key of the row yet)
    const float alpha = __builtin_amdgcn_exp2f(m - ref);
    m = bm;
    l *= alpha;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      p[v] = __builtin_amdgcn_exp2f(fmaf(p[v], scale, -ref));
      l += p[v];
    }
#pragma unroll
    for (int j = 0; j < NJ; ++j) O[j] *= alpha;
    bool finite = true;
    if (tail) {
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int v = 0; v < 4; ++v) finite = finite && fabsf(V[j][v]) < INFINITY;
    }
    if (!__any(!finite)) {
#pragma unroll
      for (int j = 0; j < NJ; ++j) O[j] = value_product(V[j], p, O[j]);
    } else {
      // an infinite or NaN value must not reach the rows of other branches as 0 * value: one branch
      // at a time, and only its rows take the result
#pragma nounroll
      for (int32_t b = 0; b < nbh; ++b) {
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
          floatx4 x;
#pragma unroll
          for (int v = 0; v < 4; ++v) x[v] = (int32_t)(owner >> (8 * v) & 255) == b ? V[j][v] : 0.f;
          const floatx4 o = value_product(x, p, O[j]);
          if (lb_row == b) O[j] = o;
        }
      }
    }
  }

  // ---- the waves' shares meet: a wave takes a row at a time, lane w (of every 16) the share of wave w, then
  //      lane c the channels c, c + 64
  l = over_row(l, add);
#pragma unroll
  for (int j = 0; j < NJ; ++j) *reinterpret_cast<floatx4*>(tile + n * PAD + 4 * kq + 16 * j) = O[j];
  if (kq == 0) {
    tile[PART_M + n] = m;
    tile[PART_L + n] = l;
  }
  __syncthreads();
  for (int32_t r = wave; r < nbh * G; r += n_waves) {
    const float* const mine = smem + min(n, n_waves - 1) * WAVE_FLOATS + r;
    const float m_mine = mine[PART_M], l_mine = mine[PART_L];
    const float mm = over_16(m_mine, larger);
    const float e_mine = n < n_waves ? __builtin_amdgcn_exp2f(m_mine - mm) : 0.f;
    const float ll = over_16(n < n_waves ? l_mine * e_mine : 0.f, add);
    // (all shares are requested before the first one is used)
    constexpr int NC = (D + 63) / 64, W = hpd_f32_max_waves(D);
    const float* src = smem + r * PAD + min(lane, D - 1);
    float x[W][NC], o[NC];
#pragma unroll
    for (int w = 0; w < W; ++w)
#pragma unroll
      for (int c = 0; c < NC; ++c) x[w][c] = src[min(w, n_waves - 1) * WAVE_FLOATS + 64 * c];
#pragma unroll
    for (int c = 0; c < NC; ++c) o[c] = 0.f;
#pragma unroll
    for (int w = 0; w < W; ++w) {
      const float e = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(e_mine), w));
      if (w < n_waves) {
#pragma unroll
        for (int c = 0; c < NC; ++c) o[c] = fmaf(x[w][c], e, o[c]);
      }
    }
    const int32_t lb = row_branch(r);
    float* const dst = out + ((int64_t)(row0 + br0 + lb) * Hq + hk * G + (r - lb * G)) * D + lane;
    if (lane < D) {
#pragma unroll
      for (int c = 0; c < NC; ++c) dst[64 * c] = o[c] / ll;
    }
  }
}

template <int D>
hipError_t launch(const hpd_layout* L, int32_t step, const void* q, const void* k_prefix, const void* v_prefix,
                  void* k_tail, void* v_tail, const void* k_new, const void* v_new, void* out, hipStream_t s) {
  const int32_t Hq = L->cfg.n_q_heads, Hkv = L->cfg.n_kv_heads, G = Hq / Hkv;
  const hpd_f32_step& st = L->f32_steps[step];
  const size_t lds = ((size_t)st.waves * 32 + ROWS) * D * sizeof(float);
  // (st.rg: st.groups / st.rg units with rg row groups each)
  const int32_t rg = std::max(st.rg, 1);
  const int64_t n_groups = st.groups / rg * Hkv, octets = (n_groups + 7) / 8;
  if (octets > 0x7fffffff / 8) return hipErrorInvalidValue;
  const int2* groups = st.rg ? nullptr : reinterpret_cast<const int2*>(L->dev.f32_groups) + st.list;
  // i / step = the high half of i * magic for step > 1 and i * step < 2^32: the keys of a group, i < 16 * step, with
  // at most 15000 keys per row
  const uint32_t magic = step > 1 ? (uint32_t)((((uint64_t)1 << 32) + step - 1) / step) : 0;
  // (x and y of a grid go together: one (unit, kv head) on each XCD, its row groups one after the other.  Where that leaves
  // a tenth of the XCDs' places empty and gives an XCD more workgroups than it has CUs, row groups go to the XCDs in turn:
  // one document of 666 keys, 50 branches, 32/2 heads x 64, step 55, 27.1 us on two XCDs, 14.4 on eight; but 35 documents
  // with 5 row groups, 16/1 heads x 128, 15.1 on one XCD each, 17.9 in turn.  The plan lists the groups from 65536 per unit
  // on, z is at most 65535.)
  const bool in_turn = 10 * n_groups < 9 * 8 * octets && octets * rg * 8 > L->n_cus;
  const int64_t layers = in_turn ? 1 : octets;
  for (int64_t z = 0; z < layers; z += 65535) {
    attention_f32_kernel<D><<<dim3(in_turn ? (unsigned)n_groups : 8u, (unsigned)rg, (unsigned)std::min<int64_t>(layers - z, 65535)),
                              st.waves * 64, lds, s>>>(
        L->dev.unit_desc + (int64_t)L->unit_ptr[step] * 8, groups, (int32_t)z, in_turn ? (int32_t)n_groups : 8, (int32_t)n_groups, Hkv,
        st.per_group, L->dev, L->dev.live_branch + L->live_ptr[step], step, magic, Hq, G, (uint32_t)(256 + G - 1) / G, L->T, L->NP,
        (const float*)q,
        (const float*)k_prefix, (const float*)v_prefix, (float*)k_tail, (float*)v_tail, (const float*)k_new,
        (const float*)v_new, (float*)out);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace

hipError_t hpd_launch_attention_f32(const hpd_layout* L, int32_t step, const void* q, const void* k_prefix,
                                    const void* v_prefix, void* k_tail, void* v_tail, const void* k_new,
                                    const void* v_new, void* out, hipStream_t s) {
  switch (L->cfg.head_dim) {
    case 32: return launch<32>(L, step, q, k_prefix, v_prefix, k_tail, v_tail, k_new, v_new, out, s);
    case 64: return launch<64>(L, step, q, k_prefix, v_prefix, k_tail, v_tail, k_new, v_new, out, s);
    case 128: return launch<128>(L, step, q, k_prefix, v_prefix, k_tail, v_tail, k_new, v_new, out, s);
    default: return hipErrorInvalidValue;
  }
}
