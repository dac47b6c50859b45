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
// header, document, then the tails of the group's branches, position by position.  How many branches
// and waves a workgroup has (at most 16, 15 and 7 waves with 32, 64 and 128 channels) and which row groups
// are launched is the plan's, with the reasons and both sides' times there.  A tile is two products with v_mfma_f32_16x16x4_f32,
//     S^T[key,row] = K.Q^T   and   O^T[channel,row] += V^T.P^T,
// exact fp32 multiply-adds in both.  The K operand is one float4 per lane and 16 channels (the
// four channels of a float4 are the lane's operands of four instructions), the scores come out with
// the 4 keys 4*(lane/16) .. +3 of row lane%16 in a lane, which is how the second product takes
// them, and the 8-key interleaved V pool delivers those 4 keys of a channel in one float4.  Every
// wave keeps its own running maximum and sum per row; they meet once, through LDS.
// The step call appends in the same launch: a branch belongs to exactly one row group, which
// stores its new key and value in front of the prefix tiles and reads them behind a barrier.
// Measured (us per hpd_decode_step, generic kernels and append launch -> this): 8 prompts x 12
// branches, 16/4 heads x 64, 458 keys a row 119.2 -> 17.6 (10 MB); 4 branches, 4/4 heads x 64, 72
// keys, 8 steps in a row 12.9 -> 8.3 each, most of it the launch.  Error against 64 bits over 26
// batches: 1.3e-7 .. 2.1e-7, generic kernel 2.1e-7 .. 3.8e-7.
#include <algorithm>

#include "hpd_internal.h"
#include "hpd_device.h"

namespace {

typedef float floatx4 __attribute__((ext_vector_type(4)));
constexpr int ROWS = HPD_F32_ROWS;  // rows (branch x query head) per workgroup
template <int D>
__global__ void __launch_bounds__(hpd_f32_max_waves(D) * 64)
attention_f32_kernel(hpd_dev_tables tb, const int32_t* __restrict__ units, const int32_t* __restrict__ live,
                     const int2* __restrict__ groups, int32_t step, int32_t Hq, int32_t Hkv, int32_t Tcap, int32_t RG,
                     int32_t BPG, int64_t NP,
                     const float* __restrict__ q, const float* __restrict__ k_prefix,
                     const float* __restrict__ v_prefix, float* k_tail, float* v_tail,
                     const float* __restrict__ k_new, const float* __restrict__ v_new, float* __restrict__ out) {
  constexpr int NJ = D / 16, half = D / 2;
  extern __shared__ float smem[];
  const int n_waves = blockDim.x >> 6;
  float* const part_o = smem;                        // [waves][ROWS][D]
  float* const part_m = smem + n_waves * ROWS * D;   // [waves][ROWS]
  float* const part_l = part_m + n_waves * ROWS;     // [waves][ROWS]
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int n = lane & 15, kq = lane >> 4;

  // BPG branches per row group; unit and row group from the list if the step has one
  const int32_t G = Hq / Hkv;
  int32_t rg, hk, u;
  if (groups) {
    const int2 g = groups[blockIdx.x / Hkv];
    rg = g.y; hk = blockIdx.x % Hkv; u = g.x;
  } else {
    const int32_t grp = blockIdx.x / RG;
    rg = blockIdx.x % RG; hk = grp % Hkv; u = grp / Hkv;
  }
  const int32_t* desc = units + (int64_t)u * 8;
  const int32_t hoff = desc[0], Hlen = desc[1], doff = desc[2], Llen = desc[3], row0 = desc[4], nb = desc[5], ub0 = desc[7];
  const int32_t br0 = rg * BPG;
  if (br0 >= nb) return;  // uniform over the workgroup
  const int32_t nbh = min(BPG, nb - br0);
  auto branch_id = [&](int32_t lb) -> int32_t { return ub0 >= 0 ? ub0 + br0 + lb : live[row0 + br0 + lb]; };

  // ---- append (the arithmetic of hpd_kv_append)
  if (k_new) {
    for (int32_t i = tid; i < nbh * half; i += blockDim.x) {
      const int32_t lb = i / half, c = i % half, b = branch_id(lb);
      const float2 cs = tb.rope[(int64_t)(tb.branch_base_pos[b] + 1 + step) * half + c];
      const int64_t src = ((int64_t)(row0 + br0 + lb) * Hkv + hk) * D;
      const int64_t dst = hpd_tail_row(tb, b, hk, Hkv, Tcap, step) * D;
      float r1, r2;
      hpd::rope_pair(k_new[src + c], k_new[src + c + half], cs.x, cs.y, r1, r2);
      k_tail[dst + c] = r1;
      k_tail[dst + c + half] = r2;
      v_tail[dst + c] = v_new[src + c];
      v_tail[dst + c + half] = v_new[src + c + half];
    }
  }

  // ---- the rotated query of row n: channels 16 j + 4 kq + e (instruction 4 j + e of the first product)
  const int32_t lb_row = n / G, head = hk * G + n % G;
  const bool row_valid = lb_row < nbh;
  float Q[NJ][4];
  if (row_valid) {
    const int32_t pos = tb.branch_base_pos[branch_id(lb_row)] + 1 + step;
    const float* qp = q + ((int64_t)(row0 + br0 + lb_row) * Hq + head) * D + 4 * kq;
    const float2* cs = tb.rope + (int64_t)pos * half + 4 * kq;
#pragma unroll
    for (int j = 0; j < NJ / 2; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float2 w = cs[16 * j + e];
        hpd::rope_pair(qp[16 * j + e], qp[16 * j + e + half], w.x, w.y, Q[j][e], Q[j + NJ / 2][e]);
      }
  } else {
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) Q[j][e] = 0.f;
  }

  const float scale = 1.0f / sqrtf((float)D);
  float m = -INFINITY, l = 0.f;  // of row n over this wave's tiles; l: this lane's keys
  floatx4 O[NJ];              // channels 16 j + 4 kq + 0..3 of row n
#pragma unroll
  for (int j = 0; j < NJ; ++j) O[j] = floatx4{0.f, 0.f, 0.f, 0.f};

  // scores of a tile: value v belongs to key 4 kq + v; `ok` bit v = the row may see it
  auto weights = [&](const float4 (&K)[NJ], uint32_t ok, float (&p)[4]) {
    // a chain of 4 instructions per 16 channels, added up in pairs: a shorter chain than one over all
    // channels, and less rounding
    floatx4 C[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      C[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(K[j].x, Q[j][0], floatx4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
      C[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(K[j].y, Q[j][1], C[j], 0, 0, 0);
      C[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(K[j].z, Q[j][2], C[j], 0, 0, 0);
      C[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(K[j].w, Q[j][3], C[j], 0, 0, 0);
    }
#pragma unroll
    for (int w = NJ / 2; w > 0; w /= 2)
#pragma unroll
      for (int j = 0; j < w; ++j) C[j] += C[j + w];
    const floatx4 S = C[0];
    float bm = m;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      p[v] = (ok >> v) & 1 ? S[v] * scale : -INFINITY;
      bm = fmaxf(bm, p[v]);
    }
    bm = fmaxf(bm, __shfl_xor(bm, 16));
    bm = fmaxf(bm, __shfl_xor(bm, 32));
    const float ref = bm == -INFINITY ? 0.f : bm;  // (no key of the row yet)
    const float alpha = expf(m - ref);
    m = bm;
    l *= alpha;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      p[v] = expf(p[v] - ref);
      l += p[v];
    }
#pragma unroll
    for (int j = 0; j < NJ; ++j) O[j] *= alpha;
  };
  auto values = [&](const float4 (&V)[NJ], const float (&p)[4]) {
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      O[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(V[j].x, p[0], O[j], 0, 0, 0);
      O[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(V[j].y, p[1], O[j], 0, 0, 0);
      O[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(V[j].z, p[2], O[j], 0, 0, 0);
      O[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(V[j].w, p[3], O[j], 0, 0, 0);
    }
  };

  // ---- header and document: tiles of 16 slots (segments start on multiples of 32 slots and are
  //      padded to them; the padding's values are zero, its keys are masked)
  const int32_t nh = (Hlen + 15) >> 4, nd = (Llen + 15) >> 4;
  for (int32_t t = wave; t < nh + nd; t += n_waves) {
    const int64_t slot = t < nh ? hoff + 16 * t : doff + 16 * (t - nh);
    const int32_t cnt = t < nh ? Hlen - 16 * t : Llen - 16 * (t - nh);
    const float* kp = k_prefix + ((int64_t)hk * NP + slot + n) * D + 4 * kq;
    const float* vp = v_prefix + (((int64_t)hk * (NP / 8) + (slot + 4 * kq) / 8) * D + n) * 8 + ((4 * kq) & 7);
    float4 K[NJ], V[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j) K[j] = *reinterpret_cast<const float4*>(kp + 16 * j);
#pragma unroll
    for (int j = 0; j < NJ; ++j) V[j] = *reinterpret_cast<const float4*>(vp + 16 * 8 * j);
    float p[4];
    const int32_t mine = cnt - 4 * kq;
    weights(K, (1u << min(max(mine, 0), 4)) - 1u, p);
    values(V, p);
  }
  if (k_new) __syncthreads();  // the appended rows are visible to the workgroup

  // ---- tails: key i of the group is position i % (step + 1) of branch i / (step + 1); a row keeps
  //      the keys of its own branch.  (Handed out from the last wave down: the first ones may
  //      have a prefix tile more.)
  const int32_t len = step + 1, n_tail = nbh * len;
  for (int32_t t = n_waves - 1 - wave; t * 16 < n_tail; t += n_waves) {
    auto tail_row = [&](int32_t i) -> int64_t {
      i = min(i, n_tail - 1);
      return hpd_tail_row(tb, branch_id(i / len), hk, Hkv, Tcap, i % len) * D;
    };
    const float* kp = k_tail + tail_row(16 * t + n) + 4 * kq;
    float4 K[NJ], V[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j) K[j] = *reinterpret_cast<const float4*>(kp + 16 * j);
    uint32_t ok = 0;
    float v4[NJ][4];
    bool finite = true;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int32_t i = 16 * t + 4 * kq + v;
      const float* vp = v_tail + tail_row(i) + n;
      if (i < n_tail && i / len == lb_row) ok |= 1u << v;
#pragma unroll
      for (int j = 0; j < NJ; ++j) {
        v4[j][v] = vp[16 * j];
        finite = finite && fabsf(v4[j][v]) < INFINITY;
      }
    }
    float p[4];
    weights(K, ok, p);
    if (!__any(!finite)) {
#pragma unroll
      for (int j = 0; j < NJ; ++j) V[j] = make_float4(v4[j][0], v4[j][1], v4[j][2], v4[j][3]);
      values(V, p);
    } else {
      // an infinite or NaN value must not reach the rows of other branches as 0 * value: one branch
      // at a time, and only its rows take the result
      for (int32_t b = 16 * t / len; b <= min(16 * t + 15, n_tail - 1) / len; ++b) {
        floatx4 keep[NJ];
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
          keep[j] = O[j];
          float w[4];
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const int32_t i = 16 * t + 4 * kq + v;
            w[v] = i < n_tail && i / len == b ? v4[j][v] : 0.f;
          }
          V[j] = make_float4(w[0], w[1], w[2], w[3]);
        }
        values(V, p);
        if (lb_row != b) {
#pragma unroll
          for (int j = 0; j < NJ; ++j) O[j] = keep[j];
        }
      }
    }
  }

  // ---- the waves' shares meet
  l += __shfl_xor(l, 16);
  l += __shfl_xor(l, 32);
  float* const po = part_o + (wave * ROWS + n) * D + 4 * kq;
#pragma unroll
  for (int j = 0; j < NJ; ++j) *reinterpret_cast<floatx4*>(po + 16 * j) = O[j];
  if (kq == 0) {
    part_m[wave * ROWS + n] = m;
    part_l[wave * ROWS + n] = l;
  }
  __syncthreads();
  for (int32_t i = tid; i < nbh * G * D; i += blockDim.x) {
    const int32_t r = i / D, c = i % D;
    float mm = -INFINITY;
    for (int w = 0; w < n_waves; ++w) mm = fmaxf(mm, part_m[w * ROWS + r]);
    float o = 0.f, ll = 0.f;
    for (int w = 0; w < n_waves; ++w) {
      const float e = expf(part_m[w * ROWS + r] - mm);
      ll = fmaf(part_l[w * ROWS + r], e, ll);
      o = fmaf(part_o[(w * ROWS + r) * D + c], e, o);
    }
    out[((int64_t)(row0 + br0 + r / G) * Hq + hk * G + r % G) * D + c] = o / ll;
  }
}

template <int D>
hipError_t launch(const hpd_layout* L, int32_t step, const void* q, const void* k_prefix, const void* v_prefix,
                  void* k_tail, void* v_tail, const void* k_new, const void* v_new, void* out, hipStream_t s) {
  const int32_t Hq = L->cfg.n_q_heads, Hkv = L->cfg.n_kv_heads;
  const hpd_f32_step& st = L->f32_steps[step];
  const size_t lds = (size_t)st.waves * ROWS * (D + 2) * sizeof(float);
  const int64_t grid = st.groups * Hkv;
  if (grid > 0x7fffffff) return hipErrorInvalidValue;
  const int2* groups = st.rg ? nullptr : reinterpret_cast<const int2*>(L->dev.f32_groups) + st.list;
  attention_f32_kernel<D><<<dim3((unsigned)grid), st.waves * 64, lds, s>>>(
      L->dev, L->dev.unit_desc + (int64_t)L->unit_ptr[step] * 8, L->dev.live_branch + L->live_ptr[step], groups, step,
      Hq, Hkv, L->T, st.rg, st.per_group, L->NP, (const float*)q, (const float*)k_prefix, (const float*)v_prefix,
      (float*)k_tail, (float*)v_tail, (const float*)k_new, (const float*)v_new, (float*)out);
  return hipGetLastError();
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
