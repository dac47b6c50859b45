// Host-side exerciser for a sanitizer build (-fsanitize=address,undefined on the host pass) of
// hpd_host.cpp: random valid and invalid batch descriptions through hpd_build_layout with
// HPD_FLAG_HOST_ONLY (no GPU call), every table read back into a buffer of exactly the
// reported size, the host-side argument checks of the other entry points.  The kernel
// launchers are stubbed out: nothing here may reach them.  Exit code 0 = no finding; a
// sanitizer report aborts the program.
#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <functional>
#include <limits>
#include <numeric>
#include <random>
#include <vector>

#include "hpd_internal.h"

static int g_stub_calls = 0;
#define STUB(...) { ++g_stub_calls; return hipErrorInvalidValue; }
hipError_t hpd_launch_prefix_fill(const hpd_layout*, const void*, const void*, void*, void*, hipStream_t) STUB()
hipError_t hpd_launch_positions(const hpd_layout*, int32_t, int32_t*, hipStream_t) STUB()
hipError_t hpd_launch_append(const hpd_layout*, int32_t, const void*, const void*, void*, void*, int64_t*,
                             hipStream_t) STUB()
hipError_t hpd_launch_attention_generic(const hpd_layout*, int32_t, const void*, const void*, const void*,
                                        const void*, const void*, void*, hipStream_t) STUB()
hipError_t hpd_launch_expand_mask(const int32_t*, int32_t, int32_t, uint8_t*, hipStream_t) STUB()
hipError_t hpd_launch_finetune_mask(const int32_t*, int32_t, int32_t*, uint8_t*, hipStream_t) STUB()
int64_t hpd_generic_max_keys(const hpd_layout*, int32_t) { ++g_stub_calls; return 0; }
bool hpd_stream_supported(const hpd_layout*) { return false; }
hipError_t hpd_launch_prefill_stream(const hpd_layout*, const void*, const void*, const void*, void*, hipStream_t) STUB()
hipError_t hpd_launch_prefill_generic(const hpd_layout*, const void*, const void*, const void*, void*, hipStream_t) STUB()
hipError_t hpd_launch_attention_stream(const hpd_layout*, int32_t, const void*, const void*, const void*, void*,
                                       void*, const void*, const void*, void*, hipStream_t, bool) STUB()
hipError_t hpd_launch_attention_f32(const hpd_layout*, int32_t, const void*, const void*, const void*, void*, void*,
                                    const void*, const void*, void*, hipStream_t) STUB()
hipError_t hpd_launch_dynamic_prune(const hpd_layout*, int32_t, const uint8_t*, hipStream_t) STUB()
hipError_t hpd_dynamic_scratch(int, void**, size_t*) STUB()

#define CHECK(cond)                                                          \
  do {                                                                       \
    if (!(cond)) {                                                           \
      std::fprintf(stderr, "CHECK failed at line %d: %s\n", __LINE__, #cond); \
      std::exit(1);                                                          \
    }                                                                        \
  } while (0)

// reads a table into a heap buffer of exactly `n` elements: one element too many written by the
// library is a heap-buffer-overflow report
template <typename T>
static std::vector<T> query(const hpd_layout* L, int32_t what, size_t n) {
  std::vector<T> v(n);
  T dummy;
  CHECK(hpd_layout_query(L, what, n ? (void*)v.data() : (void*)&dummy, n * sizeof(T)) == HPD_OK);
  if (n > 0) CHECK(hpd_layout_query(L, what, v.data(), n * sizeof(T) - 1) == HPD_E_INVALID);
  return v;
}

// every row group of a step is launched exactly once: by its number, or by one pair of a list inside f32_groups
static bool check_f32_steps(const hpd_layout* L) {
  bool listed = false;
  for (size_t t = 0; t < L->f32_steps.size(); ++t) {
    const hpd_f32_step& s = L->f32_steps[t];
    const int32_t G = L->cfg.n_q_heads / L->cfg.n_kv_heads, u0 = L->unit_ptr[t], n = L->unit_ptr[t + 1] - u0;
    CHECK(s.per_group >= 1 && s.per_group * G <= HPD_F32_ROWS);
    CHECK(s.waves >= 1 && s.waves <= hpd_f32_max_waves(L->cfg.head_dim));
    auto groups = [&](int32_t u) { return (L->unit_desc[(size_t)(u0 + u) * 8 + 5] + s.per_group - 1) / s.per_group; };
    int64_t exist = 0;
    for (int32_t u = 0; u < n; ++u) exist += groups(u);
    if (s.rg || n == 0) {
      for (int32_t u = 0; u < n; ++u) CHECK(groups(u) <= s.rg);
      CHECK(s.groups == (int64_t)n * s.rg);
      continue;
    }
    listed = true;
    CHECK(s.groups == exist && s.list * 2 + (size_t)exist * 2 <= L->f32_groups.size());
    const int32_t* pair = L->f32_groups.data() + s.list * 2;
    for (int32_t u = 0; u < n; ++u)
      for (int32_t g = 0; g < groups(u); ++g, pair += 2) CHECK(pair[0] == u && pair[1] == g);
  }
  return listed;
}

// waves of a workgroup in the last step of an fp32 batch
static int32_t f32_waves(int32_t hq, int32_t hkv, int32_t D, int32_t T, int32_t docs, int32_t doc, int32_t branches) {
  hpd_config cfg{};
  cfg.n_q_heads = hq; cfg.n_kv_heads = hkv; cfg.head_dim = D; cfg.dtype = HPD_F32; cfg.rope_base = 10000.0; cfg.max_new = T;
  cfg.flags = HPD_FLAG_HOST_ONLY;
  const int32_t header = 0;
  std::vector<int32_t> doc_ptr{0, docs}, doc_len(docs, doc), branch_ptr{0};
  for (int32_t d = 0; d < docs; ++d) branch_ptr.push_back(branch_ptr.back() + branches);
  hpd_layout* L = nullptr;
  CHECK(hpd_build_layout(&cfg, 1, &header, doc_ptr.data(), doc_len.data(), branch_ptr.data(), nullptr, nullptr, nullptr, &L) == HPD_OK);
  const int32_t waves = L->f32_steps[T - 1].waves;
  hpd_layout_free(L);
  return waves;
}

// the steps of an even bf16 batch that run the kernel for many rows per unit: all of them, some, none
enum { NONE = 0, SOME = 1, ALL = 2 };
// attn_prefill_kernel's list: every row group of every segment once, with its segment's words.  With more than two row groups per CU
// those of a segment are dealt to one XCD for every kv head (workgroup b: record b / Hkv, kv head b % Hkv, XCD b % 8); otherwise no
// record is without tokens, so that every XCD has the same number of row groups, or one more.
static void check_prefill_groups(const hpd_layout* L) {
  const int32_t Hkv = L->cfg.n_kv_heads, Gr = L->cfg.n_q_heads / Hkv;
  if (L->cfg.dtype != HPD_BF16 || L->cfg.head_dim != 128 || Gr > 8) {
    CHECK(L->fgroup_desc.empty());
    return;
  }
  const int32_t per = 128 / (Gr <= 2 ? Gr : Gr <= 4 ? 4 : 8);
  const size_t n_units = L->funit_desc.size() / 8;
  std::vector<std::vector<int>> seen(n_units), xcd(n_units, std::vector<int>(Hkv, -1));
  int64_t n = 0;
  const bool few = L->prefill_groups <= 2 * (int64_t)L->n_cus;
  for (size_t u = 0; u < n_units; ++u) seen[u].assign((L->funit_desc[u * 8 + 5] + per - 1) / per, 0);
  for (size_t r = 0; r < L->fgroup_desc.size() / 8; ++r) {
    const int32_t* d = L->fgroup_desc.data() + r * 8;
    if (d[5] == 0) {
      CHECK(!few);
      continue;
    }
    size_t u = 0;  // (a segment is told by its first pool slot and its kind)
    while (u < n_units && !std::equal(d, d + 7, L->funit_desc.data() + u * 8)) ++u;
    CHECK(u < n_units && d[7] % per == 0 && d[7] >= 0 && d[7] < d[5]);
    ++seen[u][d[7] / per];
    for (int32_t hk = 0; hk < Hkv; ++hk, ++n) {
      int& x = xcd[u][hk];
      const int now = (int)((r * Hkv + hk) % 8);
      CHECK(few || x < 0 || x == now);
      x = now;
    }
  }
  for (auto& s : seen)
    for (int c : s) CHECK(c == 1);
  CHECK(n == L->prefill_groups);
  // the order of each lane, and that the lanes are as even as their units allow
  const size_t lanes = few ? 1 : 8 / std::gcd(8, Hkv), row = (size_t)L->n_cus / lanes / Hkv;
  auto blocks = [&](const int32_t* d, int32_t tok) {
    return (L->cfg.mask_mode == HPD_MASK_PAPER ? d[1] : (d[1] + 31) / 32) + (std::min(tok + per, d[5]) + 31) / 32;
  };
  int64_t heaviest = 0, least = std::numeric_limits<int64_t>::max(), greatest = 0;
  for (size_t u = 0; u < n_units; ++u) {
    int64_t load = 0;
    for (int32_t t = 0; t < L->funit_desc[u * 8 + 5]; t += per) load += blocks(L->funit_desc.data() + u * 8, t) + 6;
    heaviest = std::max(heaviest, load);
  }
  for (size_t i = 0; i < lanes; ++i) {
    std::vector<const int32_t*> of;
    for (size_t r = i; r < L->fgroup_desc.size() / 8; r += lanes)
      if (L->fgroup_desc[r * 8 + 5]) of.push_back(L->fgroup_desc.data() + r * 8);
    std::vector<int32_t> b;
    int64_t load = 0;
    for (const int32_t* d : of) {
      b.push_back(blocks(d, d[7]));
      load += b.back() + 6;
    }
    least = std::min(least, load);
    greatest = std::max(greatest, load);
    if (L->prefill_groups > 16 * (int64_t)L->n_cus) {  // unit after unit, each from its last row group to its first
      for (size_t k = 1; k < of.size(); ++k)
        CHECK(std::equal(of[k], of[k] + 7, of[k - 1]) ? of[k][7] == of[k - 1][7] - per
                                                      : of[k - 1][7] == 0 && of[k][7] + per >= of[k][5]);
      continue;
    }
    std::vector<int32_t> want = b;
    std::sort(want.begin(), want.end(), std::greater<int32_t>());
    if (of.size() > row && of.size() <= 2 * row) {  // the first that shares its CU is the longest of them, with the shortest of all
      const std::vector<int32_t> longest = want;
      for (size_t k = 0; k < of.size(); ++k)
        want[k] = k < row ? longest[(2 * row - of.size() + k) % row] : longest[of.size() - 1 - (k - row)];
    }
    CHECK(b == want);
  }
  CHECK(n_units == 0 || greatest - least <= heaviest);
}

static int dense_steps(int32_t hq, int32_t hkv, int32_t D, int32_t T, int32_t P, int32_t header, int32_t J, std::vector<int32_t> doc,
                       std::vector<int32_t> branches, bool paper) {
  hpd_config cfg{};
  cfg.n_q_heads = hq; cfg.n_kv_heads = hkv; cfg.head_dim = D; cfg.dtype = HPD_BF16; cfg.rope_base = 10000.0; cfg.max_new = T;
  cfg.flags = HPD_FLAG_HOST_ONLY;
  cfg.pos_mode = paper ? HPD_POS_PAPER_GAP : HPD_POS_CONTIG;
  cfg.mask_mode = paper ? HPD_MASK_PAPER : HPD_MASK_BLOCK;
  std::vector<int32_t> headers(P, header), doc_ptr{0}, doc_len, branch_ptr{0};
  for (int32_t p = 0; p < P; ++p) {
    for (int32_t j = 0; j < J; ++j) {
      doc_len.push_back(doc[doc_len.size() % doc.size()]);
      branch_ptr.push_back(branch_ptr.back() + branches[(branch_ptr.size() - 1) % branches.size()]);
    }
    doc_ptr.push_back((int32_t)doc_len.size());
  }
  const std::vector<int32_t> attr(branch_ptr.back(), 1);
  hpd_layout* L = nullptr;
  CHECK(hpd_build_layout(&cfg, P, headers.data(), doc_ptr.data(), doc_len.data(), branch_ptr.data(), nullptr,
                         paper ? attr.data() : nullptr, nullptr, &L) == HPD_OK);
  CHECK(L->dense_steps.size() == (D == 128 && hq / hkv <= 8 ? (size_t)T : 0));
  int32_t n = 0;
  for (uint8_t s : L->dense_steps) n += s;
  hpd_layout_free(L);
  return n == 0 ? NONE : n == T ? ALL : SOME;
}

// workgroups per CU at a time in the steps of a bf16 batch, 0 where the streaming kernel runs; branch b ends after blen(b) steps
// and has attr(b) name tokens (literal mask)
static std::vector<int> workgroups_per_cu(int32_t hq, int32_t hkv, int32_t T, const std::vector<int32_t>& header, int32_t docs,
                                          const std::vector<int32_t>& doc, const std::vector<int32_t>& branches, bool paper,
                                          const std::function<int32_t(int32_t)>& blen, const std::function<int32_t(int32_t)>& attr) {
  hpd_config cfg{};
  cfg.n_q_heads = hq; cfg.n_kv_heads = hkv; cfg.head_dim = 128; cfg.dtype = HPD_BF16; cfg.rope_base = 500000.0; cfg.max_new = T;
  cfg.flags = HPD_FLAG_HOST_ONLY;
  cfg.pos_mode = paper ? HPD_POS_PAPER_GAP : HPD_POS_CONTIG;
  cfg.mask_mode = paper ? HPD_MASK_PAPER : HPD_MASK_BLOCK;
  std::vector<int32_t> doc_ptr{0}, branch_ptr{0}, lens, names;
  for (size_t p = 0; p < header.size(); ++p) doc_ptr.push_back(doc_ptr.back() + docs);
  for (int32_t n : branches) branch_ptr.push_back(branch_ptr.back() + n);
  for (int32_t b = 0; b < branch_ptr.back(); ++b) {
    lens.push_back(blen(b));
    names.push_back(attr(b));
  }
  hpd_layout* L = nullptr;
  CHECK(hpd_build_layout(&cfg, (int32_t)header.size(), header.data(), doc_ptr.data(), doc.data(), branch_ptr.data(), lens.data(),
                         paper ? names.data() : nullptr, nullptr, &L) == HPD_OK);
  CHECK(L->n_cus == 256);
  std::vector<int> per_cu;
  for (int32_t t = 0; t < T; ++t) per_cu.push_back(L->dense_steps[t] ? hpd_plan_dense_launch(L, t).per_cu : 0);
  hpd_layout_free(L);
  return per_cu;
}

// the batches of the GPU tests that are there for one of the two shapes of the kernel for many rows per unit: what they run
static void many_rows_of_the_gpu_tests() {
  auto steps_of = [](const std::vector<int>& v, int per_cu) { return std::count(v.begin(), v.end(), per_cu); };
  // test_decode_of_many_rows_per_unit_by_workgroups_per_cu
  const struct { int g, tenths; } shapes[] = {{1, 15}, {2, 25}, {8, 25}, {3, 25}, {8, 50}, {1, 50}, {2, 50}};
  for (const auto& x : shapes)
    for (bool literal : {false, true}) {
      const int pad = x.g <= 2 ? x.g : x.g <= 4 ? 4 : 8, n = 256 / pad, prompts = x.tenths * 256 / 160, per = literal ? 1 : 2;
      const int heads[] = {0, 33, 64, 7, 95}, docs[] = {1, 31, 64, 33, 97, 32};
      std::vector<int32_t> header, doc, branches;
      for (int p = 0; p < (literal ? prompts : prompts / 2); ++p) header.push_back(heads[p % 5]);
      for (int d = 0; d < (int)header.size() * per; ++d) {
        doc.push_back(docs[d % 6]);
        branches.push_back(n - d % 3 % 2);
      }
      const auto v = workgroups_per_cu(x.g * 8, 8, 21, header, per, doc, branches, literal,
                                       [](int32_t b) { return b % 11 == 7 ? 18 : b % 9 == 5 ? 14 : 21; },
                                       [](int32_t b) { return 1 + b % 4; });
      const int want = x.tenths < 20 ? 2 : 3;
      CHECK(steps_of(v, want) >= 7 && steps_of(v, 5 - want) == 0);
      if (x.g > 1) CHECK(steps_of(v, want) >= 15);
    }
  // test_non_finite_values_of_a_branch_in_decode_with_many_rows, test_literal_decode_of_many_rows_and_few_shared_blocks
  for (int prompts : {24, 48}) {
    const int want = prompts == 24 ? 2 : 3;
    const std::vector<int32_t> doc40(prompts, 40), doc20(prompts, 20);
    for (bool literal : {false, true})
      CHECK(steps_of(workgroups_per_cu(64, 8, 12, std::vector<int32_t>(prompts, 7), 1, doc40, std::vector<int32_t>(prompts, 32), literal,
                                       [](int32_t) { return 12; }, [](int32_t) { return 1; }), want) == 12);
    const struct { int hq, header, n; } few[] = {{64, 0, 32}, {64, 7, 32}, {32, 0, 64}, {16, 0, 128}};
    for (const auto& x : few)
      CHECK(steps_of(workgroups_per_cu(x.hq, 8, 26, std::vector<int32_t>(prompts, x.header), 1, doc20, std::vector<int32_t>(prompts, x.n),
                                       true, [](int32_t b) { return b % 11 == 4 ? 13 : 26; }, [](int32_t) { return 1; }), want) == 26);
  }
}

// random batches of the bf16 kernels' shape, from fewer row groups than CUs to more than 16 per CU
static void prefill_lists() {
  std::mt19937 rng(30);
  auto uni = [&](int lo, int hi) { return std::uniform_int_distribution<int>(lo, hi)(rng); };
  int64_t fewest = 1 << 30, most = 0;
  for (int iter = 0; iter < 60; ++iter) {
    hpd_config cfg{};
    const int hkvs[] = {1, 2, 3, 4, 6, 8, 12, 16};
    cfg.n_kv_heads = hkvs[iter % 8]; cfg.n_q_heads = cfg.n_kv_heads * uni(1, 8);
    cfg.head_dim = 128; cfg.dtype = HPD_BF16; cfg.rope_base = 500000.0; cfg.max_new = 2; cfg.flags = HPD_FLAG_HOST_ONLY;
    const bool paper = iter % 3 == 0;
    cfg.pos_mode = paper ? HPD_POS_PAPER_GAP : HPD_POS_CONTIG;
    cfg.mask_mode = paper ? HPD_MASK_PAPER : HPD_MASK_BLOCK;
    const int P = 1 << uni(0, 6), longest = 1 << uni(0, 11);
    std::vector<int32_t> header, doc_ptr{0}, doc_len, branch_ptr{0}, attr;
    doc_len.reserve(1);  // (so that its address is one without documents)
    for (int p = 0; p < P; ++p) {
      header.push_back(uni(0, 3) ? uni(1, 200) : 0);
      for (int j = uni(0, 3); j > 0; --j) {
        doc_len.push_back(uni(1, longest));
        branch_ptr.push_back(branch_ptr.back() + uni(0, 3));
      }
      doc_ptr.push_back((int32_t)doc_len.size());
    }
    for (int32_t b = 0; b < branch_ptr.back(); ++b) attr.push_back(uni(1, 40));
    attr.push_back(1);  // (so that its address is one where no branch is)
    hpd_layout* L = nullptr;
    CHECK(hpd_build_layout(&cfg, P, header.data(), doc_ptr.data(), doc_len.data(), branch_ptr.data(), nullptr,
                           paper ? attr.data() : nullptr, nullptr, &L) == HPD_OK);
    check_prefill_groups(L);
    fewest = std::min(fewest, L->prefill_groups);
    most = std::max(most, L->prefill_groups);
    hpd_layout_free(L);
  }
  CHECK(fewest < 256 && most > 16 * 256);
}

int main() {
  std::mt19937 rng(26209);
  auto uni = [&](int lo, int hi) { return std::uniform_int_distribution<int>(lo, hi)(rng); };
  int built = 0, refused = 0;
  for (int iter = 0; iter < 400; ++iter) {
    hpd_config cfg{};
    const int hkv = 1 << uni(0, 3);
    cfg.n_kv_heads = hkv; cfg.n_q_heads = hkv * uni(1, 8);
    cfg.head_dim = 8 * uni(1, 32); cfg.dtype = uni(0, 1); cfg.rope_base = iter % 2 ? 10000.0 : 500000.0;
    cfg.max_new = uni(1, 12); cfg.flags = HPD_FLAG_HOST_ONLY; cfg.out_dtype = uni(0, 1);
    const bool paper = iter % 3 == 0, gap = paper || iter % 5 == 0;
    cfg.pos_mode = gap ? HPD_POS_PAPER_GAP : HPD_POS_CONTIG;
    cfg.mask_mode = paper ? HPD_MASK_PAPER : HPD_MASK_BLOCK;
    const int P = uni(1, 6);
    std::vector<int32_t> header(P), doc_ptr(P + 1, 0), doc_len, branch_ptr{0}, branch_len, attr_len;
    for (int p = 0; p < P; ++p) {
      header[p] = uni(0, 70);
      const int J = uni(0, 4);  // a prompt without documents is allowed
      doc_ptr[p + 1] = doc_ptr[p] + J;
      for (int j = 0; j < J; ++j) {
        doc_len.push_back(uni(1, 200));
        const int N = uni(0, 9);
        branch_ptr.push_back(branch_ptr.back() + N);
        for (int n = 0; n < N; ++n) { branch_len.push_back(uni(1, cfg.max_new)); attr_len.push_back(uni(1, 5)); }
      }
    }
    // every fourth batch is broken in one place and has to be refused
    const int breakage = iter % 4 == 3 ? uni(0, 6) : -1;
    if (breakage == 0 && !branch_len.empty()) branch_len[uni(0, (int)branch_len.size() - 1)] = cfg.max_new + 1;
    if (breakage == 1 && !doc_len.empty()) doc_len[uni(0, (int)doc_len.size() - 1)] = 0;
    if (breakage == 2) header[uni(0, P - 1)] = -1;
    if (breakage == 3) doc_ptr[0] = 1;
    if (breakage == 4) cfg.head_dim += 1;
    if (breakage == 5) { cfg.n_kv_heads = 3; cfg.n_q_heads = 4; }
    if (breakage == 6 && !attr_len.empty() && gap) attr_len[0] = 0;
    static int32_t none = 0;
    hpd_layout* L = nullptr;
    const int rc = hpd_build_layout(&cfg, P, header.data(), doc_ptr.data(), doc_len.empty() ? &none : doc_len.data(),
                                    branch_ptr.data(), branch_len.empty() ? &none : branch_len.data(),
                                    gap ? (attr_len.empty() ? &none : attr_len.data()) : nullptr, nullptr, &L);
    if (rc != HPD_OK) {
      CHECK(L == nullptr);
      CHECK(hpd_status_string(rc) != nullptr);
      ++refused;
      continue;
    }
    ++built;
    const auto c = query<int64_t>(L, HPD_Q_COUNTS, HPD_N_COUNTS);
    CHECK(c[HPD_C_N_PROMPTS] == P && c[HPD_C_N_DOCS] == (int64_t)doc_len.size());
    const size_t B = (size_t)c[HPD_C_N_BRANCHES], T = (size_t)cfg.max_new;
    const size_t n_seg = (size_t)P + doc_len.size() + (paper ? P : 0);
    check_f32_steps(L);
    check_prefill_groups(L);
    query<int64_t>(L, HPD_Q_POOL_BYTES, 4);
    const auto n_live = query<int32_t>(L, HPD_Q_N_LIVE, T);
    int64_t total = 0;
    for (int32_t x : n_live) total += x;
    CHECK(total == c[HPD_C_TOTAL_LIVE]);
    const auto live = query<int32_t>(L, HPD_Q_LIVE_BRANCH, (size_t)total);
    for (int32_t b : live) CHECK(b >= 0 && (size_t)b < B);
    const auto base = query<int32_t>(L, HPD_Q_BRANCH_BASE_POS, B);
    for (size_t b = 0; b < B; ++b) CHECK(base[b] + (int64_t)T <= c[HPD_C_MAX_POS]);
    query<int32_t>(L, HPD_Q_BRANCH_DOC, B);
    const auto seg_off = query<int32_t>(L, HPD_Q_SEG_OFF, n_seg);
    const auto seg_len = query<int32_t>(L, HPD_Q_SEG_LEN, n_seg);
    for (size_t s = 0; s < n_seg; ++s) CHECK(seg_off[s] % HPD_KEY_BLOCK == 0 && seg_off[s] + seg_len[s] <= c[HPD_C_N_PREFIX_SLOTS]);
    query<int32_t>(L, HPD_Q_SEG_POS0, n_seg);
    query<int32_t>(L, HPD_Q_SEG_RAW_OFF, n_seg);
    query<int32_t>(L, HPD_Q_N_UNITS, T);
    CHECK(hpd_layout_query(L, 99, (void*)&none, 4) == HPD_E_INVALID);
    // a host-only layout refuses every device call before anything is launched
    CHECK(hpd_rope_positions(L, 0, &none, nullptr, nullptr) == HPD_E_INVALID);
    CHECK(hpd_kv_append(L, 0, &none, &none, &none, &none, nullptr, nullptr) == HPD_E_INVALID);
    CHECK(hpd_decode_attention(L, 0, &none, &none, &none, &none, &none, &none, nullptr) == HPD_E_INVALID);
    CHECK(hpd_decode_step(L, 0, &none, &none, &none, &none, &none, &none, &none, &none, nullptr) == HPD_E_INVALID);
    CHECK(hpd_prefix_fill(L, &none, &none, &none, &none, nullptr) == HPD_E_INVALID);
    CHECK(hpd_prefill_attention(L, &none, &none, &none, &none, nullptr) == HPD_E_INVALID);
    CHECK(hpd_dynamic_begin(L, nullptr) == HPD_E_INVALID);
    CHECK(hpd_dynamic_begin_static(L, nullptr) == HPD_E_INVALID);
    CHECK(hpd_set_tail_pages(L, 8, 4, &none) == HPD_E_INVALID);
    int32_t s_out = 0;
    CHECK(hpd_expand_mask(L, 0, -1, nullptr, &s_out, nullptr) == HPD_E_INVALID);
    CHECK(hpd_set_kernel_mode(L, 7) == HPD_E_INVALID);
    hpd_layout_free(L);
  }
  // fp32 steps of batches with a few documents of many branches, whose row groups are listed: branches that end at
  // different steps, documents that lose all of theirs
  int with_list = 0;
  for (int iter = 0; iter < 60; ++iter) {
    hpd_config cfg{};
    const int G = uni(1, 17);
    cfg.n_kv_heads = uni(1, 3); cfg.n_q_heads = cfg.n_kv_heads * G;
    cfg.head_dim = 32 << uni(0, 2); cfg.dtype = HPD_F32; cfg.rope_base = 10000.0; cfg.max_new = uni(1, 9);
    cfg.flags = HPD_FLAG_HOST_ONLY;
    const int n_docs = uni(1, 40);
    std::vector<int32_t> doc_ptr{0, n_docs}, doc_len, branch_ptr{0}, branch_len;
    for (int d = 0; d < n_docs; ++d) {
      doc_len.push_back(uni(1, iter % 7 == 0 ? 900 : 40));
      branch_ptr.push_back(branch_ptr.back() + (uni(0, 9) ? uni(0, 2) : uni(30, 200)));
      while ((int)branch_len.size() < branch_ptr.back()) branch_len.push_back(uni(1, cfg.max_new));
    }
    const int32_t header = uni(0, 40), none = 1;
    hpd_layout* L = nullptr;
    CHECK(hpd_build_layout(&cfg, 1, &header, doc_ptr.data(), doc_len.data(), branch_ptr.data(),
                           branch_len.empty() ? &none : branch_len.data(), nullptr, nullptr, &L) == HPD_OK);
    CHECK(L->f32_steps.size() == (G <= HPD_F32_ROWS ? (size_t)cfg.max_new : 0));
    with_list += check_f32_steps(L);
    hpd_layout_free(L);
  }
  CHECK(with_list >= 10);
  prefill_lists();
  many_rows_of_the_gpu_tests();
  // short workgroups: four waves where all of them are at work at once, two where they queue up; a wave per tile and one
  // for the newest tokens where there are few workgroups
  CHECK(f32_waves(8, 2, 32, 1, 500, 5, 4) == 4);
  CHECK(f32_waves(10, 2, 32, 1, 2000, 5, 3) == 1);
  CHECK(f32_waves(8, 2, 128, 1, 340, 5, 4) == 2);
  CHECK(f32_waves(10, 2, 64, 4, 3739, 54, 1) == 2);
  CHECK(f32_waves(16, 4, 64, 10, 8, 64, 4) == 8);
  // the plan of the kernel for many rows per unit: even batches with full workgroups run it, few rows per unit and launches
  // of mostly narrow units do not, nor does a layout that the streaming kernels do not serve
  CHECK(dense_steps(64, 8, 128, 32, 16, 128, 2, {2048}, {48}, false) == ALL);
  CHECK(dense_steps(64, 8, 128, 32, 16, 128, 2, {2048}, {40}, false) == ALL);
  CHECK(dense_steps(64, 8, 128, 32, 16, 128, 2, {2048}, {12}, false) == NONE);
  CHECK(dense_steps(32, 8, 128, 16, 32, 64, 1, {512}, {16}, false) == NONE);
  CHECK(dense_steps(48, 8, 128, 4, 26, 1278, 4, {1, 5, 9}, {64, 1, 3, 5, 7}, false) == NONE);
  CHECK(dense_steps(32, 8, 128, 4, 64, 859, 5, {20, 60, 110}, {113, 2, 5, 8, 14}, false) == NONE);
  CHECK(dense_steps(32, 8, 128, 12, 64, 64, 4, {384}, {24}, true) == ALL);
  CHECK(dense_steps(32, 8, 128, 24, 64, 0, 1, {20}, {64}, true) == ALL);
  CHECK(dense_steps(32, 8, 128, 12, 64, 64, 1, {384}, {4}, true) == NONE);
  CHECK(dense_steps(32, 4, 128, 64, 1, 0, 1, {20}, {16}, true) == NONE);
  CHECK(dense_steps(64, 8, 64, 4, 16, 128, 2, {2048}, {48}, false) == NONE);
  CHECK(dense_steps(72, 8, 128, 4, 16, 128, 2, {2048}, {48}, false) == NONE);
  // fine-tuning mask: sizes and argument checks (outputs NULL: nothing is launched)
  for (int iter = 0; iter < 200; ++iter) {
    const int n = uni(0, 12), k_max = uni(1, 9);
    std::vector<int32_t> a(n), v(n);
    int64_t want = uni(0, 50);
    const int32_t plen = (int32_t)want;
    for (int i = 0; i < n; ++i) { a[i] = uni(1, 6); v[i] = uni(0, k_max); want += a[i] + v[i]; }
    int64_t S = -1;
    CHECK(hpd_finetune_mask(plen, n, a.data(), v.data(), k_max, nullptr, nullptr, &S, nullptr) == HPD_OK && S == want);
    if (n > 0) {
      v[uni(0, n - 1)] = k_max + 1;
      CHECK(hpd_finetune_mask(plen, n, a.data(), v.data(), k_max, nullptr, nullptr, &S, nullptr) == HPD_E_INVALID);
    }
  }
  hpd_layout_free(nullptr);
  CHECK(g_stub_calls == 0);
  std::printf("host sanitizer run: %d layouts built, %d refused, no finding\n", built, refused);
  return 0;
}
