// Extend (re-prefill) attention: host planner and entry point.
//
// A re-prefill recomputes a resumed trajectory's KV cache (Sec. 2.3, partial
// rollout and migration). Its cost per new token grows with the token's
// position, so a sequence's new tokens are cut into blocks of
// floor(384 / g) tokens, one work item per (sequence, KV head, block), and
// the items are launched longest first: the GPU starts the longest key walks
// early and fills the tail with the short ones. The rule is stated in
// sf_decode_attn.h next to sf_extend_attn_plan.
#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <new>
#include <vector>

#include "sf_internal.h"

static_assert(sizeof(sf_extend_info) == 32, "sf_extend_info layout is part of the ABI");

using namespace sf;

namespace {

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
bool aligned4(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 3u) == 0; }

struct Item {
  int32_t seq, kvh, t0, nt, prefix, qrow0, steps;
};

// Checks the lengths and counts the query rows.
sf_status check_lengths(const sf_attn_desc* desc, const int32_t* seq_lens_host, const int32_t* q_lens_host,
                        int64_t* rows) {
  sf_status st = validate_desc(desc);
  if (st != SF_OK) return st;
  if (desc->num_seqs > 0 && (!seq_lens_host || !q_lens_host)) return SF_ERR_INVALID_ARG;
  *rows = 0;
  for (int32_t s = 0; s < desc->num_seqs; ++s) {
    const int32_t L = seq_lens_host[s], e = q_lens_host[s];
    if (e < 0 || L < e || int64_t(L) > int64_t(kPage) * desc->block_table_stride) return SF_ERR_INVALID_ARG;
    if (L > 0 && desc->num_pages == 0) return SF_ERR_INVALID_ARG;
    *rows += e;
  }
  if (*rows > INT32_MAX / (int64_t(desc->num_q_heads) * desc->head_dim)) return SF_ERR_INVALID_ARG;
  return SF_OK;
}

void fill_info(const sf_attn_desc* desc, int64_t items, int64_t rows, sf_extend_info* info) {
  info->num_items = int32_t(items);
  info->tokens_per_item = kExtendRows / (desc->num_q_heads / desc->num_kv_heads);
  info->num_q_rows = int32_t(rows);
  info->reserved = 0;
  info->work_bytes = uint64_t(items) * kItemInts * 4;
  info->desc_key = desc_key(desc);
}

}  // namespace

extern "C" sf_status sf_extend_attn_plan(const sf_attn_desc* desc, const int32_t* seq_lens_host,
                                         const int32_t* q_lens_host, int32_t* work_host,
                                         uint64_t work_capacity_bytes, sf_extend_info* info) {
  int64_t rows = 0;
  sf_status st = validate_desc(desc);
  if (st != SF_OK) return st;
  if (!info) return SF_ERR_INVALID_ARG;
  if ((st = check_lengths(desc, seq_lens_host, q_lens_host, &rows)) != SF_OK) return st;
  const int32_t per_item = kExtendRows / (desc->num_q_heads / desc->num_kv_heads);

  std::vector<Item> items;
  int32_t qrow0 = 0;
  for (int32_t s = 0; s < desc->num_seqs; ++s) {
    const int32_t L = seq_lens_host[s], e = q_lens_host[s];
    for (int32_t kvh = 0; kvh < desc->num_kv_heads; ++kvh)
      for (int32_t t0 = 0; t0 < e; t0 += per_item) {
        const int32_t nt = std::min(per_item, e - t0);
        const int32_t prefix = L - e;
        items.push_back({s, kvh, t0, nt, prefix, qrow0, (prefix + t0 + nt + 2 * kPage - 1) / (2 * kPage)});
      }
    qrow0 += e;
  }
  // Longest key walk first; ties keep (sequence, KV head, block) order.
  std::stable_sort(items.begin(), items.end(), [](const Item& x, const Item& y) { return x.steps > y.steps; });

  fill_info(desc, int64_t(items.size()), rows, info);
  if (!work_host) return SF_OK;
  if (work_capacity_bytes < info->work_bytes) return SF_ERR_CAPACITY;
  for (size_t i = 0; i < items.size(); ++i) {
    const Item& it = items[i];
    int32_t* r = work_host + i * kItemInts;
    r[0] = it.seq;
    r[1] = it.kvh;
    r[2] = it.t0;
    r[3] = it.nt;
    r[4] = it.prefix;
    r[5] = it.qrow0;
    r[6] = it.steps;
    r[7] = 0;
  }
  return SF_OK;
}

namespace {

constexpr int32_t kStepKeys = 2 * kPage;

// Lengths go up to INT32_MAX, so rounding one up takes 64 bits.
int32_t steps_of(int32_t keys) { return int32_t((int64_t(keys) + kStepKeys - 1) / kStepKeys); }
int32_t pages_of(int32_t tokens) { return int32_t((int64_t(tokens) + kPage - 1) / kPage); }

// Calls f(sequence, first new token, tokens, steps) for every block of at
// most `per` new tokens (each is one item per KV head).
template <class F>
void for_blocks(const sf_attn_desc* desc, const int32_t* lens, const int32_t* new_lens, int32_t per, F f) {
  for (int32_t s = 0; s < desc->num_seqs; ++s)
    for (int32_t t0 = 0; t0 < new_lens[s]; t0 += per) {
      const int32_t nt = std::min(per, new_lens[s] - t0);
      f(s, t0, nt, steps_of(lens[s] - new_lens[s] + t0 + nt));
    }
}

// How sf_runner_extend cuts its work: rows per item, and the longest part of a
// key walk (steps).
struct Split {
  int32_t rows;
  int32_t most;
};

// The cut is chosen by estimated time. A workgroup takes kStart + kStep *
// steps (us at D = 128; half the step at D = 64), measured with one 384-row
// item per CU (12 waves) and one or two 128-row items per CU (4 waves each):
// one 16384-token walk cut into 1, 2, 4 .. 32 parts took 582, 295, 154, 84, 50,
// 35 us with 384 rows and 486, 250, 128, 69, 39, 32 us with 128. kStart holds
// the launch, the first loads and the result's store. Cut walks add the merge
// launch: kMerge plus the partial rows' bytes. Uncut 384-row items are best
// whenever they fill the chip several times over; short grids gain from parts
// that fill it once (or 2 .. 4 times): 4 sequences with 256 new tokens after
// 8000 cached ones, 28/4 heads, 305 us whole, 130 + 11 us in parts of 88 steps,
// 156 + 21 in parts of 32; one prompt of 1000 tokens 48 us whole, 38 us as
// whole 128-row items, 26 + 5 us as 128-row items in parts of at most 16 steps.
struct Cost {
  double start, step;
};
constexpr Cost kLarge = {14.0, 1.12}, kSmallAlone = {10.0, 0.94}, kSmallPaired = {16.0, 1.0};
constexpr double kMerge = 4.0, kMergeBytesPerUs = 4.4e6;
constexpr int32_t kSmallestPart = 4;   // steps
constexpr int32_t kRounds = 4;

struct Totals {
  int64_t parts = 0, steps = 0, cut_rows = 0;
  int32_t longest = 0, shortest = INT32_MAX;
};

Split choose_split(const sf_attn_desc* desc, const int32_t* lens, const int32_t* new_lens, int32_t num_cus) {
  const int32_t g = desc->num_q_heads / desc->num_kv_heads;
  const int64_t hkv = desc->num_kv_heads;
  const double step_scale = desc->head_dim / 128.0;
  // The blocks by length: (steps, blocks, rows), made once per item size; the
  // search below asks for the totals of many cuts.
  struct Walk {
    int32_t steps, blocks;
    int64_t rows;
  };
  thread_local std::vector<Walk> walks;
  auto measure = [&](int32_t rows) {
    walks.clear();
    for_blocks(desc, lens, new_lens, rows / g, [&](int32_t, int32_t, int32_t nt, int32_t steps) {
      if (walks.empty() || walks.back().steps != steps) walks.push_back({steps, 0, 0});
      ++walks.back().blocks;
      walks.back().rows += int64_t(nt) * g;
    });
    std::sort(walks.begin(), walks.end(), [](const Walk& x, const Walk& y) { return x.steps < y.steps; });
    size_t n = 0;
    for (const Walk& w : walks) {
      if (n > 0 && walks[n - 1].steps == w.steps) {
        walks[n - 1].blocks += w.blocks;
        walks[n - 1].rows += w.rows;
      } else {
        walks[n++] = w;
      }
    }
    walks.resize(n);
  };
  auto totals = [&](int32_t most) {
    Totals t;
    const float inv = 1.f / float(most);   // an estimate: the plan itself counts exactly
    for (const Walk& w : walks) {
      const int32_t k = w.steps <= most ? 1 : int32_t(float(w.steps - 1) * inv) + 1;
      const int32_t len = k == 1 ? w.steps : int32_t(float(w.steps) / float(k));
      t.parts += int64_t(k) * w.blocks;
      t.steps += int64_t(w.steps) * w.blocks;
      if (k > 1) t.cut_rows += k * w.rows;
      t.longest = std::max(t.longest, k == 1 ? w.steps : len + 1);
      t.shortest = std::min(t.shortest, len);
    }
    t.parts *= hkv;
    t.steps *= hkv;
    t.cut_rows *= hkv;
    return t;
  };
  // Estimated time of a plan on `slots` concurrent workgroups: no less than
  // its longest part, and its average load plus what a partial last round of
  // the shortest parts leaves idle.
  auto estimate = [&](const Totals& t, bool small) {
    // 128-row items: one per CU, two per CU, or in between
    const double pair = std::min(1.0, std::max(0.0, double(t.parts) / num_cus - 1.0));
    const Cost c = small ? Cost{kSmallAlone.start + pair * (kSmallPaired.start - kSmallAlone.start),
                                kSmallAlone.step + pair * (kSmallPaired.step - kSmallAlone.step)}
                         : kLarge;
    const int64_t slots = small ? 2 * num_cus : num_cus;
    const double step = c.step * step_scale;
    const int64_t rest = t.parts % slots;
    const double idle = rest ? 1.0 - double(rest) / double(slots) : 0.0;
    const double load = (double(t.parts) * c.start + step * double(t.steps)) / double(slots);
    return std::max(c.start + step * t.longest, load + idle * (c.start + step * t.shortest)) +
           (t.cut_rows ? kMerge + double(t.cut_rows) * desc->head_dim * 4 / kMergeBytesPerUs : 0.0);
  };

  Split best = {kExtendRows, INT32_MAX};
  int64_t items = 0;
  for (int32_t s = 0; s < desc->num_seqs; ++s) items += (new_lens[s] + kExtendRows / g - 1) / (kExtendRows / g) * hkv;
  if (items == 0 || items > int64_t(kRounds) * 2 * num_cus) return best;
  measure(kExtendRows);
  const Totals whole = totals(INT32_MAX);
  double best_us = estimate(whole, false);
  auto consider = [&](int32_t rows, const Totals& uncut) {
    const bool small = rows == kExtendSmallRows;
    const int64_t slots = small ? 2 * num_cus : num_cus;
    auto take = [&](const Totals& t, int32_t most) {
      const double us = estimate(t, small);
      if (us < best_us) best_us = us, best = {rows, most};
    };
    take(uncut, INT32_MAX);
    // no cut beats the average load
    const Cost least = small ? kSmallAlone : kLarge;
    if ((double(uncut.parts) * least.start + least.step * step_scale * double(uncut.steps)) / double(slots) >= best_us) return;
    for (int32_t r = 1; r <= kRounds; ++r) {
      // the shortest parts that number at most r per slot, and somewhat longer ones
      if (uncut.parts >= r * slots) continue;
      int32_t lo = int32_t(std::max<int64_t>(kSmallestPart, uncut.steps / (r * slots))), hi = uncut.longest - 1;
      if (lo > hi) break;   // parts of the least length already fill fewer rounds
      Totals t = totals(hi);
      if (t.parts > r * slots) continue;
      while (lo < hi) {
        const int32_t mid = lo + (hi - lo) / 2;
        const Totals m = totals(mid);
        if (m.parts <= r * slots)
          hi = mid, t = m;
        else
          lo = mid + 1;
      }
      take(t, hi);
      for (const int32_t longer : {hi + hi / 4, hi + hi / 2})
        if (longer < uncut.longest) take(totals(longer), longer);
    }
  };
  consider(kExtendRows, whole);
  if (whole.parts <= 2 * num_cus) {
    measure(kExtendSmallRows);
    consider(kExtendSmallRows, totals(INT32_MAX));
  }
  return best;
}

}  // namespace

sf_status sf::extend_plan_parts(const sf_attn_desc* desc, const int32_t* seq_lens_host, const int32_t* q_lens_host,
                                int32_t num_cus, bool store, int32_t* work, uint64_t capacity, ExtendPlan* plan,
                                sf_extend_info* info) {
  int64_t q_rows = 0;
  sf_status st = check_lengths(desc, seq_lens_host, q_lens_host, &q_rows);
  if (st != SF_OK) return st;
  const int32_t g = desc->num_q_heads / desc->num_kv_heads, hkv = desc->num_kv_heads;
  const int32_t *lens = seq_lens_host, *news = q_lens_host;

  int64_t items = 0;
  for (int32_t s = 0; s < desc->num_seqs; ++s) items += (news[s] + kExtendRows / g - 1) / (kExtendRows / g);
  fill_info(desc, items * hkv, q_rows, info);

  const Split split = choose_split(desc, lens, news, num_cus > 0 ? num_cus : kDefaultNumCus);
  const int32_t rows = split.rows, most = split.most;
  const int32_t per = rows / g;
  auto parts_of = [&](int32_t steps) { return steps <= most ? 1 : (steps - 1) / most + 1; };
  // Calls f(first step, end step) for the k parts of a walk: part i ends at
  // floor((i + 1) steps / k), stepped forward without divisions.
  auto each_cut = [](int32_t steps, int32_t k, auto f) {
    const int32_t q = k > 1 ? steps / k : steps, rem = k > 1 ? steps % k : 0;
    for (int32_t i = 0, b = 0, over = 0; i < k; ++i) {
      int32_t e = b + q;
      if ((over += rem) >= k) {
        over -= k;
        ++e;
      }
      f(b, e);
      b = e;
    }
  };
  int64_t parts = 0, merges = 0, slots = 0, longest = 0;
  for_blocks(desc, lens, news, per, [&](int32_t, int32_t, int32_t, int32_t steps) {
    const int32_t k = parts_of(steps);
    parts += int64_t(k) * hkv;
    if (k > 1) {
      merges += hkv;
      slots += int64_t(k) * hkv;
    }
    longest = std::max<int64_t>(longest, (int64_t(steps) + k - 1) / k);
  });
  int64_t stores = 0, store_pages = 0;
  if (store)
    for (int32_t s = 0; s < desc->num_seqs; ++s)
      if (news[s] > 0) store_pages += pages_of(lens[s]) - (lens[s] - news[s]) / kPage;
  // Runs of 4 pages above 2048 keep the list, and the slots that hold it, a
  // quarter as long; the launch takes the same there (us at runs of 1, 2, 4 and
  // 8, 28/4 heads: 6016 pages 102, 106, 106, 102; 2000 pages 38, 36, 36, 43).
  // Fewer pages want every workgroup: 504 pages 12, 10, 13, 21, 63 pages 7.2,
  // 9.5, 13, 22.
  const int32_t run = store_pages > 2048 ? 4 : 1;
  if (store)
    for (int32_t s = 0; s < desc->num_seqs; ++s)
      if (news[s] > 0) stores += (pages_of(lens[s]) - (lens[s] - news[s]) / kPage + run - 1) / run;
  if (parts + merges + stores > INT32_MAX / kItemInts) return SF_ERR_INVALID_ARG;
  plan->rows = rows;
  plan->num_parts = int32_t(parts);
  plan->num_merge = int32_t(merges);
  plan->num_store = int32_t(stores);
  plan->num_slots = int32_t(slots);
  if (capacity < plan->bytes()) return SF_ERR_CAPACITY;

  // Part rows, longest first (a counting sort by length; ties keep the order
  // block, KV head, part).
  thread_local std::vector<int32_t> at;
  at.assign(size_t(longest) + 2, 0);
  auto each_part = [&](auto f) {
    int32_t s_prev = 0;
    int64_t qrow0 = 0;
    for_blocks(desc, lens, news, per, [&](int32_t s, int32_t t0, int32_t nt, int32_t steps) {
      for (; s_prev < s; ++s_prev) qrow0 += news[s_prev];
      const int32_t k = parts_of(steps);
      for (int32_t h = 0; h < hkv; ++h) f(s, h, lens[s] - news[s] + t0, nt, int32_t(qrow0 + t0), steps, k);
    });
  };
  for_blocks(desc, lens, news, per, [&](int32_t, int32_t, int32_t, int32_t steps) {
    each_cut(steps, parts_of(steps), [&](int32_t b, int32_t e) { at[size_t(longest - (e - b)) + 1] += hkv; });
  });
  for (size_t i = 1; i < at.size(); ++i) at[i] += at[i - 1];
  int32_t slot = 0, merge = 0;
  int32_t* merge_rows = work + parts * kItemInts;
  each_part([&](int32_t s, int32_t h, int32_t first, int32_t nt, int32_t qrow, int32_t steps, int32_t k) {
    if (k > 1) {
      const int32_t m8[kItemInts] = {slot, k, nt, qrow, h, 0, 0, 0};
      std::memcpy(merge_rows + int64_t(merge++) * kItemInts, m8, sizeof m8);
    }
    each_cut(steps, k, [&](int32_t b, int32_t e) {
      const int32_t r8[kItemInts] = {s, h, b, nt, first, qrow, e, k > 1 ? ++slot : 0};
      std::memcpy(work + int64_t(at[size_t(longest - (e - b))]++) * kItemInts, r8, sizeof r8);
    });
  });
  if (store) {
    int32_t* r = merge_rows + merges * kItemInts;
    int32_t qrow0 = 0;
    for (int32_t s = 0; s < desc->num_seqs; qrow0 += news[s++]) {
      const int32_t first = lens[s] - news[s], end_page = pages_of(lens[s]);
      for (int32_t p = first / kPage; news[s] > 0 && p < end_page; p += run, r += kItemInts) {
        const int32_t r8[kItemInts] = {s, p, std::min(run, end_page - p), first, lens[s], qrow0, 0, 0};
        std::memcpy(r, r8, sizeof r8);
      }
    }
  }
  return SF_OK;
}

sf_status sf::extend_args(const sf_attn_desc* desc, const int32_t* work_dev, const void* q, const void* k_new,
                          const void* v_new, void* k_pool, void* v_pool, const int32_t* block_table, float* out,
                          float* lse, ExtendArgs* args) {
  if ((k_new == nullptr) != (v_new == nullptr)) return SF_ERR_INVALID_ARG;
  if (!work_dev || !q || !k_pool || !v_pool || !block_table || !out) return SF_ERR_INVALID_ARG;
  if (!aligned16(work_dev) || !aligned16(q) || !aligned16(k_pool) || !aligned16(v_pool) || !aligned16(out) ||
      !aligned4(block_table) || (lse && !aligned4(lse)) || (k_new && (!aligned16(k_new) || !aligned16(v_new))))
    return SF_ERR_INVALID_ARG;
  ExtendArgs a = {};
  a.items = work_dev;
  a.q = static_cast<const uint16_t*>(q);
  a.k_pool = static_cast<const uint16_t*>(k_pool);
  a.v_pool = static_cast<const uint16_t*>(v_pool);
  a.block_table = block_table;
  a.out = out;
  a.lse = lse;
  a.num_q_heads = desc->num_q_heads;
  a.num_kv_heads = desc->num_kv_heads;
  a.group = desc->num_q_heads / desc->num_kv_heads;
  a.head_dim = desc->head_dim;
  a.bt_stride = desc->block_table_stride;
  // Negating bf16 queries is exact, so a negative scale becomes a positive one.
  a.scale_log2 = float(std::fabs(double(desc->softmax_scale)) * 1.4426950408889634074);
  a.q_sign = desc->softmax_scale < 0.f ? 0x80008000u : 0u;
  a.k_new = static_cast<const uint16_t*>(k_new);
  a.v_new = static_cast<const uint16_t*>(v_new);
  a.k_dst = static_cast<uint16_t*>(k_pool);
  a.v_dst = static_cast<uint16_t*>(v_pool);
  *args = a;
  return SF_OK;
}

extern "C" sf_status sf_extend_attn(const sf_attn_desc* desc, const sf_extend_info* info,
                                    const int32_t* work_host, int32_t* work_dev, const void* q,
                                    const void* k_new, const void* v_new, void* k_pool, void* v_pool,
                                    const int32_t* block_table, float* out, float* lse, void* stream) {
  sf_status st = validate_desc(desc);
  if (st != SF_OK) return st;
  if (!info) return SF_ERR_INVALID_ARG;
  if (info->desc_key != desc_key(desc)) return SF_ERR_PLAN_MISMATCH;
  if (info->num_items < 0 || info->num_q_rows < 0 || info->reserved != 0 ||
      info->work_bytes != uint64_t(info->num_items) * kItemInts * 4 ||
      info->tokens_per_item != kExtendRows / (desc->num_q_heads / desc->num_kv_heads))
    return SF_ERR_PLAN_MISMATCH;
  if (info->num_items == 0) return SF_OK;
  ExtendArgs a;
  if ((st = extend_args(desc, work_dev, q, k_new, v_new, k_pool, v_pool, block_table, out, lse, &a)) != SF_OK)
    return st;
  a.num_items = info->num_items;
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (work_host) {
    hipError_t e = hipMemcpyAsync(work_dev, work_host, info->work_bytes, hipMemcpyHostToDevice, s);
    if (e != hipSuccess) return SF_ERR_HIP;
  }
  return launch_extend(a, s) == hipSuccess ? SF_OK : SF_ERR_HIP;
}

extern "C" sf_status sf_debug_extend_plan(const sf_attn_desc* desc, const int32_t* seq_lens_host,
                                          const int32_t* q_lens_host, int32_t num_cus, int32_t store,
                                          int32_t* work_host, uint64_t work_capacity_bytes, int32_t* counts) {
  if (!counts || num_cus < 0 || (work_capacity_bytes > 0 && !work_host)) return SF_ERR_INVALID_ARG;
  ExtendPlan plan = {};
  sf_extend_info info;
  sf_status st = SF_OK;
  try {
    st = extend_plan_parts(desc, seq_lens_host, q_lens_host, num_cus, store != 0, work_host, work_capacity_bytes, &plan,
                           &info);
  } catch (const std::bad_alloc&) {
    return SF_ERR_HIP;
  }
  const int32_t c[5] = {plan.rows, plan.num_parts, plan.num_merge, plan.num_store, plan.num_slots};
  std::memcpy(counts, c, sizeof c);
  return st;
}
