// Host-side length-aware split-K planner (pure integer work, no device calls).
//
// Rollout batches mix a few very long trajectories with many short ones
// (Sec. 2.3 of the paper); the paper balances that skew across rollout
// instances by routing and migration (Sec. 5.3). Inside one GPU the same job
// falls to this planner: it lays every (sequence, KV head) page range end to
// end and gives each resident attention wave (a worker) an equal slice of the
// pages, cut at pair boundaries into segments. Long sequences are then read
// by many waves at once and every wave finishes at about the same time,
// whatever the skew. The exact rule is stated in sf_decode_attn.h next to
// sf_decode_attn_plan.
#include <algorithm>
#include <cfloat>
#include <cmath>
#include <cstring>
#include <memory>
#include <new>
#include <vector>

#include "sf_internal.h"

static_assert(sizeof(sf_attn_desc) == 32, "sf_attn_desc layout is part of the ABI");
static_assert(sizeof(sf_plan_opts) == 20, "sf_plan_opts layout is part of the ABI");
static_assert(sizeof(sf_plan_info) == 48, "sf_plan_info layout is part of the ABI");
static_assert(sizeof(sf_cost_model) == 48 && sizeof(sf_instance_state) == 24 && sizeof(sf_trajectory) == 16,
              "cost-model structs are part of the ABI");

namespace sf {

uint64_t align256(uint64_t x) { return (x + 255u) & ~uint64_t(255u); }

sf_status validate_desc(const sf_attn_desc* d) {
  if (!d) return SF_ERR_INVALID_ARG;
  if (d->num_seqs < 0 || d->num_q_heads < 1 || d->num_kv_heads < 1) return SF_ERR_INVALID_ARG;
  if (d->num_q_heads % d->num_kv_heads != 0) return SF_ERR_INVALID_ARG;
  if (d->block_table_stride < 1 || d->num_pages < 0) return SF_ERR_INVALID_ARG;
  // The kernels scale scores by |softmax_scale| * log2(e) in float, which must
  // be finite (false for NaN as well).
  if (!(std::fabs(double(d->softmax_scale)) * 1.4426950408889634074 <= double(FLT_MAX))) return SF_ERR_INVALID_ARG;
  if (d->head_dim != 64 && d->head_dim != 128) return SF_ERR_UNSUPPORTED;
  if (d->page_size != kPage) return SF_ERR_UNSUPPORTED;
  if (d->num_q_heads / d->num_kv_heads > kMaxGroup) return SF_ERR_UNSUPPORTED;
  return SF_OK;
}

uint64_t desc_key(const sf_attn_desc* d) {
  // FNV-1a over the shape fields a plan depends on.
  const int32_t f[8] = {0x5f440001, d->num_seqs, d->num_q_heads, d->num_kv_heads,
                        d->head_dim, d->page_size, d->block_table_stride, d->num_pages};
  uint64_t h = 1469598103934665603ull;
  const unsigned char* p = reinterpret_cast<const unsigned char*>(f);
  for (size_t i = 0; i < sizeof f; ++i) {
    h ^= p[i];
    h *= 1099511628211ull;
  }
  return h;
}

Workspace carve_workspace(void* base, int32_t slots, int32_t g, int32_t d) {
  Workspace w;
  char* b = static_cast<char*>(base);
  w.part_o = reinterpret_cast<float*>(b);
  w.part_lse = reinterpret_cast<float*>(b + align256(uint64_t(slots) * g * d * 4));
  return w;
}

}  // namespace sf

using namespace sf;

extern "C" sf_status sf_decode_attn_plan(const sf_attn_desc* desc, const int32_t* seq_lens_host,
                                         const sf_plan_opts* opts, int32_t* work_host,
                                         uint64_t work_capacity_bytes, sf_plan_info* info) {
  sf_status st = validate_desc(desc);
  if (st != SF_OK) return st;
  if (!info || (desc->num_seqs > 0 && !seq_lens_host)) return SF_ERR_INVALID_ARG;

  const int32_t B = desc->num_seqs;
  const int32_t hkv = desc->num_kv_heads;
  int32_t num_cus = kDefaultNumCus, forced = 0, wpc = kDefaultWorkersPerCu, mn = kDefaultMinChunk;
  int32_t skew = 0;
  if (opts) {
    if (opts->num_cus < 0 || opts->chunk_pages < 0 || opts->workers_per_cu < 0 ||
        opts->min_chunk_pages < 0 || opts->xcd_parity_skew < -kMaxParitySkew ||
        opts->xcd_parity_skew > kMaxParitySkew)
      return SF_ERR_INVALID_ARG;
    if (opts->num_cus) num_cus = opts->num_cus;
    forced = opts->chunk_pages;
    if (opts->workers_per_cu) wpc = opts->workers_per_cu;
    if (opts->min_chunk_pages) mn = opts->min_chunk_pages;
    skew = opts->xcd_parity_skew;
  }

  // Pages per sequence (every KV head of a sequence has the same count).
  thread_local std::vector<int32_t> spg_buf;
  spg_buf.resize(size_t(B));
  int32_t* spg = spg_buf.data();
  int64_t total = 0;
  for (int32_t s = 0; s < B; ++s) {
    const int32_t L = seq_lens_host[s];
    if (L < 0 || (L > 0 && desc->num_pages == 0)) return SF_ERR_INVALID_ARG;
    const int64_t npg = (int64_t(L) + kPage - 1) / kPage;
    if (npg > desc->block_table_stride) return SF_ERR_INVALID_ARG;
    spg[s] = int32_t(npg);
    total += npg * hkv;
  }
  if (total > (int64_t(1) << 40)) return SF_ERR_INVALID_ARG;
  const int64_t num_pairs = int64_t(B) * hkv;
  int64_t workers;
  if (num_pairs == 0) {
    workers = 0;
  } else if (total == 0) {
    workers = 1;  // only empty pairs: one worker writes their zero rows
  } else if (forced > 0) {
    workers = (total + forced - 1) / forced;
  } else {
    workers = std::min<int64_t>(int64_t(wpc) * num_cus, (total + mn - 1) / mn);
  }
  if (workers > INT32_MAX / 2) return SF_ERR_INVALID_ARG;

  // The attention launch runs workers G b .. G b + G - 1 as workgroup b
  // (one wave each), and workgroup b runs on XCD b mod 8. G is the largest
  // of 8, 4, 2 that packs the workers into whole rounds of one workgroup per
  // CU (W a multiple of G num_cus), else 1: a partial round would leave some
  // CUs with one group more than others.
  int32_t group = 1;
  for (const int32_t g : {8, 4, 2})
    if (workers >= g * int64_t(num_cus) && workers % (g * int64_t(num_cus)) == 0) {
      group = g;
      break;
    }

  // Worker range starts lo(w) = floor(T C(w) / C(W)) with the cumulative
  // weight C(v) = 1000 v + p D(v), D(v) = v mod G if floor(v / G) is even,
  // else G - v mod G: a worker of an even group weighs 1000 + p, of an odd
  // group 1000 - p (|p| <= 250; p = 0 for a forced slice size). Walked
  // forward without divisions: T C(v) grows by T (1000 + p) or T (1000 - p),
  // each positive and below 2^51, and quotient and remainder advance by
  // those over C(W) > 0.
  if (forced > 0) skew = 0;
  struct Cuts {
    int64_t q = 0, r = 0, den = 1, idx = 0, g = 1;
    int64_t dq[2] = {0, 0}, dr[2] = {0, 0};   // [group parity of v]: step from C(v) to C(v + 1)
    void init(int64_t t, int64_t w, int64_t p, int64_t grp) {
      q = r = idx = 0;
      g = grp;
      const int64_t rem = w % g;
      den = w > 0 ? 1000 * w + p * (((w / g) & 1) ? g - rem : rem) : 1;
      for (int k = 0; k < 2; ++k) {
        const int64_t inc = t * (k == 0 ? 1000 + p : 1000 - p);
        dq[k] = inc / den;
        dr[k] = inc % den;
      }
    }
    void next() {
      const int k = int((idx / g) & 1);
      q += dq[k];
      r += dr[k];
      if (r >= den) {
        r -= den;
        ++q;
      }
      ++idx;
    }
  };

  // Pass 1: segments per pair. Worker ranges are cut at pair boundaries; a
  // pair spanning k worker boundaries has k + 1 segments. Pairs are walked in
  // order (s-major, kvh-minor) with a worker cursor that only moves forward.
  // Returns the number of cut pairs.
  auto segments = [&](int64_t p_skew, int32_t* nseg) -> int64_t {
    Cuts next_lo;           // lo(cur + 1)
    next_lo.init(total, workers, p_skew, group);
    next_lo.next();
    int64_t cur = 0;        // worker whose range holds `start`
    int64_t start = 0;      // global page where the current pair starts
    int64_t p = 0, cut = 0;
    for (int32_t s = 0; s < B; ++s) {
      const int64_t npg = spg[s];
      for (int32_t h = 0; h < hkv; ++h, ++p) {
        if (npg == 0) {
          nseg[p] = 1;
          continue;
        }
        while (cur + 1 < workers && next_lo.q <= start) {
          ++cur;
          next_lo.next();
        }
        // boundaries lo(w) inside (start, start + npg) each add a segment
        int32_t k = 1;
        while (cur + 1 < workers && next_lo.q < start + npg) {
          ++cur;
          next_lo.next();
          ++k;
        }
        nseg[p] = k;
        cut += k > 1;
        start += npg;
      }
    }
    return cut;
  };
  if (skew != 0 && workers > 1) {
    // Slices near one page: a skew that would leave a worker without a page
    // falls back to equal slices (which give every worker at least one, since
    // W <= T), so every worker has a segment.
    Cuts c;
    c.init(total, workers, skew, group);
    int64_t prev = 0;
    for (int64_t w = 0; w < workers; ++w) {
      c.next();
      if (c.q == prev) {
        skew = 0;
        break;
      }
      prev = c.q;
    }
  }
  thread_local std::vector<int32_t> nseg_buf, nseg_alt;
  nseg_buf.resize(size_t(num_pairs));
  int32_t* nseg = nseg_buf.data();
  if (skew != 0 && workers > 1) {
    // The skew moves every boundary off the equal cuts; where those fall on
    // pair boundaries (equal lengths, page-aligned) it would cut pairs the
    // equal slices leave whole. Keep it unless it cuts more than W / 8 pairs
    // more than they do.
    nseg_alt.resize(size_t(num_pairs));
    const int64_t cut_skew = segments(skew, nseg);
    const int64_t cut_equal = segments(0, nseg_alt.data());
    if (cut_skew - cut_equal > workers / 8) {
      skew = 0;
      nseg_buf.swap(nseg_alt);
      nseg = nseg_buf.data();
    }
  } else {
    segments(skew, nseg);
  }
  int64_t n_work = 0, n_comb = 0, n_part = 0;
  for (int64_t p = 0; p < num_pairs; ++p) {
    n_work += nseg[p];
    if (nseg[p] > 1) {
      ++n_comb;
      n_part += nseg[p];
    }
  }
  const int64_t table_rows = workers;   // one row per worker
  if (table_rows + n_work + n_comb > INT32_MAX / kItemInts || n_part > INT32_MAX) return SF_ERR_INVALID_ARG;
  const int32_t g = desc->num_q_heads / hkv;
  info->num_workers = int32_t(workers);
  info->num_work = int32_t(n_work);
  info->num_combine = int32_t(n_comb);
  info->num_partials = int32_t(n_part);
  {
    // the widest slice (an even group's worker's when the slices are skewed)
    Cuts c;
    c.init(total, workers, skew, group);
    int64_t prev = 0, widest = 0;
    for (int64_t w = 0; w < workers; ++w) {
      c.next();
      widest = std::max(widest, c.q - prev);
      prev = c.q;
    }
    info->chunk_pages = int32_t(widest);
  }
  info->workers_per_group = group;
  info->work_bytes = uint64_t(table_rows + n_work + n_comb) * kItemInts * 4;
  info->workspace_bytes =
      n_part ? align256(uint64_t(n_part) * g * desc->head_dim * 4) + align256(uint64_t(n_part) * g * 4) : 0;
  info->desc_key = desc_key(desc);
  if (!work_host) return SF_OK;
  if (work_capacity_bytes < info->work_bytes) return SF_ERR_CAPACITY;

  // Pass 2: partial slots and combine rows (pairs with several segments, in pair order).
  int32_t* table = work_host;
  int32_t* items = work_host + table_rows * kItemInts;
  int32_t* comb = items + n_work * kItemInts;
  std::memset(table, 0, size_t(table_rows) * kItemInts * 4);
  thread_local std::vector<int32_t> base_buf, cidx_buf;
  base_buf.assign(size_t(num_pairs), -1);
  cidx_buf.assign(size_t(num_pairs), -1);
  {
    int32_t slot = 0, ci = 0;
    int64_t p = 0;
    for (int32_t s = 0; s < B; ++s) {
      for (int32_t h = 0; h < hkv; ++h, ++p) {
        if (nseg[p] <= 1) continue;
        base_buf[size_t(p)] = slot;
        cidx_buf[size_t(p)] = ci;
        const int32_t c8[kItemInts] = {s, h, slot, nseg[p], seq_lens_host[s], 0, 0, 0};
        std::memcpy(comb + int64_t(ci) * kItemInts, c8, sizeof c8);
        slot += nseg[p];
        ++ci;
      }
    }
  }
  const int32_t* base = base_buf.data();
  const int32_t* cidx = cidx_buf.data();

  // Pass 3: items, worker by worker; a worker's segments in pair order, then
  // the empty pairs e with e mod workers == w.
  thread_local std::vector<int64_t> empty_buf;
  empty_buf.clear();
  int64_t n_empty = 0;
  for (int32_t s = 0; s < B; ++s) n_empty += spg[s] == 0 ? hkv : 0;
  empty_buf.reserve(size_t(n_empty));
  for (int32_t s = 0; s < B; ++s)
    if (spg[s] == 0)
      for (int32_t h = 0; h < hkv; ++h) empty_buf.push_back(int64_t(s) * hkv + h);
  // Cursor over the non-empty pairs: pair p = (ps, ph).
  int64_t p = 0;
  int32_t ps = 0, ph = 0;
  auto skip_empty = [&]() {
    while (ps < B && spg[ps] == 0) {
      ++ps;
      p = int64_t(ps) * hkv;
      ph = 0;
    }
  };
  auto advance = [&]() {
    ++p;
    if (++ph == hkv) {
      ph = 0;
      ++ps;
    }
    skip_empty();
  };
  skip_empty();
  int64_t row = 0, pstart = 0;
  int32_t seg_c = 0;  // segment index within the current pair
  Cuts lo_w, hi_w;
  lo_w.init(total, workers, skew, group);
  hi_w.init(total, workers, skew, group);
  hi_w.next();
  for (int64_t w = 0; w < workers; ++w, lo_w.next(), hi_w.next()) {
    const int64_t lo = lo_w.q, hi = hi_w.q;
    const int64_t first = row;
    int64_t cnt = 0;
    while (ps < B && pstart < hi) {
      const int64_t npg = spg[ps];
      const int64_t b = std::max(lo, pstart) - pstart, e = std::min(hi, pstart + npg) - pstart;
      int32_t* r = items + row * kItemInts;
      r[0] = ps;
      r[1] = ph;
      r[2] = int32_t(b);
      r[3] = int32_t(e);
      r[4] = seq_lens_host[ps];
      r[5] = nseg[p] > 1 ? base[p] + seg_c : -1;
      r[6] = cidx[p];
      r[7] = nseg[p];
      ++row;
      ++cnt;
      if (pstart + npg <= hi) {  // pair finished inside this worker
        pstart += npg;
        seg_c = 0;
        advance();
      } else {
        ++seg_c;
        break;
      }
    }
    for (size_t e = size_t(w); e < empty_buf.size(); e += size_t(workers)) {
      const int64_t q = empty_buf[e];
      int32_t* r = items + row * kItemInts;
      const int32_t r8[kItemInts] = {int32_t(q / hkv), int32_t(q % hkv), 0, 0, 0, -1, -1, 1};
      std::memcpy(r, r8, sizeof r8);
      ++row;
      ++cnt;
    }
    // the worker's row: first item, item count, the first item's fields
    int32_t* t = table + w * kItemInts;
    t[0] = int32_t(first);
    t[1] = int32_t(cnt);
    if (cnt > 0) std::memcpy(t + 2, items + first * kItemInts, 6 * sizeof(int32_t));
  }
  return row == n_work ? SF_OK : SF_ERR_INVALID_ARG;
}

// ---------------------------------------------------------------------------
// the runner's plan
// ---------------------------------------------------------------------------
namespace {

// Batches of few pages per worker are latency bound: the attention kernel
// takes as long as its slowest worker, and each segment after a worker's first
// costs about 3 us of dependent loads (query, block table, first block), more
// than the equal slices save. For them the runner cuts the pairs themselves
// into equal segments of at most `most` pages, one per workgroup of 1 to 8
// waves that share its pages and merge in LDS; where no pair is cut there is
// no merge launch. Attention + merge kernels (us) with equal slices and with
// whole segments (28/4 heads, head_dim 128, unless noted; W waves in groups
// of G):
//   4 sequences of 17 .. 300 tokens, 4/1 heads, D = 64   12.2   6.2 (W 16, G 4)
//   1 of 1000 tokens                                     10.5  10.5 (W 256, G 4, cut)
//   1 of 32768                                           22.9  20.5 (W 1024, G 4, cut)
//   16 of 1000                                           19.8  16.5 (W 1024, G 4, cut)
//   64 of up to 600                                      20.9  15.8 (W 2048, G 8)
//   300 of up to 80                                      29.0  15.5 (W 1200, G 1)
//   40 of up to 300, 40/8 heads                          26.5  13.4 (W 1280, G 4)
//   200 of up to 200 and two of 16000 and 9000           41.6  35.2 (W 1020, G 1, cut)
//   the last four over an fp8 cache: 19.7  16.8, 27.1  12.9, 24.3  11.3, 39.8  24.3
// With many pages per worker the slices' balance wins: 64 sequences of 512 to
// 4096 tokens 57.1 and 56.9 us, 128 of them 99.3 and 104.4. Groups of 8 where
// workgroups are few load few CUs: 16 sequences of 1000 tokens 17.9 us with G
// 8 and no cut, against 12.2 + 4.3.
//
// Both plans' times are estimated (us, fitted to those measurements): the
// attention kernel is the longer of its slowest worker (launch, waves to start,
// pages one after another, segments after its first) and the stream of the
// whole batch's bytes; cut pairs add the merge launch (depth: segments of the
// pair cut most).
struct RunnerCost {
  double page;       // a page in one of many waves; half that in a lone one
  double gbytes;     // GB/s of the whole chip
  double bytes;      // K and V bytes of a page
  double merge;      // the merge launch, or what cut pairs add to an appending step's
  int64_t cus;
};
constexpr double kLaunchUs = 4.0, kWaveUs = 0.002, kSegmentUs = 3.0, kStreamUs = 6.5;
constexpr double kShareUs = 0.3, kMergeUs = 4.0, kMergeAppendUs = 0.5, kPartialUs = 0.0005, kDepthUs = 0.014;
constexpr int64_t kDepth = 128;   // segments of a pair that the merge takes without more time
// Pages per worker (at 4 per CU) beyond which the slices are always taken.
constexpr int64_t kRunnerPages = 40;

double runner_estimate(const RunnerCost& c, int64_t total, int64_t workers, int64_t longest, int64_t extra_segments,
                       int64_t partials, int64_t depth, int32_t sharing = 1) {
  const double page = c.page * (0.5 + 0.5 * std::min(1.0, double(workers) / double(2 * c.cus))) * (1.0 + 0.065 * (sharing - 1));
  const double worker = kLaunchUs + kWaveUs * double(workers) + page * double(longest) + kSegmentUs * double(extra_segments) +
                        kShareUs * (sharing - 1);
  // workers of unequal length do not draw the full rate to the end
  const double uneven = std::max(1.0, double(longest) * double(workers) / double(total));
  const double stream = kStreamUs + double(total) * c.bytes / (c.gbytes * 1e3) * (0.5 + 0.5 * uneven);
  return std::max(worker, stream) +
         (partials > 0 ? c.merge + kPartialUs * double(partials) + kDepthUs * double(std::max<int64_t>(0, depth - kDepth)) : 0.0);
}

int32_t pages_of(int32_t tokens) { return int32_t((int64_t(tokens) + kPage - 1) / kPage); }

bool slices_left_to_planner(const sf_plan_opts& o) {
  return o.chunk_pages == 0 && o.workers_per_cu == 0 && o.min_chunk_pages == 0 && o.xcd_parity_skew == 0 && o.num_cus >= 0;
}

}  // namespace

sf_status sf::decode_plan_runner(const sf_attn_desc* desc, const int32_t* seq_lens_host, const sf_plan_opts* opts,
                                 StepKind kind, int32_t* work_host, uint64_t work_capacity_bytes, sf_plan_info* info) {
  const bool fp8 = kind == StepKind::kFp8, append = kind == StepKind::kAppend;
  sf_plan_opts o = {};
  if (opts) o = *opts;
  const bool free_choice = slices_left_to_planner(o);   // the caller's own choice of slices stands
  // An fp8 block moves half the bytes of a bf16 one: unless the caller chose,
  // fp8 steps plan two waves per SIMD (measured: kernel 129 us instead of 136
  // on the long-tail batch; bf16 is slower at 8).
  if (fp8 && o.workers_per_cu == 0) o.workers_per_cu = kFp8WorkersPerCu;
  auto slices = [&]() {
    return sf_decode_attn_plan(desc, seq_lens_host, &o, work_host, work_capacity_bytes, info);
  };
  if (!free_choice || validate_desc(desc) != SF_OK || !info || desc->num_seqs == 0 || !seq_lens_host) return slices();

  const int64_t cus = o.num_cus ? o.num_cus : kDefaultNumCus;
  const int64_t hkv = desc->num_kv_heads, g = desc->num_q_heads / hkv;
  const int32_t B = desc->num_seqs;
  // Pages of the sequences that have any, as floats (exact below kExact).
  constexpr int64_t kExact = int64_t(1) << 23;
  const std::unique_ptr<float[]> pages(new (std::nothrow) float[size_t(B)]);
  if (!pages) return slices();
  int64_t total = 0, longest_pair = 0;
  int32_t some = 0;
  for (int32_t s = 0; s < B; ++s) {
    const int32_t L = seq_lens_host[s];
    if (L < 0 || (L > 0 && desc->num_pages == 0)) return SF_ERR_INVALID_ARG;
    const int64_t npg = pages_of(L);
    if (npg > desc->block_table_stride) return SF_ERR_INVALID_ARG;
    total += npg * hkv;
    longest_pair = std::max(longest_pair, npg);
    pages[some] = float(npg);
    some += npg > 0;
  }
  const int64_t pairs = some * hkv, empty = int64_t(B) * hkv - pairs;
  if (total == 0 || total > kRunnerPages * 4 * cus || pairs + empty > 8 * cus || longest_pair >= kExact) return slices();

  // Segments of at most `most` pages: their number (an empty pair is one), the
  // cut pairs and their segments. The search below counts several dozen times
  // at most, each on the critical path of a step: without a division per
  // sequence, in a loop that the compiler turns into vector code.
  struct Count {
    int64_t segments = 0, cut = 0, partials = 0, longest = 0;
  };
  auto count = [&](int64_t most) {
    const float m = float(most), inv = 1.f / m;
    int32_t segments = 0, cut = 0, longest = 0;
    for (int32_t s = 0; s < some; ++s) {
      const float n = pages[s];
      float q = float(int32_t((n - 1.f) * inv));          // floor((n - 1) / most), or one off:
      const float rem = (n - 1.f) - q * m;                // whole numbers below kExact, so exact
      q += rem >= m ? 1.f : 0.f;
      q -= rem < 0.f ? 1.f : 0.f;
      const float length = n / (q + 1.f);                 // rounds to no other whole number
      segments += int32_t(q) + 1;
      cut += q > 0.f ? 1 : 0;
      longest = std::max(longest, int32_t(length) + (float(int32_t(length)) < length ? 1 : 0));
    }
    Count c;
    c.segments = segments * hkv + empty;
    c.cut = cut * hkv;
    c.partials = (int64_t(segments) - (some - cut)) * hkv;
    c.longest = longest;
    return c;
  };
  const RunnerCost cost = {(fp8 ? 0.75 : 0.95) * (desc->head_dim == 64 ? 0.75 : 1.0),
                           (fp8 ? 5700.0 : 6000.0) * double(cus) / 256, double(kPage) * desc->head_dim * (fp8 ? 2 : 4),
                           append ? kMergeAppendUs : kMergeUs, cus};
  // The slices: segments of the worker that has most, i.e. pairs that a window
  // of one slice can touch, walked over the sequences (hkv equal pairs each).
  const int64_t wpc = o.workers_per_cu ? o.workers_per_cu : kDefaultWorkersPerCu;
  const int64_t slice_workers = std::min<int64_t>(wpc * cus, (total + kDefaultMinChunk - 1) / kDefaultMinChunk);
  const int64_t slice = (total + slice_workers - 1) / slice_workers;
  int64_t most_segments = 1, window = 0, window_pairs = 0;
  bool whole_pairs = total % slice_workers == 0;   // every slice is one pair
  for (int32_t s = 0, first = 0; s < some; ++s) {
    const int64_t n = int64_t(pages[s]);
    whole_pairs = whole_pairs && n == slice;
    window += n * hkv;
    window_pairs += hkv;
    while (window > slice && first < s) {
      window -= int64_t(pages[first++]) * hkv;
      window_pairs -= hkv;
    }
    // (slice / n: both below 2^31, as slice < n hkv here)
    most_segments = std::max(most_segments, window <= slice ? window_pairs + 1
                                            : n > slice     ? 1
                                                            : std::min<int64_t>(hkv, int32_t(slice) / int32_t(n)) + 1);
  }
  double best_us = runner_estimate(cost, total, slice_workers, slice, whole_pairs ? 0 : most_segments - 1,
                                   whole_pairs ? 0 : slice_workers + std::min(pairs, slice_workers), longest_pair / slice + 1);
  int32_t best = 0, waves = 1;
  Count chosen;
  struct Found {
    int64_t target = 0, least = 0, most = 0;
    Count c;
  } seen[12];   // cuts found so far (the group sizes share targets)
  int32_t num_seen = 0;
  for (const int32_t g8 : {1, 2, 4, 8}) {
    if ((pairs + empty) * g8 > 8 * cus) break;
    int64_t last = 0;
    auto consider = [&](int64_t most, const Count& c) {
      if (most == last) return;
      last = most;
      const double us = runner_estimate(cost, total, c.segments * g8, (c.longest + g8 - 1) / g8, 0, c.partials,
                                        (longest_pair + most - 1) / most, g8);
      if (us < best_us) best_us = us, best = int32_t(most), waves = g8, chosen = c;
    };
    Count whole;
    whole.segments = pairs + empty;
    whole.longest = longest_pair;
    consider(longest_pair, whole);
    for (int32_t r = 1; r <= 3; ++r) {
      // the shortest segments that take at most `target` waves, within 1/32;
      // more than four waves per CU only where the pairs alone need them. Best
      // group at 4 and at 8 waves per CU, 28/4 heads, steps in us: one sequence
      // of 32768 16.4 and 17.7, over fp8 14.7 and 17.4, one of 8192 14.7 and
      // 17.6, 16 of 1000 14.7 and 17.7, 16 of 4000 26.1 and 25.9
      const int64_t target = (cus << r) / g8;   // workgroups
      if (pairs + empty > target || (r == 3 && (pairs + empty) * g8 <= 4 * cus)) continue;
      const int64_t least = std::max<int64_t>(g8, (total + target - 1) / target);
      if (least >= longest_pair) continue;   // no pair would be cut
      // no plan with a merge beats the stream of the batch's bytes and the merge
      if (kStreamUs + double(total) * cost.bytes / (cost.gbytes * 1e3) + cost.merge >= best_us) continue;
      bool found = false;
      for (const Found& f : seen)
        if (f.target == target && f.least <= least && least <= f.most) consider(f.most, f.c), found = true;
      if (found) continue;
      // About A + B / m segments of at most m pages: each count moves one end of
      // the bracket there, a little to the side that fits.
      int64_t most = longest_pair, low = 0;
      double low_segments = 0;
      Count c = whole;
      for (int64_t m = least;; ) {
        const Count n = count(m);
        if (n.segments <= target)
          most = m, c = n;
        else
          low = m, low_segments = double(n.segments);
        if (low == 0 || most - low <= std::max<int64_t>(1, low / 32)) break;
        const double b = (low_segments - double(c.segments)) / (1.0 / double(low) - 1.0 / double(most));
        const double at = b / (double(target) - low_segments + b / double(low));
        const int64_t gap = std::max<int64_t>(1, (most - low) / 8);
        m = std::min(most - gap, std::max(low + gap, int64_t(std::min(at * 1.02, double(most))) + 1));
      }
      seen[num_seen++] = {target, least, most, c};
      consider(most, c);
    }
  }
  if (best == 0) return slices();

  const int64_t work = chosen.segments, workers = work * waves;
  int32_t group = waves;
  if (waves == 1)   // one segment per worker: the fewest waves per workgroup that give one round of workgroups
    for (group = 1; group < 8 && workers > group * cus;) group *= 2;
  info->num_workers = int32_t(workers);
  info->num_work = int32_t(work);
  info->num_combine = int32_t(chosen.cut);
  info->num_partials = int32_t(chosen.partials);
  info->chunk_pages = int32_t((chosen.longest + waves - 1) / waves);
  info->workers_per_group = waves > 1 ? kSharedGroups + group : group;
  info->work_bytes = uint64_t(workers + work + chosen.cut) * kItemInts * 4;
  info->workspace_bytes = chosen.partials ? align256(uint64_t(chosen.partials) * g * desc->head_dim * 4) +
                                                align256(uint64_t(chosen.partials) * g * 4)
                                          : 0;
  info->desc_key = desc_key(desc);
  if (!work_host) return SF_OK;
  if (work_capacity_bytes < info->work_bytes) return SF_ERR_CAPACITY;

  int32_t* table = work_host;
  int32_t* items = table + workers * kItemInts;
  int32_t* comb = items + work * kItemInts;
  int32_t item = 0, slot = 0, cut = 0;
  for (int32_t s = 0; s < B; ++s) {
    const int32_t L = seq_lens_host[s], n = pages_of(L);
    const int32_t k = n <= best ? 1 : (n + best - 1) / best;
    for (int32_t h = 0; h < hkv; ++h) {
      if (k > 1) {
        const int32_t c8[kItemInts] = {s, h, slot, k, L, 0, 0, 0};
        std::memcpy(comb + int64_t(cut) * kItemInts, c8, sizeof c8);
      }
      for (int32_t i = 0; i < k; ++i, ++item) {
        const int32_t b = int32_t(int64_t(i) * n / k), e = int32_t(int64_t(i + 1) * n / k);
        const int32_t r8[kItemInts] = {s, h, b, e, L, k > 1 ? slot++ : -1, k > 1 ? cut : -1, k};
        std::memcpy(items + int64_t(item) * kItemInts, r8, sizeof r8);
        for (int32_t j = 0; j < waves; ++j) {
          const int32_t pb = b + int32_t(int64_t(j) * (e - b) / waves), pe = b + int32_t(int64_t(j + 1) * (e - b) / waves);
          const int32_t t8[kItemInts] = {item, 1, s, h, pb, pe, L, r8[5]};
          std::memcpy(table + (int64_t(item) * waves + j) * kItemInts, t8, sizeof t8);
        }
      }
      cut += k > 1;
    }
  }
  return SF_OK;
}

// A batch of at most num_seqs sequences and total_pages pages (of all its pairs;
// < 0: any number), whatever the kind of its step, is planned as one of
//   equal slices: at most W workers (the options' per CU; left to the planner,
//     kDefaultWorkersPerCu, or kFp8WorkersPerCu over an fp8 cache; no more than
//     one per smallest slice). Each of the W - 1 boundaries between them adds a
//     segment to a pair and may cut it;
//   segments of pairs (options left to the planner): at most 8 workers per CU
//     and 8 per pair and page, and at most one segment per pair and page, 8 per
//     CU where the pairs alone are more than 4 per CU, 4 per CU otherwise (or
//     where a workgroup's waves share a segment).
// Without total_pages a forced slice size has no such bound, and more than
// kReserveWorkers workers are beyond what any batch here needs: the caller's
// bytes stand alone then.
constexpr int64_t kReserveWorkers = 1 << 14;

sf::ReserveBytes sf::reserve_bytes(const sf_attn_desc* shape, const sf_plan_opts* opts, uint64_t workspace_bytes,
                                   uint64_t work_bytes, int32_t num_seqs, int64_t total_pages) {
  const sf_plan_opts none = {};
  const sf_plan_opts& o = opts ? *opts : none;
  const int64_t cus = o.num_cus > 0 ? o.num_cus : kDefaultNumCus;
  const int64_t pairs = int64_t(num_seqs) * shape->num_kv_heads;
  const uint64_t pages = (uint64_t(num_seqs) * 4 + 31) / 32 * 32;   // an appending step's new pages, as kept
  // an appending step also keeps a copy of at most one row per work item
  int64_t partials = 0, rows = 0, append_rows = 0;
  auto plan = [&](int64_t workers, int64_t segments, int64_t cut_segments, int64_t cut, bool appending) {
    partials = std::max(partials, cut_segments);
    rows = std::max(rows, workers + segments + cut);
    if (appending) append_rows = std::max(append_rows, workers + 2 * segments + cut);
  };
  const bool known = total_pages >= 0;
  auto slices = [&](int64_t w, int64_t least, bool appending) {
    if (known)
      w = std::max<int64_t>(1, std::min(w, (total_pages + least - 1) / least));
    else if (w > kReserveWorkers)
      return;
    const int64_t cut = std::min(pairs, w - 1);
    plan(w, pairs + w - 1, w - 1 + cut, cut, appending);
  };
  if (o.chunk_pages > 0) {
    slices(INT64_MAX, o.chunk_pages, true);
  } else {
    const int64_t least = o.min_chunk_pages ? o.min_chunk_pages : kDefaultMinChunk;
    slices((o.workers_per_cu ? o.workers_per_cu : kDefaultWorkersPerCu) * cus, least, true);
    if (o.workers_per_cu == 0) slices(kFp8WorkersPerCu * cus, least, false);
    if (slices_left_to_planner(o) && (known || 8 * cus <= kReserveWorkers)) {
      const int64_t each = known ? total_pages + pairs : INT64_MAX / 8;
      const int64_t segments = std::min(pairs > 4 * cus ? 8 * cus : 4 * cus, each);
      plan(std::min(8 * cus, 8 * each), segments, segments, std::min(pairs, segments / 2), true);
    }
  }
  const uint64_t head_rows = uint64_t(partials) * (shape->num_q_heads / shape->num_kv_heads);
  workspace_bytes = std::max(workspace_bytes, align256(head_rows * shape->head_dim * 4) + align256(head_rows * 4));
  const uint64_t row_bytes = kItemInts * 4;
  const uint64_t slot = std::max(2 * work_bytes, std::max(uint64_t(rows), uint64_t(append_rows)) * row_bytes) + pages;
  // on the device: the partial results, then copies of the merge rows (at most
  // the work list), and of an appending step's rows and new pages
  return {align256(workspace_bytes) + std::max(work_bytes, uint64_t(std::max(rows, append_rows)) * row_bytes) + pages,
          (slot + 4095) / 4096 * 4096};
}

extern "C" sf_status sf_debug_runner_reserve(const sf_attn_desc* shape, const sf_plan_opts* opts,
                                             uint64_t workspace_bytes, uint64_t work_bytes, int32_t max_num_seqs,
                                             int64_t total_pages, uint64_t* bytes) {
  if (!shape || !bytes || max_num_seqs < 0 || shape->num_kv_heads <= 0) return SF_ERR_INVALID_ARG;
  const ReserveBytes b = reserve_bytes(shape, opts, workspace_bytes, work_bytes, max_num_seqs, total_pages);
  bytes[0] = b.device;
  bytes[1] = b.slot;
  return SF_OK;
}

extern "C" sf_status sf_runner_plan(const sf_attn_desc* desc, const int32_t* seq_lens_host, const sf_plan_opts* opts,
                                    int32_t kind, int32_t* work_host, uint64_t work_capacity_bytes,
                                    sf_plan_info* info) {
  if (kind < 0 || kind > 2) return SF_ERR_INVALID_ARG;
  return decode_plan_runner(desc, seq_lens_host, opts, StepKind(kind), work_host, work_capacity_bytes, info);
}
