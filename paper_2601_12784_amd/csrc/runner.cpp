// Native per-step runner: plan -> attention (-> merge) in one call.
//
// A rollout instance runs one batched decode step after another (App. B.1:
// each step generates one token per running trajectory), so the host work
// between two steps is on the critical path once the kernels are short:
// small batches, late steps of a long-tail batch, an fp8 cache. This object
// keeps that work native. It owns a ring of pinned host buffers that the
// planner writes into and the kernels read in place (mapped host memory,
// zero-copy), the split-K workspace, and a few events:
//   - a slot is rewritten only after the step that read it has ended;
//   - nothing else orders the steps, so the host plans step i + 1 while the
//     kernels of step i run.
// An event recorded on the stream after every step delayed the next step's
// first launch by ~4.4 us (the marker's own dispatch; 2 % of a long-tail
// step), so one event marks a run of kMarkEvery steps on one stream instead;
// the ring holds kRing > kMarkEvery slots, so the run that holds a slot's
// last step is always marked before the slot comes round again.
// A separate upload (a copy stream, a device work list and a cross-stream
// wait) cost more per step than the kernels' in-place reads of the list, and
// how much more depended on whether the two streams shared a hardware queue.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <new>

#include "sf_internal.h"

static_assert(sizeof(sf_runner_memory) == 56, "sf_runner_memory layout is part of the ABI");
static_assert(sizeof(sf_runner_extras) == 56, "sf_runner_extras layout is part of the ABI");

namespace {

constexpr int kRing = 32;
constexpr int kMarkEvery = 16;
constexpr int kMarks = 4;
// Without a store launch to copy the rows, a copy launch (about 4 us) pays from
// about two rounds of workgroups on, each starting with a read over PCIe.
constexpr int kExtendCopyParts = 512;
const hipStream_t kNoStream = reinterpret_cast<hipStream_t>(~uintptr_t(0));   // no call yet
static_assert(kMarkEvery < kRing, "a slot's last step must be marked before the slot comes round again");

struct Pinned {
  int32_t* ptr = nullptr;          // host address (the planner writes here)
  const int32_t* dev = nullptr;    // the same memory as the kernels address it
  uint64_t bytes = 0;
  uint64_t last_step = 0;          // the step that last read it
  bool used = false;
  bool in_arena = false;           // part of sf_runner::arena, not an allocation of its own
};

// An event recorded on one stream after steps [begin, end), all on that stream.
struct Mark {
  hipEvent_t ev = nullptr;
  uint64_t begin = 0, end = 0;
  bool valid = false;
};

// Memory lent by sf_runner_extend's caller. Every few calls (a run: half the
// slots) the last launch of the call completes an event, which stands for the
// calls since the event before. Nothing is recorded on a stream after the call
// that was given it, so the caller may destroy it between calls: where calls
// without an event have to be waited for (the next call is on another stream,
// other memory comes, the runner goes), the device is. A runner that has seen
// two streams gives every call its event. (On every call of a single stream the
// events cost up to 2 us: three prompts of up to 61 tokens 16.4 against 14.4.)
struct Lent {
  void* pinned = nullptr;
  const char* pinned_dev = nullptr;   // the same memory as the kernels address it
  int32_t slots = 0;
  uint64_t slot_bytes = 0;
  void* device = nullptr;             // of the last call that lent it for longer than the call
  uint64_t device_bytes = 0;
  uint64_t next = 0;                  // slots go round
  hipEvent_t done[kRing] = {};        // created with the first call of the slot that takes one
  bool used[kRing] = {};              // a call whose end has not been waited for read the slot
  int event[kRing] = {};              // the slot whose event stands for that call; -1: none yet
  int unmarked = 0;                   // calls without an event so far
  bool streams = false;               // calls came on more than one stream
  hipStream_t last_stream = kNoStream;   // of the last call (compared, never used)
};

}  // namespace

struct sf_runner {
  sf_attn_desc shape;      // heads, head_dim, page size (per-step fields are overwritten)
  sf_plan_opts opts;
  int device = 0;
  Pinned ring[kRing];
  void* arena = nullptr;   // one allocation that sf_runner_reserve cut into slots
  Mark marks[kMarks];
  uint64_t num_marks = 0;  // marks recorded so far (the next one reuses marks[num_marks % kMarks])
  uint64_t unmarked = 0;   // steps [unmarked, steps) have no mark yet
  hipStream_t last_stream = nullptr;
  void* workspace = nullptr;
  uint64_t workspace_bytes = 0;
  Lent lent;
  uint64_t steps = 0;
  sf_plan_info last;
};

namespace {

// Records a mark after the unmarked steps, on the stream they ran on. The
// mark it reuses is waited for first, so a recycled event never stands for
// steps of another run.
sf_status mark_steps(sf_runner* r) {
  if (r->unmarked == r->steps) return SF_OK;
  Mark& m = r->marks[r->num_marks % kMarks];
  if (m.valid && hipEventSynchronize(m.ev) != hipSuccess) return SF_ERR_HIP;
  m.valid = false;
  if (hipEventRecord(m.ev, r->last_stream) != hipSuccess) return SF_ERR_HIP;
  m.begin = r->unmarked;
  m.end = r->steps;
  m.valid = true;
  r->unmarked = r->steps;
  ++r->num_marks;
  return SF_OK;
}

// Returns once step u (< steps) has ended on the GPU.
sf_status wait_step(sf_runner* r, uint64_t u) {
  if (u >= r->unmarked) {
    sf_status st = mark_steps(r);
    if (st != SF_OK) return st;
  }
  for (auto& m : r->marks)
    if (m.valid && m.begin <= u && u < m.end) return hipEventSynchronize(m.ev) == hipSuccess ? SF_OK : SF_ERR_HIP;
  return SF_OK;  // its mark was waited for and reused: the step has ended
}

// Returns once every step so far has ended.
sf_status wait_all(sf_runner* r) {
  sf_status st = mark_steps(r);
  for (auto& m : r->marks)
    if (m.valid && hipEventSynchronize(m.ev) != hipSuccess) st = SF_ERR_HIP;
  return st;
}

// Called only when no step in flight reads the slot (its last step has ended).
sf_status grow_pinned(Pinned& p, uint64_t bytes) {
  if (p.bytes >= bytes) return SF_OK;
  if (p.ptr && !p.in_arena && hipHostFree(p.ptr) != hipSuccess) return SF_ERR_HIP;
  p.in_arena = false;
  p.ptr = nullptr;
  p.dev = nullptr;
  p.bytes = 0;
  const uint64_t want = bytes + bytes / 4 + 4096;
  if (hipHostMalloc(reinterpret_cast<void**>(&p.ptr), want, hipHostMallocDefault) != hipSuccess) return SF_ERR_HIP;
  void* dev = nullptr;
  if (hipHostGetDevicePointer(&dev, p.ptr, 0) != hipSuccess) {
    (void)hipHostFree(p.ptr);
    p.ptr = nullptr;
    return SF_ERR_HIP;
  }
  p.dev = static_cast<const int32_t*>(dev);
  p.bytes = want;
  return SF_OK;
}

// The workspace grows only when nothing in flight can still use it: growing
// waits for the runner's steps and the stream (sf_runner_reserve does it
// ahead of the steps).
sf_status grow_device(sf_runner* r, void** ptr, uint64_t* have, uint64_t bytes, hipStream_t main) {
  if (*have >= bytes) return SF_OK;
  sf_status st = wait_all(r);
  if (st != SF_OK) return st;
  if (hipStreamSynchronize(main) != hipSuccess) return SF_ERR_HIP;
  if (*ptr && hipFree(*ptr) != hipSuccess) return SF_ERR_HIP;
  *ptr = nullptr;
  *have = 0;
  const uint64_t want = bytes + bytes / 4 + 4096;
  if (hipMalloc(ptr, want) != hipSuccess) return SF_ERR_HIP;
  *have = want;
  return SF_OK;
}

// Waits for the device where calls have no event.
sf_status wait_unmarked(Lent& l) {
  if (l.unmarked == 0) return SF_OK;
  if (hipDeviceSynchronize() != hipSuccess) return SF_ERR_HIP;
  std::fill(l.used, l.used + kRing, false);
  l.unmarked = 0;
  return SF_OK;
}

// Returns once the call that last read the lent slot has ended.
sf_status wait_slot(Lent& l, int slot) {
  if (!l.used[slot]) return SF_OK;
  if (l.event[slot] < 0) return wait_unmarked(l);
  if (hipEventSynchronize(l.done[l.event[slot]]) != hipSuccess) return SF_ERR_HIP;
  l.used[slot] = false;
  return SF_OK;
}

// Returns once every call on the lent memory has ended.
sf_status wait_lent(Lent& l) {
  sf_status st = wait_unmarked(l);
  for (int i = 0; i < kRing; ++i)
    if (wait_slot(l, i) != SF_OK) st = SF_ERR_HIP;
  return st;
}

}  // namespace

extern "C" sf_status sf_runner_create(const sf_attn_desc* shape, const sf_plan_opts* opts, sf_runner** out) {
  if (!out) return SF_ERR_INVALID_ARG;
  *out = nullptr;
  if (!shape) return SF_ERR_INVALID_ARG;
  sf_attn_desc probe = *shape;
  probe.num_seqs = 0;
  probe.block_table_stride = probe.block_table_stride > 0 ? probe.block_table_stride : 1;
  probe.num_pages = probe.num_pages >= 0 ? probe.num_pages : 0;
  sf_status st = sf::validate_desc(&probe);
  if (st != SF_OK) return st;
  if (opts && (opts->xcd_parity_skew < -sf::kMaxParitySkew || opts->xcd_parity_skew > sf::kMaxParitySkew))
    return SF_ERR_INVALID_ARG;
  sf_runner* r = new (std::nothrow) sf_runner();
  if (!r) return SF_ERR_HIP;
  r->shape = probe;
  if (opts) r->opts = *opts;
  else std::memset(&r->opts, 0, sizeof r->opts);
  if (hipGetDevice(&r->device) != hipSuccess) {
    delete r;
    return SF_ERR_HIP;
  }
  // The events only order the host's reuse of a slot after the GPU's reads
  // of it; they publish no GPU writes, so they skip the system-scope fence.
  for (auto& m : r->marks)
    if (hipEventCreateWithFlags(&m.ev, hipEventDisableTiming | hipEventDisableSystemFence) != hipSuccess)
      st = SF_ERR_HIP;
  if (st != SF_OK) {
    sf_runner_destroy(r);
    return st;
  }
  *out = r;
  return SF_OK;
}

// Teardown cannot report errors: every call is made, whatever the others return.
extern "C" void sf_runner_destroy(sf_runner* r) {
  if (!r) return;
  // a garbage collector may be here with any device current
  int current = r->device;
  (void)hipGetDevice(&current);
  if (current != r->device) (void)hipSetDevice(r->device);
  // Steps not yet marked ran on the caller's stream, which may be gone by
  // now: nothing is recorded on it here, the device is waited for instead.
  if (r->unmarked < r->steps) (void)hipDeviceSynchronize();
  for (auto& m : r->marks) {
    if (m.ev && m.valid) (void)hipEventSynchronize(m.ev);
    if (m.ev) (void)hipEventDestroy(m.ev);
  }
  (void)wait_lent(r->lent);
  for (auto ev : r->lent.done)
    if (ev) (void)hipEventDestroy(ev);
  for (auto& p : r->ring)
    if (p.ptr && !p.in_arena) (void)hipHostFree(p.ptr);
  if (r->arena) (void)hipHostFree(r->arena);
  if (r->workspace) {
    (void)hipDeviceSynchronize();
    (void)hipFree(r->workspace);
  }
  if (current != r->device) (void)hipSetDevice(current);
  delete r;
}

extern "C" sf_status sf_runner_step(sf_runner* r, const sf_attn_desc* desc, const int32_t* seq_lens_host,
                                    const void* q, const void* k_pool, const void* v_pool,
                                    const int32_t* block_table, float* out, float* lse,
                                    const sf_runner_extras* extras, void* stream, sf_plan_info* info_out) {
  if (!r || !desc || (desc->num_seqs > 0 && !seq_lens_host)) return SF_ERR_INVALID_ARG;
  if (desc->num_q_heads != r->shape.num_q_heads || desc->num_kv_heads != r->shape.num_kv_heads ||
      desc->head_dim != r->shape.head_dim || desc->page_size != r->shape.page_size)
    return SF_ERR_INVALID_ARG;
  const bool append = extras && extras->k_new;
  const bool fp8 = extras && extras->k_scale;
  if (extras && (append && fp8)) return SF_ERR_INVALID_ARG;
  if (append && !lse) return SF_ERR_INVALID_ARG;
  hipStream_t main = static_cast<hipStream_t>(stream);

  // 1. plan into the next ring slot (after the step that last read it has
  //    ended); grow it and plan again only if the plan does not fit
  Pinned& pin = r->ring[r->steps % kRing];
  sf_status st = pin.used ? wait_step(r, pin.last_step) : SF_OK;
  if (st != SF_OK) return st;
  pin.used = false;
  // A mark stands for steps of one stream: a new stream closes the run.
  if (r->unmarked < r->steps && main != r->last_stream && (st = mark_steps(r)) != SF_OK) return st;
  // Appending: after the work list, copies of the rows the merge launch acts
  // on (pairs with one segment and len > 0, at most one per item), then
  // new_pages. The work list ends with the combine rows, so the merge
  // launch's rows are one contiguous range, which the attention launch
  // copies to device memory (RowCopy).
  const uint64_t pages_bytes = append ? (uint64_t(desc->num_seqs) * 4 + 31) / 32 * 32 : 0;
  sf_plan_info info;
  const sf::StepKind kind = fp8 ? sf::StepKind::kFp8 : append ? sf::StepKind::kAppend : sf::StepKind::kPlain;
  st = sf::decode_plan_runner(desc, seq_lens_host, &r->opts, kind, pin.ptr, pin.bytes, &info);
  auto need = [&]() { return info.work_bytes + (append ? uint64_t(info.num_work) * 32 + pages_bytes : 0); };
  if (st == SF_ERR_CAPACITY || (st == SF_OK && pin.bytes < need())) {
    if ((st = grow_pinned(pin, need())) != SF_OK) return st;
    st = sf::decode_plan_runner(desc, seq_lens_host, &r->opts, kind, pin.ptr, pin.bytes, &info);
  }
  if (st != SF_OK) return st;
  const bool shared = info.workers_per_group > sf::kSharedGroups;
  if (shared) info.workers_per_group -= sf::kSharedGroups;
  int32_t num_single = 0;
  uint64_t pages_off = info.work_bytes;
  if (append && desc->num_seqs > 0) {
    if (!extras->new_pages_host) return SF_ERR_INVALID_ARG;
    char* base = reinterpret_cast<char*>(pin.ptr);
    const int32_t* items = pin.ptr + sf::table_rows(info.num_workers) * sf::kItemInts;
    int32_t* singles = reinterpret_cast<int32_t*>(base + info.work_bytes);
    for (int32_t i = 0; i < info.num_work; ++i) {
      const int32_t* row = items + int64_t(i) * sf::kItemInts;
      if (row[7] == 1 && row[4] > 0)
        std::memcpy(singles + int64_t(num_single++) * sf::kItemInts, row, sf::kItemInts * 4);
    }
    pages_off = info.work_bytes + uint64_t(num_single) * 32;
    std::memcpy(base + pages_off, extras->new_pages_host, uint64_t(desc->num_seqs) * 4);
  }
  if (info_out) *info_out = info;
  r->last = info;
  if (info.num_workers == 0) return SF_OK;

  // 2. workspace (grown only while idle): the partial results, then the
  //    device copy of what the merge launch reads from the ring: the combine
  //    rows and, appending, the single rows and new_pages (contiguous there)
  const uint64_t rows_off = sf::align256(info.workspace_bytes);
  const int64_t rows_ints = (int64_t(info.num_combine) + (append ? num_single : 0)) * sf::kItemInts;
  const int64_t copy_ints = rows_ints + (append && desc->num_seqs > 0 ? int64_t(pages_bytes / 4) : 0);
  if ((st = grow_device(r, &r->workspace, &r->workspace_bytes, rows_off + uint64_t(copy_ints) * 4, main)) != SF_OK)
    return st;
  int32_t* work = const_cast<int32_t*>(pin.dev);
  const sf::RowCopy copy = {work + (sf::table_rows(info.num_workers) + info.num_work) * sf::kItemInts,
                            reinterpret_cast<int32_t*>(static_cast<char*>(r->workspace) + rows_off),
                            int32_t(copy_ints), append ? int32_t(info.num_combine) * sf::kItemInts : -1,
                            append && desc->num_seqs > 0 ? int32_t(rows_ints) : -1};
  const sf::RowCopy* cp = copy_ints > 0 ? &copy : nullptr;

  // 3. kernels on the caller's stream (the caller's events, if any, take the
  //    attention kernel's own start and end times)
  void* ev0 = extras ? extras->attn_start : nullptr;
  void* ev1 = extras ? extras->attn_end : nullptr;
  // From here on a launch may have been enqueued that reads the slot, so the
  // step counts (and is marked in its turn) whatever the launches return.
  if (append) {
    const char* wbase = reinterpret_cast<const char*>(work);
    st = sf::decode_attn_append_rows(desc, &info, work, q, extras->k_new, extras->v_new,
                                     reinterpret_cast<const int32_t*>(wbase + pages_off),
                                     reinterpret_cast<const int32_t*>(wbase + info.work_bytes), num_single,
                                     const_cast<void*>(k_pool), const_cast<void*>(v_pool),
                                     const_cast<int32_t*>(block_table), out, lse, r->workspace,
                                     r->workspace_bytes, stream, cp, ev0, ev1, shared);
  } else {
    st = sf::decode_attn_rows(desc, &info, work, q, k_pool, v_pool, fp8 ? extras->k_scale : nullptr,
                              fp8 ? extras->v_scale : nullptr, block_table, out, lse, r->workspace,
                              r->workspace_bytes, stream, cp, ev0, ev1, shared);
  }
  pin.used = true;
  pin.last_step = r->steps;
  r->last_stream = main;
  ++r->steps;
  if (r->steps - r->unmarked >= kMarkEvery && mark_steps(r) != SF_OK) {
    // Without the mark nothing orders a later rewrite of these slots after
    // the steps' reads: wait for the stream instead.
    (void)hipStreamSynchronize(main);
    for (auto& p : r->ring) p.used = false;
    r->unmarked = r->steps;
    if (st == SF_OK) st = SF_ERR_HIP;
  }
  return st;
}

// Extend attention, in memory that the caller lends: the pinned part is cut
// into slots that the plans go round, the device part is the workspace.
extern "C" sf_status sf_runner_extend(sf_runner* r, const sf_attn_desc* desc, const int32_t* seq_lens_host,
                                      const int32_t* q_lens_host, const void* q, const void* k_new,
                                      const void* v_new, void* k_pool, void* v_pool, const int32_t* block_table,
                                      float* out, float* lse, sf_runner_memory* memory, void* stream,
                                      sf_extend_info* info_out) {
  if (!r || !desc || !info_out || !memory) return SF_ERR_INVALID_ARG;
  if (desc->num_q_heads != r->shape.num_q_heads || desc->num_kv_heads != r->shape.num_kv_heads ||
      desc->head_dim != r->shape.head_dim || desc->page_size != r->shape.page_size)
    return SF_ERR_INVALID_ARG;
  if ((reinterpret_cast<uintptr_t>(memory->pinned) | reinterpret_cast<uintptr_t>(memory->device)) & 15u)
    return SF_ERR_INVALID_ARG;
  hipStream_t main = static_cast<hipStream_t>(stream);
  // Slots are reused by waiting for events on the host, which a graph's
  // replays would not: a capturing stream is left to sf_extend_attn.
  hipStreamCaptureStatus capturing = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(main, &capturing) != hipSuccess) return SF_ERR_HIP;
  if (capturing != hipStreamCaptureStatusNone) return SF_ERR_UNSUPPORTED;

  // Other memory than the last call's: nothing may still use either.
  const bool per_call = memory->device_per_call == 1;
  sf_status st = SF_OK;
  Lent& lent = r->lent;
  const uint64_t slot_bytes = memory->slots > 0 ? memory->pinned_bytes / memory->slots / 32 * 32 : 0;
  if (!per_call && (lent.device != memory->device || lent.device_bytes != memory->device_bytes)) {
    if ((st = wait_lent(lent)) != SF_OK) return st;
    lent.device = memory->device;
    lent.device_bytes = memory->device_bytes;
  }
  if (lent.pinned != memory->pinned || lent.slots != memory->slots || lent.slot_bytes != slot_bytes) {
    if ((st = wait_lent(lent)) != SF_OK) return st;
    if (memory->slots < 0 || memory->slots > kRing || (memory->pinned == nullptr) != (memory->slots == 0))
      return SF_ERR_INVALID_ARG;
    void* dev = nullptr;
    if (memory->pinned && hipHostGetDevicePointer(&dev, memory->pinned, 0) != hipSuccess) return SF_ERR_HIP;
    lent.pinned = memory->pinned;
    lent.pinned_dev = static_cast<const char*>(dev);
    lent.slots = memory->slots;
    lent.slot_bytes = slot_bytes;
    lent.next = 0;
  }
  const int slot = lent.slots > 0 ? lent.next % lent.slots : 0;
  if ((st = wait_slot(lent, slot)) != SF_OK) return st;

  const bool store = k_new != nullptr;
  sf::ExtendPlan plan;
  try {
    int32_t* work = reinterpret_cast<int32_t*>(static_cast<char*>(lent.pinned) + uint64_t(slot) * lent.slot_bytes);
    st = sf::extend_plan_parts(desc, seq_lens_host, q_lens_host, r->opts.num_cus, store, work, lent.slot_bytes,
                               &plan, info_out);
  } catch (const std::bad_alloc&) {
    return SF_ERR_HIP;
  }
  if (st != SF_OK && st != SF_ERR_CAPACITY) return st;
  // Device memory: partial results, then the device copy of the part and
  // merge rows. The store launch makes that copy, or a launch of its own where
  // enough workgroups would otherwise read their row over PCIe.
  const uint64_t row_ints = (uint64_t(plan.num_parts) + plan.num_merge) * sf::kItemInts;
  if (row_ints > INT32_MAX) return SF_ERR_INVALID_ARG;
  const uint64_t lse_off = sf::align256(uint64_t(plan.num_slots) * plan.rows * desc->head_dim * 4);
  const uint64_t rows_off = lse_off + sf::align256(uint64_t(plan.num_slots) * plan.rows * 4);
  const bool copy = store || plan.num_parts > kExtendCopyParts;
  const uint64_t device_bytes = rows_off + (copy ? row_ints * 4 : 0);
  memory->need_slot = plan.bytes();
  memory->need_device = device_bytes;
  if (st == SF_ERR_CAPACITY || memory->device_bytes < device_bytes) return SF_ERR_CAPACITY;
  if (plan.num_parts == 0) return SF_OK;
  const int32_t* work_dev = reinterpret_cast<const int32_t*>(lent.pinned_dev + uint64_t(slot) * lent.slot_bytes);
  sf::ExtendArgs a;
  if ((st = sf::extend_args(desc, work_dev, q, k_new, v_new, k_pool, v_pool, block_table, out, lse, &a)) != SF_OK)
    return st;
  // Calls of another stream may still use the device memory: they are waited
  // for (calls on one stream are in order by themselves).
  if (main != lent.last_stream && lent.last_stream != kNoStream) {
    lent.streams = true;
    if ((st = wait_lent(lent)) != SF_OK) return st;
  }
  lent.last_stream = main;
  // The events skip HIP's system-scope fence, as the marks do.
  const bool mark = lent.streams || lent.unmarked + 1 >= lent.slots / 2;
  if (mark && !lent.done[slot] &&
      hipEventCreateWithFlags(&lent.done[slot], hipEventDisableTiming | hipEventDisableSystemFence) != hipSuccess) {
    lent.done[slot] = nullptr;
    return SF_ERR_HIP;
  }
  char* ws = static_cast<char*>(memory->device);
  a.parts = true;
  a.num_items = plan.num_parts;
  a.part_rows = plan.rows;
  a.part_o = reinterpret_cast<float*>(ws);
  a.part_lse = reinterpret_cast<float*>(ws + lse_off);
  a.num_merge = plan.num_merge;
  a.num_store = plan.num_store;
  a.store_rows = work_dev + row_ints;
  if (copy) {
    a.copy_src = work_dev;
    a.copy_dst = reinterpret_cast<int32_t*>(ws + rows_off);
    a.copy_ints = int32_t(row_ints);
    a.items = a.copy_dst;
  }
  a.merge_rows = a.items + int64_t(plan.num_parts) * sf::kItemInts;
  if (sf::launch_extend(a, main, mark ? lent.done[slot] : nullptr) != hipSuccess) {
    // An earlier launch of the call may read the slot, with no event behind it.
    (void)hipStreamSynchronize(main);
    return SF_ERR_HIP;
  }
  lent.used[slot] = true;
  lent.event[slot] = -1;
  ++lent.unmarked;
  if (mark) {
    for (int i = 0; i < kRing; ++i)
      if (lent.used[i] && lent.event[i] < 0) lent.event[i] = slot;
    lent.unmarked = 0;
  }
  ++lent.next;
  return SF_OK;
}

namespace {

sf_status reserve(sf_runner* r, const sf::ReserveBytes& need, hipStream_t main) {
  sf_status st = grow_device(r, &r->workspace, &r->workspace_bytes, need.device, main);
  if (st != SF_OK) return st;
  const uint64_t slot = need.slot;
  bool small = false;
  for (auto& p : r->ring) small = small || p.bytes < slot;
  if (!small) return SF_OK;
  // The slots that are too small come from one allocation (32 of their own take
  // 30 us each), once no step in flight reads the old ones. A slot leaves an
  // arena only for more bytes than the arena's slots have, so where any slot is
  // too small, all of an earlier arena's are.
  if ((st = wait_all(r)) != SF_OK) return st;
  void* ptr = nullptr;
  void* dev = nullptr;
  if (hipHostMalloc(&ptr, slot * kRing, hipHostMallocDefault) != hipSuccess) return SF_ERR_HIP;
  if (hipHostGetDevicePointer(&dev, ptr, 0) != hipSuccess) {
    (void)hipHostFree(ptr);
    return SF_ERR_HIP;
  }
  for (int i = 0; i < kRing; ++i) {
    Pinned& p = r->ring[i];
    if (p.bytes >= slot) continue;
    if (p.ptr && !p.in_arena && hipHostFree(p.ptr) != hipSuccess) st = SF_ERR_HIP;
    p = Pinned{};
    p.ptr = reinterpret_cast<int32_t*>(static_cast<char*>(ptr) + slot * i);
    p.dev = reinterpret_cast<const int32_t*>(static_cast<const char*>(dev) + slot * i);
    p.bytes = slot;
    p.in_arena = true;
  }
  if (r->arena && hipHostFree(r->arena) != hipSuccess) st = SF_ERR_HIP;
  r->arena = ptr;
  return st;
}

}  // namespace

extern "C" sf_status sf_runner_reserve(sf_runner* r, uint64_t workspace_bytes, uint64_t work_bytes,
                                       int32_t max_num_seqs, void* stream) {
  if (!r || max_num_seqs < 0) return SF_ERR_INVALID_ARG;
  // A smaller batch, or a step of another kind, may be planned in another way
  // than the batch reserved for and take more than it.
  return reserve(r, sf::reserve_bytes(&r->shape, &r->opts, workspace_bytes, work_bytes, max_num_seqs, -1),
                 static_cast<hipStream_t>(stream));
}

extern "C" sf_status sf_runner_reserve_batch(sf_runner* r, const int32_t* seq_lens_host, int32_t num_seqs, void* stream) {
  if (!r || num_seqs < 0 || (num_seqs > 0 && !seq_lens_host)) return SF_ERR_INVALID_ARG;
  int64_t pages = 0;
  for (int32_t s = 0; s < num_seqs; ++s) {
    if (seq_lens_host[s] < 0) return SF_ERR_INVALID_ARG;
    pages += (int64_t(seq_lens_host[s]) + sf::kPage - 1) / sf::kPage;
  }
  // Room for the batch to grow: the bounds stop at the planner's workers soon.
  return reserve(r, sf::reserve_bytes(&r->shape, &r->opts, 0, 0, num_seqs, 2 * (pages + num_seqs) * r->shape.num_kv_heads),
                 static_cast<hipStream_t>(stream));
}
