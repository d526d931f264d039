// C ABI of libdbsp: argument checks, plan life cycle, device upload, kernel launches.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <new>
#include <string>
#include <thread>
#include <type_traits>
#include <vector>

#include "dbsp.h"
#include "dbsp_diag.h"
#include "fwd_params.hpp"
#include "plan.hpp"

namespace {
thread_local std::string g_err;
}

int dbsp_set_error(int code, const std::string& msg) {
  g_err = msg;
  return code;
}

namespace {

int fail(int code, const std::string& msg) { return dbsp_set_error(code, msg); }

int fail_hip(hipError_t e, const char* what) {
  g_err = std::string(what) + ": " + hipGetErrorString(e);
  (void)hipGetLastError();  // clear the sticky error so that later calls report their own
  return DBSP_EHIP;
}

#define DBSP_HIP(call)                                  \
  do {                                                  \
    hipError_t e_ = (call);                             \
    if (e_ != hipSuccess) return fail_hip(e_, #call);   \
  } while (0)

constexpr int kMaxWaves = 8;     // waves of the largest workgroup: a split row has a counter for each

// ---- process-wide resources: upload stream, device and pinned-host buffer pools -------------
// Plans are created and destroyed per attention call when masks are dynamic, so their buffers are
// recycled instead of going through hipMalloc / hipFree (which synchronises the device) each time.
// Entries remember the device that was current when they were allocated and only go back to it.
// The buffers of a released plan that the GPU still uses are retired together with the plan's events
// and join the pools once those have passed: releasing a plan does not wait, unless the calling thread has
// kMaxRetired retired plans on the device already: then for the oldest of these.  So a caller that plans every
// step stays that many steps ahead of the GPU, which hides the planning, and the pools can hold all the buffers
// in flight; a host further ahead would gain nothing and allocate (40 heads, 256 x 256 blocks, 5 to 60 % of them active: 350 us more per step of 5840 with 16 let ahead and pools of 8).
struct BufferPool {
  struct Entry {
    void* ptr;
    size_t bytes;
    int device;
    bool front_zero;               // device buffers: the first kFrontBytes are zero, see forward()
  };
  size_t max_cached;
  std::vector<Entry> free_list;
};
struct Retired {
  std::thread::id by;
  hipEvent_t events[2];            // last use, upload; null = nothing to wait for
  BufferPool::Entry dev, pin[2];
};

constexpr int kMaxDevices = 64;
constexpr size_t kMaxRetired = 3;
std::mutex g_mu;
hipStream_t g_upload_stream[kMaxDevices] = {};
BufferPool g_dev_pool{8, {}}, g_pin_pool{16, {}};      // one and two buffers a plan
std::vector<Retired> g_retired;

// g_mu is held.  Surplus buffers go to `surplus` (to be freed without the lock: freeing synchronises).
struct Surplus { std::vector<void*> dev, pin; };
void pool_put(BufferPool& pool, const BufferPool::Entry& e, std::vector<void*>& surplus) {
  if (!e.ptr) return;
  pool.free_list.push_back(e);
  if (pool.free_list.size() > pool.max_cached) {
    size_t smallest = 0;
    for (size_t i = 1; i < pool.free_list.size(); ++i)
      if (pool.free_list[i].bytes < pool.free_list[smallest].bytes) smallest = i;
    surplus.push_back(pool.free_list[smallest].ptr);
    pool.free_list.erase(pool.free_list.begin() + smallest);
  }
}

// Asking for an event's state, waiting for it and freeing buffers are no part of any capture: they neither fail in
// nor spoil one that is under way.
struct OutsideCapture {
  hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
  OutsideCapture() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
  ~OutsideCapture() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
};

// g_mu is held.
void recycle(const Retired& r, Surplus& surplus) {
  for (hipEvent_t ev : r.events)
    if (ev) (void)hipEventDestroy(ev);
  pool_put(g_dev_pool, r.dev, surplus.dev);
  for (const BufferPool::Entry& e : r.pin) pool_put(g_pin_pool, e, surplus.pin);
}

// g_mu is held.  Recycles what the GPU is known to be done with: any answer but success leaves a plan retired.
void reap(Surplus& surplus) {
  if (g_retired.empty()) return;
  OutsideCapture relaxed;
  for (size_t i = 0; i < g_retired.size();) {
    bool done = true;
    for (hipEvent_t ev : g_retired[i].events) done = done && (!ev || hipEventQuery(ev) == hipSuccess);
    if (!done) { ++i; continue; }
    recycle(g_retired[i], surplus);
    g_retired.erase(g_retired.begin() + i);
  }
  (void)hipGetLastError();         // a query's "not ready" is no error
}

void release(const Surplus& surplus) {
  if (surplus.dev.empty() && surplus.pin.empty()) return;
  OutsideCapture relaxed;
  for (void* p : surplus.dev) (void)hipFree(p);
  for (void* p : surplus.pin) (void)hipHostFree(p);
}

hipError_t pool_get(BufferPool& pool, bool pinned, int device, size_t bytes, void** out, size_t* cap, bool* front_zero = nullptr) {
  Surplus surplus;
  bool found = false;
  {
    std::lock_guard<std::mutex> lk(g_mu);
    reap(surplus);
    int best = -1;
    for (size_t i = 0; i < pool.free_list.size(); ++i)
      if (pool.free_list[i].device == device && pool.free_list[i].bytes >= bytes &&
          (best < 0 || pool.free_list[i].bytes < pool.free_list[best].bytes))
        best = (int)i;
    if (best >= 0) {
      *out = pool.free_list[best].ptr;
      *cap = pool.free_list[best].bytes;
      if (front_zero) *front_zero = pool.free_list[best].front_zero;
      pool.free_list.erase(pool.free_list.begin() + best);
      found = true;
    }
  }
  release(surplus);
  if (found) return hipSuccess;
  const size_t rounded = (bytes + (size_t(1) << 20) - 1) & ~((size_t(1) << 20) - 1);   // 1 MiB granules
  hipError_t e = pinned ? hipHostMalloc(out, rounded, hipHostMallocDefault) : hipMalloc(out, rounded);
  *cap = rounded;
  return e;
}

// One upload stream per device (created on first use, with that device current).
hipError_t upload_stream(int device, hipStream_t* out) {
  if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lk(g_mu);
  if (!g_upload_stream[device]) {
    hipError_t e = hipStreamCreateWithFlags(&g_upload_stream[device], hipStreamNonBlocking);
    if (e != hipSuccess) return e;
  }
  *out = g_upload_stream[device];
  return hipSuccess;
}

// Hands the plan's buffers back once its events have passed: waits for them, or leaves them to later calls.
void free_device(dbsp_device_plan& d, bool wait) {
  Retired r = {std::this_thread::get_id(), {nullptr, nullptr}, {d.blob, d.blob_bytes, d.device, d.sent || d.front_zero},
               {{d.staging, d.staging_bytes, d.device, false}, {d.staging_kv, d.staging_kv_bytes, d.device, false}}};
  if (d.last_use) {
    if (d.used) r.events[0] = static_cast<hipEvent_t>(d.last_use);
    else (void)hipEventDestroy(static_cast<hipEvent_t>(d.last_use));
  }
  if (d.uploaded) {
    if (d.sent) r.events[1] = static_cast<hipEvent_t>(d.uploaded);
    else (void)hipEventDestroy(static_cast<hipEvent_t>(d.uploaded));
  }
  Surplus surplus;
  if (!wait) {
    std::lock_guard<std::mutex> lk(g_mu);
    g_retired.push_back(r);
    reap(surplus);
    size_t mine = 0, oldest = 0;
    for (size_t i = g_retired.size(); i-- > 0;)
      if (g_retired[i].by == r.by && g_retired[i].dev.device == d.device) { ++mine; oldest = i; }
    if (mine > kMaxRetired) {
      r = g_retired[oldest];       // waited for without the lock: others go on planning
      g_retired.erase(g_retired.begin() + oldest);
      wait = true;
    }
  }
  if (wait) {
    OutsideCapture relaxed;
    bool done = true;
    for (hipEvent_t ev : r.events) done = done && (!ev || hipEventSynchronize(ev) == hipSuccess);
    std::lock_guard<std::mutex> lk(g_mu);
    if (done) recycle(r, surplus);
    else g_retired.push_back(r);   // the GPU may still use its buffers
  }
  release(surplus);
  (void)hipGetLastError();
  d = dbsp_device_plan();
}

// Pinned memory for the index lists (the plan's kv_ints() + 8 int32): the compaction writes straight into it, it is
// the source of the upload and the plan's host copy of the lists.
int get_kv_staging(dbsp_plan* plan) {
  dbsp_device_plan& dv = plan->dev;
  DBSP_HIP(hipGetDevice(&dv.device));
  const size_t bytes = ((size_t)plan->host.kv_ints() + 8) * sizeof(int32_t);
  hipError_t e = pool_get(g_pin_pool, true, dv.device, bytes, &dv.staging_kv, &dv.staging_kv_bytes);
  if (e != hipSuccess) { (void)hipGetLastError(); return fail(DBSP_ENOMEM, std::string("plan staging buffer: ") + hipGetErrorString(e)); }
  return DBSP_OK;
}

constexpr size_t kFrontBytes = size_t(4) << 10;      // of every plan's device buffer: counters, zero between launches

// Sends the plan to the device on the library's upload stream, asynchronously, with one event that forward
// launches wait for: the small arrays from their staging buffer, the index lists from theirs.  Behind a first launch
// that reads them where they are staged, which may still run, the arrays only: what it counts and measures lies in
// front of and behind them, and nothing would order the staged zeros with that.
int send_upload(dbsp_device_plan& dv) {
  hipStream_t us;
  DBSP_HIP(upload_stream(dv.device, &us));
  const size_t from = dv.used ? kFrontBytes : 0, to = dv.used ? dv.arrays_end : dv.up_bytes;
  DBSP_HIP(hipMemcpyAsync(dv.blob + from, static_cast<const unsigned char*>(dv.staging) + from, to - from, hipMemcpyHostToDevice, us));
  if (dv.kv_bytes) DBSP_HIP(hipMemcpyAsync(dv.blob + dv.up_bytes, dv.staging_kv, dv.kv_bytes, hipMemcpyHostToDevice, us));
  DBSP_HIP(hipEventRecord(static_cast<hipEvent_t>(dv.uploaded), us));
  dv.sent = true;
  return DBSP_OK;
}

// Lays the plan out for the device and sends it; the host does not wait.  A plan of up to kInStreamBytes is
// not sent here: its first forward launch is preceded, on its own stream, by a kernel that fetches the
// plan from the pinned buffers (64 KiB take it about 3 us).  Two streams and the wait between them cost the
// host 12 us and more; for larger plans they let the copy run beside the kernels before it.
constexpr size_t kInStreamBytes = (size_t(64) << 10) + kFrontBytes;

__global__ __launch_bounds__(256) void dbsp_fetch_kernel(uint4* __restrict__ dst, const uint4* __restrict__ a, uint32_t na, const uint4* __restrict__ b, uint32_t n) {
  for (uint32_t i = blockIdx.x * 256 + threadIdx.x; i < n; i += gridDim.x * 256) dst[i] = i < na ? a[i] : b[i - na];
}

// The record behind the launch that follows vouches for the fetch as well (see forward).
int fetch_in_stream(dbsp_device_plan& dv, hipStream_t st) {
  // the index lists' last 16 bytes may reach into the slack both buffers have behind them
  const uint32_t na = (uint32_t)(dv.up_bytes / 16), n = na + (uint32_t)((dv.kv_bytes + 15) / 16);
  hipLaunchKernelGGL(dbsp_fetch_kernel, dim3((n + 255) / 256), dim3(256), 0, st,
                        reinterpret_cast<uint4*>(dv.blob), static_cast<const uint4*>(dv.staging), na, static_cast<const uint4*>(dv.staging_kv), n);
  DBSP_HIP(hipGetLastError());
  dv.sent = true;
  return DBSP_OK;
}

// Whose items the workgroups of a launch run, and in what order.
struct RunOrder {
  int32_t parts = 0, run_log2 = 0;         // workgroup b has partition dbsp_part_of(b, parts, run_log2)
  int32_t groups = 0, longest_list = 0;    // workgroups up to the last one that has items, items the longest list has
  bool own = false;                        // by the lists below instead of the placement's own
  bool local = false;                      // see dbsp_fwd_params
  std::vector<int32_t> ptr, run;           // [P + 1] where the workgroups' lists begin, and the lists
};

// The lists.  Of a greedy placement a workgroup has its partition's items, the longest first, equal ones by their id.  The
// greedy deals items in that order, one to every partition before anybody gets a second one: run so, all partitions are at
// items of about the same length at the same time, that is of the few heads whose rows are about that long, and find each
// other's KV blocks in the L2.  In the lists' own order (head by head) they drift apart by as many heads as a partition has
// items more or fewer of them than the mean.
// (Lists are short where a partition gets few items, and sorted one by one then, else all at once by counting: 2406 items on
// 1024 partitions, a step of 77 us, took 12 us more by counting.)
constexpr int32_t kShortList = 8;
void order_lists(const dbsp_host_plan& hp, bool sorted, RunOrder& o) {
  const int32_t n = (int32_t)hp.part_items.size();          // every item: a greedy placement has no queue
  o.ptr.resize((size_t)hp.P + 1);
  o.run.resize(n);
  o.ptr[0] = 0;
  auto weight = [&](int32_t i) { return hp.items[4 * (size_t)i + 3] - hp.items[4 * (size_t)i + 2]; };
  if (!sorted || o.longest_list <= kShortList) {
    int32_t* to = o.run.data();
    for (int32_t b = 0; b < hp.P; ++b) {
      const int32_t g = dbsp_part_of(b, o.parts, o.run_log2);
      int32_t w[kShortList], m = 0;
      for (int32_t k = hp.part_ptr[g]; k < hp.part_ptr[g + 1]; ++k, ++m) {
        const int32_t i = hp.part_items[k];
        int32_t at = m;
        if (sorted) {
          const int32_t wi = weight(i);
          for (; at > 0 && w[at - 1] < wi; --at) {
            w[at] = w[at - 1];
            to[at] = to[at - 1];
          }
          w[at] = wi;
        }
        to[at] = i;
      }
      to += m;
      o.ptr[b + 1] = o.ptr[b] + m;
    }
    return;
  }
  std::vector<int32_t> next(hp.P);            // of every partition: where its next item goes
  for (int32_t b = 0; b < hp.P; ++b) {
    const int32_t g = dbsp_part_of(b, o.parts, o.run_log2);
    next[g] = o.ptr[b];
    o.ptr[b + 1] = o.ptr[b] + hp.part_ptr[g + 1] - hp.part_ptr[g];
  }
  int32_t longest = 0;
  for (int32_t i = 0; i < n; ++i) longest = std::max(longest, weight(i));
  std::vector<int32_t> first((size_t)longest + 2, 0), part_of(n), by_weight(n);
  for (int32_t g = 0; g < hp.P; ++g)
    for (int32_t k = hp.part_ptr[g]; k < hp.part_ptr[g + 1]; ++k) part_of[hp.part_items[k]] = g;
  for (int32_t i = 0; i < n; ++i) ++first[longest - weight(i) + 1];
  for (int32_t w = 0; w <= longest; ++w) first[w + 1] += first[w];
  for (int32_t i = 0; i < n; ++i) by_weight[first[longest - weight(i)]++] = i;
  for (int32_t i : by_weight) o.run[next[part_of[i]]++] = i;
}

// Which partitions share an L2 (see dbsp_part_of).  Workgroup b runs on compute die b mod 8, and the greedy hands neighbouring
// items, of one head mostly, to neighbouring partitions, as many in a row as have the same load so far: of its placements
// every die runs 2^result partitions in a row, an eighth of all where it can.  Partitions differ in load where each has few
// items (970 rows of 97 blocks on 256: four or three), and then the ones with more lie together: no run is so long that
// some die gets 3 % more blocks than the mean (those rows, in runs of 1 / 16 / 32: 667 / 692 / 691 us).
// Both together, us a pass before / the order alone / runs alone / both, in turn, defaults: 30 heads, 137 x 137 blocks of 128 at
// d = 64, B = 2 1571 / 1552 / 1527 / 1511; 12 heads, 21 x 23 at d = 128 59.5 / 60.0 / 55.4 / 55.2; 40 heads, 256 x 256 6940 /
// 6645 / 6531 / 6201; 16 heads, 513 x 513, 22 a row 1501 / 1546 / 1419 / 1420; 48 heads, 275 x 275 blocks of 64 at d = 64
// 1926 / 1767 / 1713 / 1488, 24 heads, 301 x 301 at d = 128 2127 / 1827 / 1962 / 1774.
// Runs of 2, 4, 8, 16 of the 256 partitions instead of 32, 40 heads, 256 x 256: 6668, 6518, 6506, 6495 / 6474.
constexpr int kDies = 8;
int longest_runs_log2(int32_t parts) {
  if (parts < 64) return 0;             // a handful of workgroups has an L2 almost to itself
  int lg = 0;
  while ((int64_t)kDies << (lg + 1) <= parts) ++lg;
  return lg;
}
int die_run_log2(const dbsp_host_plan& hp, int32_t parts) {
  int lg = longest_runs_log2(parts);
  if (lg == 0) return 0;
  std::vector<int64_t> before((size_t)parts + 1, 0);      // blocks of the partitions in front of each
  for (int32_t g = 0; g < parts; ++g) before[g + 1] = before[g] + hp.part_load[g];
  for (; lg > 0; --lg) {
    int64_t load[kDies] = {};
    const int32_t runs = parts >> (lg + 3) << 3;      // (the others are dealt one by one)
    for (int32_t k = 0; k < runs; ++k) load[k % kDies] += before[(size_t)(k + 1) << lg] - before[(size_t)k << lg];
    for (int32_t g = runs << lg; g < parts; ++g) load[g % kDies] += hp.part_load[g];
    if (100 * kDies * *std::max_element(load, load + kDies) <= 103 * before[parts]) break;
  }
  return lg;
}

constexpr int32_t kMostOfTheChip = 224;      // workgroups, see dbsp_launch_fwd
RunOrder run_order(const dbsp_host_plan& hp) {
  RunOrder o;
  for (int32_t g = 0; g < hp.P; ++g) {
    const int32_t n = hp.part_ptr[g + 1] - hp.part_ptr[g];
    o.longest_list = std::max(o.longest_list, n);
    if (n) o.groups = g + 1;
  }
  // Not for short items, of fewer than four blocks of 128 tokens or sixteen of 64 in the mean.  us a pass listed / ordered of a kept plan,
  // then planned on every call: 128 tokens at d = 128, 3.1 blocks an item 502 / 560, 511 / 568, 3.8 124 / 130, 128 / 136, 4.8
  // 208 / 208, 213 / 214, 5.1 (12 heads, 21 x 23) 60 / 55; at d = 64 3.8 83 / 85, 111 / 118, 4.8 134 / 134, 141 / 143; pair rows, 2.9
  // 129 / 123, 151 / 165, 4.1 196 / 186, 202 / 195.  With 64 tokens the kernel gains earlier, but the host, which has more
  // items for the same work, loses it where it plans on every call: d = 64, 6.1 64 / 59, 117 / 129, 9.4 79 / 68, 113 / 122, 15.9
  // 181 / 151, 190 / 172; at d = 128 8.4 100 / 91, 109 / 113, 12.7 137 / 118, 142 / 127.  A plan does not know how often it will be used.
  const bool worth = hp.by_greedy && hp.nnz * hp.tile_rows() * hp.tile_rows() >= 65536 * hp.n_items();
  o.parts = o.groups;
  if (hp.by_greedy && hp.by_cost && o.longest_list > 1) {
    // costs are a compute unit's: which one runs a partition must not depend on the mask that they are used for (nor on the
    // one they were measured with, see dbsp_plan_calibrate), so the runs are those of the number of partitions.  us a pass
    // with a plan's own costs, by runs that go with the loads / these: 48 heads, 275 x 275 blocks of 64 at d = 64 1932 / 1640, 24 heads,
    // 301 x 301 at d = 128 2050 / 1833, 40 heads, 256 x 256 of 128 6265 / 6216, 12 heads, 21 x 23 57.6 / 52.9; in short items 48
    // heads, 256 x 256 512 / 508, 11 heads, 212 x 212 blocks of 64 61.5 / 58.9.  (Of an item at most a workgroup, costs settle
    // nothing, and with fewer items than partitions these runs would keep to the first dies.)
    o.parts = hp.P;
    o.run_log2 = longest_runs_log2(hp.P);
  } else if (worth) {
    o.run_log2 = die_run_log2(hp, o.groups);
  }
  o.own = (worth && o.longest_list > 1) || o.run_log2 > 0;
  if (o.own) {
    order_lists(hp, worth, o);
    while (o.groups < hp.P && o.ptr[o.groups] < o.ptr[hp.P]) ++o.groups;
  }
  o.local = hp.by_rounds || (hp.by_greedy && (o.longest_list > 1 || o.groups < kMostOfTheChip));
  return o;
}

int upload(dbsp_plan* plan) {
  dbsp_host_plan& hp = plan->host;
  dbsp_device_plan& dv = plan->dev;
  // what a workgroup needs to know of an item, in the order the workgroups run them (then the shared
  // queue's): one load instead of a chain through list, item, slot and row offset
  const int64_t n_placed = (int64_t)hp.part_items.size(), n_sched = n_placed + (int64_t)hp.tail_items.size();
  std::vector<int32_t> slot_row(hp.n_slots);
  const size_t n_split = hp.split_rows.size() / 4;
  for (size_t r = 0; r < n_split; ++r)
    for (int32_t k = 0; k < hp.split_rows[4 * r + 2]; ++k) slot_row[hp.split_rows[4 * r + 1] + k] = (int32_t)r;
  const RunOrder order = run_order(hp);
  dv.groups = order.groups;
  dv.run_parts = order.parts;
  dv.run_log2 = order.run_log2;
  dv.local = order.local;
  const std::vector<int32_t>& part_ptr = order.own ? order.ptr : hp.part_ptr;
  const std::vector<int32_t>& run = order.own ? order.run : hp.part_items;
  for (size_t r = 0; r < n_split; ++r) dv.max_chunks = std::max(dv.max_chunks, hp.split_rows[4 * r + 2]);
  const std::vector<int32_t>* arrays[] = {&hp.empty_rows, &part_ptr, nullptr, &hp.split_rows};      // (the schedule is made in place)
  constexpr int NA = 4;
  const auto ints_of = [&](int i) { return arrays[i] ? arrays[i]->size() : 8 * (size_t)n_sched; };
  size_t off[NA + 1];   // in int32 units, each array 16-byte aligned
  off[0] = kFrontBytes / sizeof(int32_t);
  for (int i = 0; i < NA; ++i) off[i + 1] = off[i] + ((ints_of(i) + 3) & ~size_t(3));
  const size_t ints_bytes = off[NA] * sizeof(int32_t);
  const size_t busy_off = dv.arrays_end = (ints_bytes + 255) & ~size_t(255);
  const size_t hw_off = busy_off + (((size_t)hp.P * sizeof(uint64_t) + 255) & ~size_t(255));
  // shared queue of the dynamic tail: [0] next position, then one take count per tail item; then the split rows' counters
  // where the front does not hold them
  const size_t queue_off = hw_off + (((size_t)hp.P * sizeof(uint32_t) + 255) & ~size_t(255));
  const size_t cnt_off = queue_off + (((1 + hp.tail_items.size()) * sizeof(uint32_t) + 255) & ~size_t(255));
  const size_t cnt_bytes = (size_t)dv.max_batch * n_split * kMaxWaves * sizeof(uint32_t);
  const bool cnt_in_front = cnt_bytes <= kFrontBytes;
  dv.up_bytes = cnt_off + (cnt_in_front ? 0 : (cnt_bytes + 255) & ~size_t(255));   // staged part ends here
  const size_t up_bytes = dv.up_bytes, kv_off = up_bytes;
  const size_t kv_bytes = dv.kv_bytes = (size_t)hp.kv_ints() * sizeof(int32_t);
  // split-row scratch for max_batch batch entries at d = 128
  const int64_t rows = (int64_t)dv.max_batch * hp.n_slots * hp.tile_rows();
  const size_t lse_off = (kv_off + kv_bytes + 255) & ~size_t(255);
  const size_t po_off = lse_off + (((size_t)rows * sizeof(float) + 255) & ~size_t(255));
  const size_t total = po_off + (size_t)rows * 128 * sizeof(float);

  void* blob = nullptr;
  hipError_t e = pool_get(g_dev_pool, false, dv.device, total, &blob, &dv.blob_bytes, &dv.front_zero);
  if (e != hipSuccess) { (void)hipGetLastError(); return fail(DBSP_ENOMEM, std::string("plan device buffer: ") + hipGetErrorString(e)); }
  dv.blob = static_cast<unsigned char*>(blob);
  e = pool_get(g_pin_pool, true, dv.device, up_bytes, &dv.staging, &dv.staging_bytes);
  if (e != hipSuccess) { (void)hipGetLastError(); return fail(DBSP_ENOMEM, std::string("plan staging buffer: ") + hipGetErrorString(e)); }

  unsigned char* st = static_cast<unsigned char*>(dv.staging);
  for (int i = 0; i < NA; ++i)
    if (arrays[i] && !arrays[i]->empty()) std::memcpy(st + off[i] * sizeof(int32_t), arrays[i]->data(), arrays[i]->size() * sizeof(int32_t));
  int32_t* sched = reinterpret_cast<int32_t*>(st) + off[2];
  for (int64_t k = 0; k < n_sched; ++k) {
    const int64_t i = k < n_placed ? run[k] : hp.tail_items[k - n_placed];
    const int32_t* it = hp.items.data() + 4 * i;
    int32_t* s = sched + 8 * k;
    s[0] = it[0];                                                                                  // head
    s[1] = it[1];                                                                                  // row of the plan (query block, or pair of them)
    s[2] = (hp.row_ptr[(int64_t)it[0] * hp.nQ + it[1]] + it[2]) * (hp.pair ? 2 : 1);               // first word of its KV list
    s[3] = it[3] - it[2];                                                                          // blocks (super blocks)
    s[4] = hp.item_slot[i];
    s[5] = s[6] = s[7] = 0;
    if (s[4] >= 0) {
      const int32_t r = slot_row[s[4]];
      s[5] = r; s[6] = hp.split_rows[4 * (size_t)r + 2]; s[7] = hp.split_rows[4 * (size_t)r + 1];  // index of the split row, its chunks, its first slot
    }
  }
  std::memset(st, 0, kFrontBytes);
  std::memset(st + busy_off, 0, up_bytes - busy_off);   // busy ticks, hardware ids, the queue's counters start at zero

  hipEvent_t ev_up, ev_use;
  DBSP_HIP(hipEventCreateWithFlags(&ev_up, hipEventDisableTiming));
  dv.uploaded = ev_up;
  DBSP_HIP(hipEventCreateWithFlags(&ev_use, hipEventDisableTiming));
  dv.last_use = ev_use;
  if (up_bytes + kv_bytes > kInStreamBytes) {
    const int rc = send_upload(dv);
    if (rc != DBSP_OK) return rc;
  }

  // A launch of at most an item a workgroup, with nothing to count but what the front holds, rows merged in place: see forward()
  dv.direct = dv.front_zero && cnt_in_front && order.longest_list <= 1 && hp.tail_items.empty() && kMaxTilesPerWave * dv.max_chunks <= kTilesInPlace &&
              up_bytes + kv_bytes <= kInStreamBytes;
  for (int i = 0; i < NA; ++i) dv.array_off[i] = off[i];
  const int32_t* ints = reinterpret_cast<const int32_t*>(dv.blob);
  dv.empty_rows = ints + off[0];
  dv.part_ptr = ints + off[1];
  dv.sched = ints + off[2];
  dv.split_rows = ints + off[3];
  dv.queue = reinterpret_cast<uint32_t*>(dv.blob + queue_off);
  dv.split_cnt = reinterpret_cast<uint32_t*>(dv.blob + (cnt_in_front ? 0 : cnt_off));
  dv.kv_idx = reinterpret_cast<const int32_t*>(dv.blob + kv_off);
  dv.busy = reinterpret_cast<uint64_t*>(dv.blob + busy_off);
  dv.hw_id = reinterpret_cast<uint32_t*>(dv.blob + hw_off);
  dv.part_lse = reinterpret_cast<float*>(dv.blob + lse_off);
  dv.part_o = reinterpret_cast<float*>(dv.blob + po_off);
  dv.resident = true;
  return DBSP_OK;
}

// ---- scratch for callers that cannot allocate ------------------------------------------------
// The split-row partials of sparse_attn_fwd_static go here instead of into the plan's buffer.
// One copy of the array exists per GPU the library runs on, for the life of the process; every
// call on a GPU shares it.  In host code the array's name is only a handle for
// hipGetSymbolAddress: the device address is looked up once per device and used from then on.
constexpr size_t kStaticScratchBytes = size_t(32) << 20;   // 32 MiB
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

unsigned char* g_scratch_ptr[kMaxDevices] = {};

// Device address of this device's copy of `scratch` (the device must be current).
int static_scratch(int device, unsigned char** out) {
  if (device < 0 || device >= kMaxDevices) return fail(DBSP_EINVAL, "sparse_attn_fwd_static: device index out of range");
  std::lock_guard<std::mutex> lk(g_mu);
  if (!g_scratch_ptr[device]) {
    void* ptr = nullptr;
    hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return fail_hip(e, "hipGetSymbolAddress(scratch)");
    if (!ptr) return fail(DBSP_EHIP, "sparse_attn_fwd_static: the static scratch has no device address");
    g_scratch_ptr[device] = static_cast<unsigned char*>(ptr);
  }
  *out = g_scratch_ptr[device];
  return DBSP_OK;
}

}  // namespace

extern "C" {

const char* dbsp_last_error(void) { return g_err.c_str(); }

static int make_plan(const uint8_t* mask_host, int32_t H, int32_t nQ, int32_t nK, int32_t block,
                     const dbsp_plan_opts* opts, const dbsp_plan* previous, double reuse_threshold,
                     dbsp_plan** out_plan, const char* who) {
  const auto t_start = std::chrono::steady_clock::now();
  if (out_plan) *out_plan = nullptr;
  if (!mask_host || !out_plan) return fail(DBSP_EINVAL, std::string(who) + ": null pointer");
  if (H <= 0 || nQ <= 0 || nK <= 0 || block <= 0) return fail(DBSP_EINVAL, std::string(who) + ": H, nQ, nK and block must be positive");
  if ((int64_t)H * nQ >= INT32_MAX) return fail(DBSP_EINVAL, std::string(who) + ": too many rows");
  dbsp_plan_opts o;
  std::memset(&o, 0, sizeof(o));
  if (opts) o = *opts;
  if (o.num_partitions < 0 || o.item_overhead < 0 ||
      (o.mode != DBSP_MODE_BALANCED && o.mode != DBSP_MODE_NAIVE && o.mode != DBSP_MODE_ROUNDS && o.mode != DBSP_MODE_REWARD) ||
      (o.flags & ~(DBSP_PLAN_HOST_ONLY | DBSP_PLAN_PAIR_ROWS | DBSP_PLAN_PAIR_AUTO)) || o.locality_groups < 0 || o.max_batch < 0)
    return fail(DBSP_EINVAL, std::string(who) + ": bad option (partitions < 0, overhead < 0, groups < 0, max_batch < 0, unknown mode or flag)");
  if (o.dynamic_tail < 0 || o.dynamic_tail >= 1000 || (o.dynamic_tail > 0 && o.mode != DBSP_MODE_ROUNDS))
    return fail(DBSP_EINVAL, std::string(who) + ": dynamic_tail is a permille in [0, 1000) and goes with DBSP_MODE_ROUNDS only");
  if (!(o.reward >= 0.0) || (o.reward != 0.0 && o.mode != DBSP_MODE_REWARD) || (o.mode == DBSP_MODE_REWARD && o.partition_cost))
    return fail(DBSP_EINVAL, std::string(who) + ": reward must be >= 0, goes with DBSP_MODE_REWARD only, and that mode takes no partition_cost");
  if (o.head_dim != 0 && o.head_dim != 64 && o.head_dim != 128)
    return fail(DBSP_EINVAL, std::string(who) + ": head_dim is 0 (unknown), 64 or 128");
  const bool host_only = (o.flags & DBSP_PLAN_HOST_ONLY) != 0;
  bool pair = (o.flags & DBSP_PLAN_PAIR_ROWS) != 0;
  const bool pair_auto = (o.flags & DBSP_PLAN_PAIR_AUTO) != 0;
  if (pair && pair_auto) return fail(DBSP_EINVAL, std::string(who) + ": DBSP_PLAN_PAIR_ROWS and DBSP_PLAN_PAIR_AUTO exclude each other");
  if ((pair || pair_auto) && block != 64) return fail(DBSP_EINVAL, std::string(who) + ": pair rows go with 64-token blocks");
  if (pair_auto && o.head_dim != 128) return fail(DBSP_EINVAL, std::string(who) + ": DBSP_PLAN_PAIR_AUTO needs head_dim = 128 (pair rows run at that head dim only)");
  // DBSP_PLAN_PAIR_AUTO: a chain of plans keeps the first one's choice (items of the two kinds do not
  // match each other); else both counts are taken and pair rows chosen from a flag fill of 5 / 8
  // (2 x the mask's active blocks >= 5 x the super blocks): what the header promises.  It was the break-even while
  // the kernel of single 64-token rows ran at 0.29 of the peak; at 0.40 to 0.45 that lies near 0.87 (40 heads,
  // 512 x 512 blocks, single / pair rows: fill 1.00 5.98 / 5.38 ms, 0.80 4.69 / 5.00, 0.66 3.36 / 4.05)
  dbsp_host_plan counted;
  bool have_counts = false;
  if (pair_auto) {
    if (previous) {
      pair = previous->host.pair;
    } else {
      std::string cerr;
      dbsp_host_plan plain;
      int rc = dbsp_plan_count(mask_host, H, nQ, nK, block, true, counted, cerr);
      if (rc == DBSP_OK) rc = dbsp_plan_count(mask_host, H, nQ, nK, block, false, plain, cerr);
      if (rc != DBSP_OK) return fail(rc, std::string(who) + ": " + cerr);
      pair = 2 * plain.nnz >= 5 * counted.nnz;
      if (!pair) counted = std::move(plain);
      have_counts = true;
    }
  }
  if (previous && previous->host.pair != pair) return fail(DBSP_ESHAPE, std::string(who) + ": the previous plan differs in DBSP_PLAN_PAIR_ROWS");
  int32_t P = o.num_partitions;
  if (P == 0 && previous) P = previous->host.P;
  if (P == 0) {
    P = 256;
    if (!host_only) {
      int dev = 0;
      hipDeviceProp_t prop;
      if (hipGetDevice(&dev) == hipSuccess && hipGetDeviceProperties(&prop, dev) == hipSuccess && prop.multiProcessorCount > 0)
        P = prop.multiProcessorCount;
      else
        (void)hipGetLastError();
    }
    // a 64-token block is served by a two-wave workgroup: at d = 64 four of them fill a compute unit (also
    // where the plan does not know d), at d = 128 two; pair rows take the workgroup of 128-token blocks, one per compute unit
    if (block <= 64 && !pair) P *= (o.head_dim == 128 ? 2 : 4);
  }
  if (previous && (previous->host.H != H || previous->host.nQ_blocks != nQ || previous->host.nK != nK || previous->host.P != P))
    return fail(DBSP_ESHAPE, std::string(who) + ": the previous plan has a different geometry or partition count");
  if (o.locality_groups > 1 && P % o.locality_groups != 0)
    return fail(DBSP_EINVAL, std::string(who) + ": locality_groups must divide the number of partitions");
  if (o.partition_cost)
    for (int32_t g = 0; g < P; ++g)
      if (o.partition_cost[g] <= 0) return fail(DBSP_EINVAL, std::string(who) + ": partition_cost must be positive");
  dbsp_plan* plan = new (std::nothrow) dbsp_plan();
  if (!plan) return fail(DBSP_ENOMEM, std::string(who) + ": out of host memory");
  std::string err;
  dbsp_place_opts po;
  po.P = P; po.mode = o.mode; po.max_item_len = o.max_item_len; po.item_overhead = o.item_overhead;
  po.locality_groups = o.locality_groups; po.partition_cost = o.partition_cost;
  po.dynamic_tail = o.dynamic_tail; po.reward = o.reward; po.pair = pair;
  if (host_only) {
    int rc = dbsp_build_host_plan(mask_host, H, nQ, nK, block, po, previous ? &previous->host : nullptr, reuse_threshold, plan->host, err);
    if (rc != DBSP_OK) {
      delete plan;
      return fail(rc, std::string(who) + ": " + err);
    }
  } else {
    // counts first; then the index lists are compacted into pinned memory on helper threads while
    // this thread builds the items and the placement; then everything is sent to the device
    dbsp_host_plan& hp = plan->host;
    plan->dev.max_batch = o.max_batch > 0 ? o.max_batch : 1;
    int rc = DBSP_OK;
    if (have_counts) hp = std::move(counted);
    else rc = dbsp_plan_count(mask_host, H, nQ, nK, block, pair, hp, err);
    if (rc != DBSP_OK) {
      delete plan;
      return fail(rc, std::string(who) + ": " + err);
    }
    rc = get_kv_staging(plan);
    if (rc != DBSP_OK) {
      free_device(plan->dev, true);
      delete plan;
      return rc;
    }
    hp.kv_idx = static_cast<const int32_t*>(plan->dev.staging_kv);
    dbsp_compaction job;
    dbsp_compact_begin(mask_host, hp, static_cast<int32_t*>(plan->dev.staging_kv), job);
    rc = dbsp_plan_place(po, previous ? &previous->host : nullptr, reuse_threshold, hp, err);
    const bool compacted = dbsp_compact_end(job);
    if (rc == DBSP_OK && !compacted) { rc = DBSP_ENOMEM; err = "out of host memory while planning"; }
    if (rc != DBSP_OK) {
      free_device(plan->dev, true);
      delete plan;
      return fail(rc, std::string(who) + ": " + err);
    }
    try {
      rc = upload(plan);
    } catch (const std::bad_alloc&) {
      rc = fail(DBSP_ENOMEM, std::string(who) + ": out of host memory while planning");
    }
    if (rc != DBSP_OK) {
      free_device(plan->dev, true);
      delete plan;
      return rc;
    }
  }
  plan->plan_usec = std::chrono::duration<double, std::micro>(std::chrono::steady_clock::now() - t_start).count();
  *out_plan = plan;
  return DBSP_OK;
}

int dbsp_plan_pair_rows(const dbsp_plan* plan, int32_t* pair_rows) {
  if (!plan || !pair_rows) return fail(DBSP_EINVAL, "dbsp_plan_pair_rows: null pointer");
  *pair_rows = plan->host.pair ? 1 : 0;
  return DBSP_OK;
}

int plan_sparse_attn(const uint8_t* mask_host, int32_t H, int32_t nQ, int32_t nK, int32_t block,
                     const dbsp_plan_opts* opts, dbsp_plan** out_plan) {
  return make_plan(mask_host, H, nQ, nK, block, opts, nullptr, 0.0, out_plan, "plan_sparse_attn");
}

int plan_sparse_attn_reuse(const dbsp_plan* previous, const uint8_t* mask_host, const dbsp_plan_opts* opts,
                           double reuse_threshold, dbsp_plan** out_plan, int32_t* reused, double* rho_under_previous) {
  if (reused) *reused = 0;
  if (rho_under_previous) *rho_under_previous = 0.0;
  if (!previous) {
    if (out_plan) *out_plan = nullptr;
    return fail(DBSP_EINVAL, "plan_sparse_attn_reuse: null previous plan");
  }
  if (!(reuse_threshold >= 1.0)) {
    if (out_plan) *out_plan = nullptr;
    return fail(DBSP_EINVAL, "plan_sparse_attn_reuse: the threshold must be at least 1");
  }
  const dbsp_host_plan& ph = previous->host;
  int rc = make_plan(mask_host, ph.H, ph.nQ_blocks, ph.nK, ph.block, opts, previous, reuse_threshold, out_plan, "plan_sparse_attn_reuse");
  if (rc != DBSP_OK) return rc;
  if (reused) *reused = (*out_plan)->host.reused ? 1 : 0;
  if (rho_under_previous) *rho_under_previous = (*out_plan)->host.rho_reuse;
  return DBSP_OK;
}

static void give_up(dbsp_plan* plan, bool wait) {
  if (!plan) return;
  if (plan->dev.resident || plan->dev.blob) free_device(plan->dev, wait);
  delete plan;
}

void dbsp_plan_destroy(dbsp_plan* plan) { give_up(plan, true); }

void dbsp_plan_release(dbsp_plan* plan) { give_up(plan, false); }

static int forward(const dbsp_plan* plan, const void* q, const void* k, const void* v, void* o,
                   float* lse, int32_t B, int32_t Nq, int32_t Nk, int32_t d, float softmax_scale,
                   void* stream, bool static_scratch_wanted, const char* who) {
  auto bad = [&](int code, const std::string& what) { return fail(code, std::string(who) + what); };
  if (!plan || !q || !k || !v || !o) return bad(DBSP_EINVAL, ": null pointer");
  const dbsp_host_plan& hp = plan->host;
  if (B <= 0) return bad(DBSP_EINVAL, ": B must be positive");
  if (d != 64 && d != 128) return bad(DBSP_EINVAL, ": head dim must be 64 or 128");
  if (hp.block != 64 && hp.block != 128) return bad(DBSP_EINVAL, ": the plan's block size must be 64 or 128");
  if (Nq <= 0 || Nk <= 0 || Nq % hp.block != 0 || Nk % hp.block != 0)
    return bad(DBSP_ESHAPE, ": sequence lengths must be positive multiples of the block size");
  if (Nq / hp.block != hp.nQ_blocks || Nk / hp.block != hp.nK)
    return bad(DBSP_ESHAPE, ": Nq/Nk do not match the plan's block grid");
  if (hp.pair && d != 128) return bad(DBSP_EINVAL, ": a plan made with DBSP_PLAN_PAIR_ROWS needs head dim 128");
  if (!plan->dev.resident) return bad(DBSP_EINVAL, ": the plan was built host-only");
  if (!(softmax_scale == softmax_scale)) return bad(DBSP_EINVAL, ": softmax_scale is NaN");
  int cur = -1;
  DBSP_HIP(hipGetDevice(&cur));
  if (cur != plan->dev.device) return bad(DBSP_EINVAL, ": the plan lives on another device than the current one");

  const dbsp_device_plan& dv = plan->dev;
  float* part_o = dv.part_o;
  float* part_lse = dv.part_lse;
  if (static_scratch_wanted) {
    // partial outputs f32 [B][n_slots][block][d], then their LSE f32 [B][n_slots][block]
    const size_t rows = (size_t)B * hp.n_slots * hp.tile_rows();
    const size_t lse_off = (rows * d * sizeof(float) + 255) & ~size_t(255);
    const size_t need = lse_off + rows * sizeof(float);
    if (need > kStaticScratchBytes)
      return bad(DBSP_EINVAL, ": the split rows of this plan need " + std::to_string(need) + " bytes of scratch for B = " +
                                   std::to_string(B) + ", the static buffer holds " + std::to_string(kStaticScratchBytes));
    unsigned char* base = nullptr;
    const int rc = static_scratch(cur, &base);
    if (rc != DBSP_OK) return rc;
    part_o = reinterpret_cast<float*>(base);
    part_lse = reinterpret_cast<float*>(base + lse_off);
  } else if (B > dv.max_batch && hp.n_slots > 0) {
    return bad(DBSP_EINVAL, ": B exceeds the max_batch the plan's split-row scratch was sized for");
  }

  dbsp_fwd_params p;
  p.q = static_cast<const uint16_t*>(q);
  p.k = static_cast<const uint16_t*>(k);
  p.v = static_cast<const uint16_t*>(v);
  p.o = static_cast<uint16_t*>(o);
  p.lse = lse;
  p.kv_idx = dv.kv_idx;
  p.empty_rows = dv.empty_rows;
  p.part_ptr = dv.part_ptr;
  p.sched = dv.sched;
  p.n_placed = (int32_t)hp.part_items.size();
  p.queue = dv.queue;
  p.n_tail = (int32_t)hp.tail_items.size();
  p.part_o = part_o;
  p.part_lse = part_lse;
  p.split_cnt = dv.split_cnt;
  p.split_rows = dv.split_rows;
  p.max_chunks = dv.max_chunks;
  // (the counters of in-place merges are sized for max_batch, and calls that share the static scratch leave
  // nothing behind in it: its split rows are merged by the second launch)
  p.in_place_ok = !static_scratch_wanted && (int64_t)B * hp.n_items() <= hp.P ? 1 : 0;
  p.local = dv.local ? 1 : 0;
  p.merge_later = 0;
  p.busy = dv.busy;
  p.hw_id = dv.hw_id;
  p.B = B; p.H = hp.H; p.nQ = hp.nQ; p.nK = hp.nK;
  p.Nq = Nq; p.Nk = Nk;
  p.n_slots = hp.n_slots;
  p.n_split = (int32_t)(hp.split_rows.size() / 4);
  p.n_empty = (int32_t)hp.empty_rows.size();
  p.scale = softmax_scale > 0.f ? softmax_scale : 1.0f / std::sqrt((float)d);
  p.scale_log2 = p.scale * 1.4426950408889634f;
  hipStream_t st = static_cast<hipStream_t>(stream);
  // every list with items gets its workgroup; what is left to deal (queue items, empty rows) may ask for more, up to P
  const int64_t deal = std::max<int64_t>((int64_t)B * p.n_tail, (int64_t)B * p.n_empty);
  const int grid = (int)std::max<int64_t>(std::max<int64_t>(dv.groups, 1), std::min<int64_t>(deal, hp.P));
  dbsp_device_plan& dm = plan->dev;
  // inside a stream capture everything goes through commands that a graph can hold
  hipStreamCaptureStatus capturing = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(st, &capturing) != hipSuccess) (void)hipGetLastError();
  const bool capture = capturing != hipStreamCaptureStatusNone;
  // The first launch of a small plan, no more than an item a workgroup, reads it where it lies in pinned memory: a launch
  // less, which the host takes longer to make than the kernel runs.  What such a launch counts it counts in the device buffer's front,
  // which has to be zero: the plan that had the buffer before has sent zeros there, and every launch leaves them.  The
  // second launch of the plan fetches it like any other's first.  512 tokens, two heads, planned on every call: 22 - 24 us a
  // pass with the fetch, 20 - 21 so (runs of one side differ by up to 4; the host's 19.3 and 17.7 for planning and launching).  A workgroup's way to its first
  // blocks is three or four reads across the bus, one behind the other, as long as the fetch took; with more items a
  // workgroup they would come in between.
  const bool direct = dm.direct && !dm.sent && !capture && B == 1 && p.in_place_ok;
  if (direct) {
    const int32_t* ints = static_cast<const int32_t*>(dm.staging);
    p.empty_rows = ints + dm.array_off[0];
    p.part_ptr = ints + dm.array_off[1];
    p.sched = ints + dm.array_off[2];
    p.split_rows = ints + dm.array_off[3];
    p.kv_idx = static_cast<const int32_t*>(dm.staging_kv);
    dm.direct = false;
  }
  bool in_order = false;           // the fetch is the command before this launch
  if (!direct && !dm.upload_done) {
    if (!dm.sent) {
      const bool fetch = !capture && dm.up_bytes + dm.kv_bytes <= kInStreamBytes;
      OutsideCapture relaxed;      // the copies go to a stream that is not captured
      const int rc = fetch ? fetch_in_stream(dm, st) : send_upload(dm);
      if (rc != DBSP_OK) {
        // (the error may be an earlier call's, the fetch under way, and nothing vouches for the buffers yet)
        if (fetch) (void)hipStreamSynchronize(st);
        return rc;
      }
      in_order = fetch;
    }
    if (!in_order) {
      hipEvent_t arrived = static_cast<hipEvent_t>(dm.uploaded);
      OutsideCapture relaxed;      // the event is another stream's
      if (capture) {
        // what a graph holds cannot wait for a command outside of it, and its replays, on any stream, are not
        // known here: the plan has arrived before its launch is recorded
        DBSP_HIP(hipEventSynchronize(arrived));
        dm.upload_done = true;
      } else {
        dm.upload_done = hipEventQuery(arrived) == hipSuccess;
        if (!dm.upload_done) {
          (void)hipGetLastError();
          DBSP_HIP(hipStreamWaitEvent(st, arrived, 0));
        }
      }
    }
  }
  const hipError_t e = dbsp_launch_fwd(p, hp.block, d, hp.pair, grid, st);
  // A record behind the launch, not the kernel's own completion event.  That is 1.5 us cheaper between launches of one
  // plan (12 heads, 21 x 23 blocks of 128: 56.8 to 58.3 us in a row), but leaves the runtime work for the calls after
  // them: a first pass on a new mask of that size took 114 us with it and takes 98, of 512 tokens 75 and 60, and 60
  // small kernels of another library behind 2000 launches 715 or 1130 us, varying from process to process, and 740
  // to 800 (with neither 735).  A plan's calls do not overlap, so a fetched plan's first launch needs one record only,
  // for the launch and the fetch before it (512 tokens, planned on every call: 25.8 to 19.7 us a pass).
  // (a captured launch leaves the event to the last one that was enqueued: a graph's replays are the caller's to wait for)
  hipError_t recorded = hipSuccess;
  if (!capture) {                  // (also where a launch has failed: an earlier one of the call may be under way)
    recorded = hipEventRecord(static_cast<hipEvent_t>(in_order ? dm.uploaded : dm.last_use), st);
    if (recorded != hipSuccess) (void)hipStreamSynchronize(st);      // nothing else could vouch for the plan's buffers
    else if (!in_order) dm.used = true;
  }
  if (e != hipSuccess) return fail_hip(e, (std::string(who) + " launch").c_str());
  if (recorded != hipSuccess) return fail_hip(recorded, (std::string(who) + ": record").c_str());
  dm.ran_staged = dm.ran_staged || direct;
  dm.last_grid = grid;
  return DBSP_OK;
}

int sparse_attn_fwd(const dbsp_plan* plan, const void* q, const void* k, const void* v, void* o,
                    float* lse, int32_t B, int32_t Nq, int32_t Nk, int32_t d, float softmax_scale,
                    void* stream) {
  return forward(plan, q, k, v, o, lse, B, Nq, Nk, d, softmax_scale, stream, false, "sparse_attn_fwd");
}

int sparse_attn_fwd_static(const dbsp_plan* plan, const void* q, const void* k, const void* v, void* o,
                           float* lse, int32_t B, int32_t Nq, int32_t Nk, int32_t d, float softmax_scale,
                           void* stream) {
  return forward(plan, q, k, v, o, lse, B, Nq, Nk, d, softmax_scale, stream, true, "sparse_attn_fwd_static");
}

int imbalance_ratio(const int64_t* work, int32_t periods, int32_t partitions, double* rho_out) {
  if (!work || !rho_out) return fail(DBSP_EINVAL, "imbalance_ratio: null pointer");
  if (periods <= 0 || partitions <= 0) return fail(DBSP_EINVAL, "imbalance_ratio: periods and partitions must be positive");
  for (int64_t i = 0; i < (int64_t)periods * partitions; ++i)
    if (work[i] < 0) return fail(DBSP_EINVAL, "imbalance_ratio: negative work entry");
  *rho_out = dbsp_rho(work, periods, partitions);
  return DBSP_OK;
}

int dbsp_plan_get(const dbsp_plan* plan, int32_t what, const void** data, int64_t* count) {
  if (!plan || !data || !count) return fail(DBSP_EINVAL, "dbsp_plan_get: null pointer");
  const dbsp_host_plan& hp = plan->host;
#define DBSP_ARR(vec) do { *data = (vec).data(); *count = (int64_t)(vec).size(); return DBSP_OK; } while (0)
  switch (what) {
    case DBSP_ROW_PTR: DBSP_ARR(hp.row_ptr);
    case DBSP_KV_IDX: *data = hp.kv_idx; *count = hp.kv_ints(); return DBSP_OK;
    case DBSP_ITEMS: DBSP_ARR(hp.items);
    case DBSP_ITEM_SLOT: DBSP_ARR(hp.item_slot);
    case DBSP_SPLIT_ROWS: DBSP_ARR(hp.split_rows);
    case DBSP_PART_PTR: DBSP_ARR(hp.part_ptr);
    case DBSP_PART_ITEMS: DBSP_ARR(hp.part_items);
    case DBSP_PART_LOAD: DBSP_ARR(hp.part_load);
    case DBSP_BLOCKS_PER_HEAD: DBSP_ARR(hp.blocks_per_head);
    case DBSP_ROW_CNT: DBSP_ARR(hp.row_cnt);
    case DBSP_EMPTY_ROWS: DBSP_ARR(hp.empty_rows);
    case DBSP_TAIL_ITEMS: DBSP_ARR(hp.tail_items);
    default: return fail(DBSP_EINVAL, "dbsp_plan_get: unknown array id");
  }
#undef DBSP_ARR
}

int dbsp_plan_stats(const dbsp_plan* plan, double* rho_naive, double* rho_balanced, double* rho_plan,
                    int64_t* nnz, int64_t* n_items, int32_t* num_partitions, int32_t* max_item_len,
                    double* plan_usec) {
  if (!plan) return fail(DBSP_EINVAL, "dbsp_plan_stats: null plan");
  const dbsp_host_plan& hp = plan->host;
  if (rho_naive || rho_balanced) {
    std::lock_guard<std::mutex> lk(plan->lazy_mu);
    const bool need_n = rho_naive && !hp.have_rho_naive, need_b = rho_balanced && !hp.have_rho_balanced;
    if (need_n || need_b) {
      try {
        dbsp_host_plan_lazy_rhos(hp, need_n, need_b, &hp.rho_naive, &hp.rho_balanced);
      } catch (const std::bad_alloc&) {
        return fail(DBSP_ENOMEM, "dbsp_plan_stats: out of host memory");
      }
      hp.have_rho_naive = hp.have_rho_naive || need_n;
      hp.have_rho_balanced = hp.have_rho_balanced || need_b;
    }
    if (rho_naive) *rho_naive = hp.rho_naive;
    if (rho_balanced) *rho_balanced = hp.rho_balanced;
  }
  if (rho_plan) *rho_plan = hp.rho_mode;
  if (nnz) *nnz = hp.nnz;
  if (n_items) *n_items = hp.n_items();
  if (num_partitions) *num_partitions = hp.P;
  if (max_item_len) *max_item_len = hp.max_item_len;
  if (plan_usec) *plan_usec = plan->plan_usec;
  return DBSP_OK;
}

int dbsp_plan_busy(const dbsp_plan* plan, uint64_t* busy_ticks, uint32_t* hw_id, void* stream) {
  if (!plan) return fail(DBSP_EINVAL, "dbsp_plan_busy: null plan");
  if (!plan->dev.resident) return fail(DBSP_EINVAL, "dbsp_plan_busy: the plan was built host-only");
  DBSP_HIP(hipStreamSynchronize(static_cast<hipStream_t>(stream)));
  // partitions the last launch had no workgroup for (no items) were idle
  const dbsp_device_plan& dv = plan->dev;
  const int32_t ran = dv.last_grid;
  try {
    auto fetch = [&](auto* out, const auto* from) {
      std::fill(out, out + plan->host.P, 0);
      std::vector<std::remove_reference_t<decltype(*out)>> by_group(ran);
      const hipError_t e = ran ? hipMemcpy(by_group.data(), from, ran * sizeof(*out), hipMemcpyDeviceToHost) : hipSuccess;
      for (int32_t b = 0; b < ran && e == hipSuccess; ++b) out[dv.part_of(b)] = by_group[b];
      return e;
    };
    if (busy_ticks) DBSP_HIP(fetch(busy_ticks, dv.busy));
    if (hw_id) DBSP_HIP(fetch(hw_id, dv.hw_id));
  } catch (const std::bad_alloc&) {
    return fail(DBSP_ENOMEM, "dbsp_plan_busy: out of host memory");
  }
  return DBSP_OK;
}

int dbsp_plan_tail_takes(const dbsp_plan* plan, uint32_t* takes, void* stream) {
  if (!plan || !takes) return fail(DBSP_EINVAL, "dbsp_plan_tail_takes: null pointer");
  if (!plan->dev.resident) return fail(DBSP_EINVAL, "dbsp_plan_tail_takes: the plan was built host-only");
  DBSP_HIP(hipStreamSynchronize(static_cast<hipStream_t>(stream)));
  const size_t n = plan->host.tail_items.size();
  if (!plan->dev.sent) std::fill(takes, takes + n, 0);      // no launch yet
  else if (n) DBSP_HIP(hipMemcpy(takes, plan->dev.queue + 1, n * sizeof(uint32_t), hipMemcpyDeviceToHost));
  return DBSP_OK;
}

int dbsp_plan_calibrate(const dbsp_plan* plan, int32_t* cost, void* stream) {
  if (!plan || !cost) return fail(DBSP_EINVAL, "dbsp_plan_calibrate: null pointer");
  if (!plan->dev.resident) return fail(DBSP_EINVAL, "dbsp_plan_calibrate: the plan was built host-only");
  const dbsp_host_plan& hp = plan->host;
  const int32_t P = hp.P;
  try {
    std::vector<uint64_t> busy(P);
    const int rc = dbsp_plan_busy(plan, busy.data(), nullptr, stream);
    if (rc != DBSP_OK) return rc;
    // round(1024 * (busy[g] / load[g]) / (sum busy / sum load)), exact, round half up
    unsigned __int128 sb = 0, sl = 0;
    for (int32_t g = 0; g < P; ++g)
      if (busy[g] > 0 && hp.part_load[g] > 0) {
        sb += busy[g];
        sl += (uint64_t)hp.part_load[g];
      }
    // the workgroup that ran partition g here runs partition `to` of a plan with costs
    const int32_t cost_log2 = hp.by_greedy ? longest_runs_log2(P) : 0;
    for (int32_t b = 0; b < P; ++b) {
      const int32_t g = plan->dev.part_of(b), to = dbsp_part_of(b, P, cost_log2);
      const int64_t l = hp.part_load[g];
      if (busy[g] == 0 || l <= 0 || sb == 0) { cost[to] = 1024; continue; }
      const unsigned __int128 num = (unsigned __int128)busy[g] * 1024 * sl, den = (unsigned __int128)(uint64_t)l * sb;
      const unsigned __int128 q = (2 * num + den) / (2 * den);
      cost[to] = q < 512 ? 512 : q > 2048 ? 2048 : (int32_t)q;
    }
  } catch (const std::bad_alloc&) {
    return fail(DBSP_ENOMEM, "dbsp_plan_calibrate: out of host memory");
  }
  return DBSP_OK;
}

int dbsp_plan_run_order(const dbsp_plan* plan, int32_t* partition_of, int32_t* items, int32_t* local, int32_t* staged) {
  if (!plan) return fail(DBSP_EINVAL, "dbsp_plan_run_order: null plan");
  const dbsp_host_plan& hp = plan->host;
  try {
    const RunOrder o = run_order(hp);
    if (partition_of)
      for (int32_t b = 0; b < hp.P; ++b) partition_of[b] = dbsp_part_of(b, o.parts, o.run_log2);
    const std::vector<int32_t>& run = o.own ? o.run : hp.part_items;
    if (items) std::copy(run.begin(), run.end(), items);
    if (local) *local = o.local ? 1 : 0;
  } catch (const std::bad_alloc&) {
    return fail(DBSP_ENOMEM, "dbsp_plan_run_order: out of host memory");
  }
  if (staged) *staged = plan->dev.ran_staged ? 1 : 0;
  return DBSP_OK;
}

}  // extern "C"
