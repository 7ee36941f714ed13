#include "profile.h"

#include <mutex>
#include <new>
#include <vector>

namespace dynmo {

std::atomic<bool> g_profile_on{false};

namespace {
struct Pair {
  hipEvent_t start, stop;
  int holders;  // slots that have not folded it yet
};
struct Pending {
  Pair* pair;
  double share;  // of the pair's duration
};
struct Slot {
  std::vector<Pending> pending;
  double total_ms = 0.0;
  int64_t launches = 0;
};
Slot g_slots[K_COUNT];
std::vector<hipEvent_t> g_free;
std::mutex g_mu;
constexpr size_t kMaxPending = 1 << 16;

const char* const kNames[K_COUNT] = {
    "route_topk",    "route_capacity", "route_active", "route_topk_bwd", "route_capacity_bwd",
    "route_drop",
    "permute_count", "permute_scan",   "permute_scatter", "permute_rows", "permute_bwd",
    "combine",       "combine_bwd",    "ffn_gateup",   "ffn_down",       "ffn_dA",
    "ffn_dX",        "ffn_dWd",        "ffn_dWg",      "ffn_dWu"};

hipEvent_t get_event() {
  if (!g_free.empty()) {
    hipEvent_t e = g_free.back();
    g_free.pop_back();
    return e;
  }
  hipEvent_t e = nullptr;
  if (hipEventCreate(&e) != hipSuccess) return nullptr;
  return e;
}

// Folds finished event pairs of one slot into its totals.  Waits for each stop event.
int32_t drain(Slot& s) {
  for (const Pending& q : s.pending) {
    DYNMO_HIP_TRY(hipEventSynchronize(q.pair->stop));
    float ms = 0.f;
    DYNMO_HIP_TRY(hipEventElapsedTime(&ms, q.pair->start, q.pair->stop));
    s.total_ms += ms * q.share;
    s.launches += 1;
  }
  for (const Pending& q : s.pending) {
    if (--q.pair->holders > 0) continue;
    g_free.push_back(q.pair->start);
    g_free.push_back(q.pair->stop);
    delete q.pair;
  }
  s.pending.clear();
  return DYNMO_OK;
}
}  // namespace

hipEvent_t profile_begin(const ProfRoles& roles, hipStream_t st) {
  std::lock_guard<std::mutex> lk(g_mu);
  double all = 0.0;
  for (int i = 0; i < roles.n; ++i) {
    if (g_slots[roles.id[i]].pending.size() >= kMaxPending) return nullptr;
    all += roles.work[i];
  }
  Pair* pair = new (std::nothrow) Pair;
  hipEvent_t a = pair ? get_event() : nullptr, b = pair ? get_event() : nullptr;
  if (!a || !b) {
    if (a) g_free.push_back(a);
    if (b) g_free.push_back(b);
    delete pair;
    return nullptr;
  }
  *pair = Pair{a, b, roles.n};
  for (int i = 0; i < roles.n; ++i) g_slots[roles.id[i]].pending.push_back(Pending{pair, roles.work[i] / all});
  (void)hipEventRecord(a, st);
  return b;
}

void profile_end(hipEvent_t stop, hipStream_t st) { (void)hipEventRecord(stop, st); }

}  // namespace dynmo

using namespace dynmo;

extern "C" int32_t dynmo_profile_enable(int32_t on) {
  g_profile_on.store(on != 0);
  return DYNMO_OK;
}

extern "C" int32_t dynmo_profile_reset(void) {
  std::lock_guard<std::mutex> lk(g_mu);
  for (int i = 0; i < K_COUNT; ++i) {
    int32_t rc = drain(g_slots[i]);
    if (rc) return rc;
    g_slots[i].total_ms = 0.0;
    g_slots[i].launches = 0;
  }
  return DYNMO_OK;
}

extern "C" int32_t dynmo_profile_kernel_count(void) { return K_COUNT; }

extern "C" const char* dynmo_profile_kernel_name(int32_t id) {
  return (id >= 0 && id < K_COUNT) ? kNames[id] : nullptr;
}

extern "C" int32_t dynmo_profile_read(int32_t id, double* total_ms_host, int64_t* launches_host) {
  if (id < 0 || id >= K_COUNT || !total_ms_host || !launches_host) return DYNMO_EINVAL;
  std::lock_guard<std::mutex> lk(g_mu);
  int32_t rc = drain(g_slots[id]);
  if (rc) return rc;
  *total_ms_host = g_slots[id].total_ms;
  *launches_host = g_slots[id].launches;
  return DYNMO_OK;
}
