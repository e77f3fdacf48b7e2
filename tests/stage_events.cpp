// The staging ring and the workspaces that one call hands to the next (pool.cpp) over events of a model, built and run by
// tests/test_abi_host.py on the CPU.  An event that is inspected (hipEventQuery, hipEventSynchronize) says that its slot may be
// filled again, so it has to have been created for that: HIP documents that an event with hipEventDisableSystemFence does not
// synchronise with the work before it when it is inspected.  One that another stream waits for needs a device-scope release.
#include <cstdio>
#include <cstdlib>
#include <map>
#include <utility>
#include <vector>

#include "flp_internal.h"

flp_status flp_launch_copy_blocks(const uint8_t*, uint8_t*, const int32_t*, const int32_t*, int32_t, int64_t, int, hipStream_t) {
  std::abort();
}
flp_status flp_launch_stage_copy(const void*, void*, size_t, hipStream_t) { return FLP_OK; }
flp_status flp_static_scratch_setup(int, void**) { return FLP_EHIP; }

#define REQUIRE(cond)                                                    \
  do {                                                                   \
    if (!(cond)) {                                                       \
      std::fprintf(stderr, "stage_events: line %d: %s\n", __LINE__, #cond); \
      std::exit(1);                                                      \
    }                                                                    \
  } while (0)

namespace {
struct Event {
  unsigned flags;
  bool done;
};
std::vector<std::pair<hipStream_t, hipEvent_t>> waits;
int synchronized = 0;
Event* of(hipEvent_t e) { return reinterpret_cast<Event*>(e); }
constexpr unsigned kUnfenced = hipEventDisableSystemFence;
}  // namespace

extern "C" {
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned flags) {
  *e = reinterpret_cast<hipEvent_t>(new Event{flags, false});
  return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t e) {
  delete of(e);
  return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t) {
  of(e)->done = false;
  return hipSuccess;
}
hipError_t hipEventQuery(hipEvent_t e) {
  REQUIRE(!(of(e)->flags & kUnfenced));
  return of(e)->done ? hipSuccess : hipErrorNotReady;
}
hipError_t hipEventSynchronize(hipEvent_t e) {
  REQUIRE(!(of(e)->flags & kUnfenced));
  ++synchronized;
  of(e)->done = true;
  return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) {
  REQUIRE(!(of(e)->flags & kUnfenced));
  waits.emplace_back(s, e);
  return hipSuccess;
}
hipError_t hipMalloc(void** p, size_t n) {
  *p = std::malloc(n);
  return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { return hipMalloc(p, n); }
hipError_t hipFree(void* p) {
  std::free(p);
  return hipSuccess;
}
hipError_t hipHostFree(void* p) { return hipFree(p); }
hipError_t hipGetDevice(int*) { return hipErrorNoDevice; }
}

int main() {
  flp_pool_config cfg{};
  cfg.dtype = FLP_F16;
  cfg.block_tokens = 16;
  cfg.n_kv_heads = 1;
  cfg.head_dim = 64;
  flp_pool* p = nullptr;
  REQUIRE(flp_pool_create(&cfg, &p) == FLP_OK);
  const hipStream_t s1 = reinterpret_cast<hipStream_t>(16), s2 = reinterpret_cast<hipStream_t>(32);

  // every slot once, then again: the second time round each is still in use, or done
  FlpStageSlot* slot = nullptr;
  for (int k = 0; k < 2 * kStageSlots; ++k) {
    if (k >= kStageSlots && k % 2) of(p->stage[k - kStageSlots].ev)->done = true;
    REQUIRE(flp_stage_acquire(p, 100, &slot) == FLP_OK);
    REQUIRE(slot->cap >= 100 && !slot->in_flight);
    REQUIRE(flp_stage_release(slot, s1) == FLP_OK);
    REQUIRE(slot->in_flight);
  }
  REQUIRE(synchronized == kStageSlots / 2);

  // a call on another stream waits for the one that used the split contexts' workspace, a call on the same one does not
  void* ws = nullptr;
  p->attn_slot = slot;
  p->attn_stream = s1;
  REQUIRE(flp_attn_workspace(p, 1000, s1, &ws) == FLP_OK && waits.empty());
  REQUIRE(flp_attn_workspace(p, 1000, s2, &ws) == FLP_OK && waits.size() == 1);
  REQUIRE(waits[0].first == s2 && waits[0].second == slot->ev);

  REQUIRE(flp_dense_workspace_acquire(p, 1000, s1, &ws) == FLP_OK && waits.size() == 1);
  REQUIRE(flp_dense_workspace_release(p, s1) == FLP_OK);
  REQUIRE(flp_dense_workspace_acquire(p, 1000, s2, &ws) == FLP_OK && waits.size() == 2);
  REQUIRE(flp_pool_destroy(p) == FLP_OK);
  std::printf("every event is fenced where it is looked at\n");
  return 0;
}
