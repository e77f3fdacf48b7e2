// Which rows the launches of a layer step work on, built and run by tests/test_abi_host.py on the CPU: the library's own host code
// with its launches replaced by records.  Large batches are cut (whole rounds of tiles first, the rest behind them): every token's
// row of every product has to be written once, from its own row of the input.
#include <hip/hip_runtime.h>

#include <cstdio>
#include <cstdlib>
#include <map>
#include <vector>

#include "fllayer.h"
#include "flp_internal.h"

#define REQUIRE(cond)                                                      \
  do {                                                                     \
    if (!(cond)) {                                                         \
      std::fprintf(stderr, "layer_rows: line %d: %s (%s)\n", __LINE__, #cond, what); \
      std::exit(1);                                                        \
    }                                                                      \
  } while (0)

namespace {
char what[200] = "";
struct Product {               // one weight matrix: where its rows began, how many there have been, in how many launches
  const uint8_t* x = nullptr;
  uint8_t* y = nullptr;
  int rows = 0, launches = 0;
};
std::map<const void*, Product> products;
struct Branch {                // one projection's LoRA branch, by its table of places
  const uint8_t* x = nullptr;
  const int32_t* adapters = nullptr;
  uint8_t* y = nullptr;
  int rows = 0;
};
std::map<const void*, Branch> branches;

void add_branch(const FlpLoraArgs& a) {
  for (int p = 0; p < a.n_proj; ++p) {
    Branch& b = branches[a.proj[p].b_tab_off];
    if (!b.rows) b = Branch{(const uint8_t*)a.x, a.token_adapter, (uint8_t*)a.proj[p].y, 0};
    REQUIRE((const uint8_t*)a.x == b.x + (int64_t)b.rows * a.ld_x * 2 && a.token_adapter == b.adapters + b.rows);
    REQUIRE((uint8_t*)a.proj[p].y == b.y + (int64_t)b.rows * a.proj[p].ld_y * 2);
    b.rows += a.T;
  }
}
}  // namespace

flp_status flp_launch_gemm(int, const void* x, int64_t ld_x, int M, int, const FlpGemmPlan& plan, int n_proj, const FlpGemmOut* out,
                           bool, const FlpGemmLora*, hipStream_t) {
  for (int i = 0; i < n_proj; ++i) {
    Product& p = products[out[i].w];
    if (!p.launches) p = Product{(const uint8_t*)x, (uint8_t*)out[i].y, 0, 0};
    REQUIRE((const uint8_t*)x == p.x + (int64_t)p.rows * ld_x * 2);
    REQUIRE((uint8_t*)out[i].y == p.y + (int64_t)p.rows * out[i].ld_y * 2);
    REQUIRE((plan.splits > 1) <= (out[i].part != nullptr));
    p.rows += M;
    ++p.launches;
  }
  return FLP_OK;
}
flp_status flp_launch_lora_mfma(int, const FlpLoraArgs& a, const FlpLoraMfma&, hipStream_t) {
  add_branch(a);
  return FLP_OK;
}
flp_status flp_launch_lora_small(int, const FlpLoraArgs& a, const FlpLoraSmall&, hipStream_t) {
  add_branch(a);
  return FLP_OK;
}

extern "C" {
hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t) { return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3*, dim3*, size_t*, hipStream_t*) { return hipSuccess; }
hipError_t hipLaunchKernel(const void*, dim3, dim3, void**, size_t, hipStream_t) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipGetDevice(int*) { return hipErrorNoDevice; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
  *e = (hipEvent_t)16;
  return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipMalloc(void** p, size_t n) {
  *p = std::malloc(n);                       // never touched
  return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { return hipMalloc(p, n); }
hipError_t hipFree(void* p) {
  std::free(p);
  return hipSuccess;
}
hipError_t hipHostFree(void* p) { return hipFree(p); }
int32_t flp_dense_first_tokens(int32_t T, int32_t K, int32_t n, const int32_t* N, int32_t lora);
}

int main() {
  struct Shape {
    int hidden, heads, kv, mlp, T;
    bool branches[2];          // on q, k, v, o; on gate, up, down
    bool cut, again;           // some product is cut; the planner, asked for its first part alone, would cut that too
  };
  const Shape shapes[] = {
      {4096, 32, 32, 11008, 4400, {true, false}, true, false},    {5120, 40, 40, 13824, 9874, {true, true}, true, false},
      {8192, 64, 8, 22016, 2200, {true, false}, true, false},     {4096, 32, 32, 11008, 4400, {false, false}, true, false},
      {4096, 32, 32, 11008, 499, {true, true}, false, false},     {4096, 32, 32, 11008, 4096, {false, false}, false, false},
      {28672, 1, 1, 17920, 2564, {false, false}, true, true},     {25088, 1, 1, 17920, 2564, {false, false}, true, true},
      {22016, 1, 1, 36480, 2309, {false, false}, true, true},     {25600, 1, 1, 17920, 2616, {false, false}, true, true},
      {17920, 1, 1, 28672, 2600, {false, false}, true, false},    {35840, 1, 1, 28672, 2564, {false, false}, true, true},
  };
  for (const Shape& s : shapes) {
    std::snprintf(what, sizeof what, "hidden %d heads %d / %d mlp %d tokens %d", s.hidden, s.heads, s.kv, s.mlp, s.T);
    flp_pool_config pc{};
    pc.dtype = FLP_F16;
    pc.block_tokens = 16;
    pc.n_kv_heads = s.kv;
    pc.head_dim = 128;
    flp_pool* pool = nullptr;
    REQUIRE(flp_pool_create(&pc, &pool) == FLP_OK);
    pool->block_elems = 1 << 20;             // rows of every width fit a block
    const fll_layer_config c{s.hidden, s.heads, s.mlp, 0.f, 0.f, 0};
    const uintptr_t fake = (uintptr_t)1 << 40;             // device addresses, not to be touched
    auto at = [&](int i) { return (const void*)(fake * (i + 1)); };
    const fll_layer_weights w{at(0), at(1), at(2), at(3), at(4), at(5), at(6), at(7), at(8)};
    const int32_t cu[2] = {0, s.T}, prefix[1] = {0};
    fll_layer_batch b{};
    b.n_tokens = s.T;
    b.n_seqs = 1;
    b.n_adapters = 4;
    b.max_rank = 16;
    b.max_blocks_per_seq = (s.T + 15) / 16;
    b.cu_new = cu;
    b.prefix_len = prefix;
    b.positions = b.kv_tables = b.token_adapter = b.rank = b.lora_tables = (const int32_t*)at(9);
    b.scale = (const float*)at(9);
    for (int i = 0; i < 7; ++i)
      if (s.branches[i >= 4]) {
        const int32_t* t = (const int32_t*)at(20 + i);
        b.lora[i] = fll_lora_place{t, t, t, t};
      }
    products.clear();
    branches.clear();
    const int64_t bytes = fll_layer_scratch_bytes(pool, &c, s.T);
    const flp_status st = fll_layer_forward(pool, &c, &w, &b, (void*)at(10), (void*)at(11), bytes, nullptr);
    if (st != FLP_OK) std::fprintf(stderr, "%s\n", flp_last_error());
    REQUIRE(st == FLP_OK);
    bool cut = false, again = false;
    REQUIRE(products.size() == 7 || products.size() == 6);               // gate and up may be one product
    for (auto& [m, p] : products) {
      REQUIRE(p.rows == s.T && p.launches <= 2);
      cut = cut || p.launches == 2;
    }
    for (auto& [m, r] : branches) REQUIRE(r.rows == s.T);
    REQUIRE(branches.size() == (size_t)(4 * s.branches[0] + 3 * s.branches[1]));
    for (const auto& [K, N] : {std::pair<int, int>{s.hidden, 2 * s.mlp}, {s.mlp, s.hidden}}) {
      const int first = flp_dense_first_tokens(s.T, K, 1, &N, 0);
      again = again || flp_dense_first_tokens(first, K, 1, &N, 0) < first;
    }
    REQUIRE(cut == s.cut && again == s.again);
    REQUIRE(flp_pool_destroy(pool) == FLP_OK);
  }
  std::printf("every row of every product is written once\n");
  return 0;
}
