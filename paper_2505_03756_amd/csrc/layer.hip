// Layer glue (include/fllayer.h): root-mean-square norm (optionally fused with the residual update
// before it), rotary position embedding, gated SiLU, and the call that strings them together with the
// pool's projections (base GEMM + paged LoRA), KV append and paged prefix attention into one decoder
// layer of the models the paper serves (section 6.1).  The element-wise kernels are plain HBM streams:
// 16 bytes per lane per access, fp32 arithmetic, one rounding at the store.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <mutex>
#include <type_traits>

#include "fllayer.h"
#include "flp_internal.h"
#include "flp_types.h"

namespace {

template <typename S>
struct Vec {
  static constexpr int N = 16 / (int)sizeof(typename S::storage);
  typename S::storage e[N];
};

template <typename S>
__device__ __forceinline__ Vec<S> ldv(const void* p) {
  Vec<S> v;
  const u32x4 raw = *reinterpret_cast<const u32x4*>(p);
  __builtin_memcpy(&v, &raw, 16);
  return v;
}
template <typename S>
__device__ __forceinline__ void stv(void* p, const Vec<S>& v) {
  u32x4 raw;
  __builtin_memcpy(&raw, &v, 16);
  *reinterpret_cast<u32x4*>(p) = raw;
}

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// W waves (4 or 1) per token row, four waves to a workgroup, for rows of up to 64 W NV vectors of 16 bytes: all loads of the row
// (and of the delta and the gains) are in flight together and the row stays in registers between the sum of squares and the
// scaling, so the call is one trip to memory.  With a delta the rounded residual is stored and the sum is taken over it.  A
// batch of a few rows is bound by that trip, a large one by the bytes, or by the number of workgroups where the rows are short:
// those of up to 96 vectors take one wave.  The layer's three calls, with a wave per row in two passes, with this:
//   8 rows of 4096, bf16          6.7 10.5 5.7    4.7 3.7 4.6 us
//   9876 rows of 5120, fp16      45.8 83.8 55.8   30.8 61.1 46.4 us (6.6 TB/s in the second)
// Norm, norm with residual of short bf16 rows, in two passes, four waves, one:
//   40000 rows of   64    15.7 27.9 14.6    19.8 36.5 18.6 us
//   10000 rows of  256     9.1 11.8  8.8    11.5 15.0 11.3 us
//   40000 rows of  256    19.8 31.8 17.9    28.4 45.6 26.2 us
//   40000 rows of  512    25.4 35.5 24.3    43.2 50.3 42.7 us
//   40000 rows of  768    38.2 44.3 37.0    63.5 61.6 62.8 us
//   40000 rows of 1024    47.8 47.6 46.5    80.4 69.9 81.7 us
template <typename S, int NV, int W>
__global__ __launch_bounds__(256) void rmsnorm_kernel(const typename S::storage* x_in, typename S::storage* resid,
                                                      const typename S::storage* __restrict__ delta,
                                                      const typename S::storage* __restrict__ w,
                                                      typename S::storage* y, int T, int H, float eps) {
  typedef typename S::storage ST;
  constexpr int N = Vec<S>::N;
  __shared__ float part[4];
  const int t = W == 4 ? blockIdx.x : 4 * blockIdx.x + (threadIdx.x >> 6);
  if (W < 4 && t >= T) return;                         // W == 1: the waves of a workgroup share nothing
  const int64_t row = (int64_t)t * H;
  const int c0 = (threadIdx.x & (64 * W - 1)) * N;
  const ST* xr = (delta ? resid : x_in) + row;
  Vec<S> a[NV], d[NV], g[NV];
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const int c = c0 + i * 64 * W * N;
    if (c >= H) break;
    a[i] = ldv<S>(xr + c);
    if (delta) d[i] = ldv<S>(delta + row + c);
    if (y) g[i] = ldv<S>(w + c);
  }
  float ss = 0.f;
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const int c = c0 + i * 64 * W * N;
    if (c >= H) break;
    if (delta) {
#pragma unroll
      for (int j = 0; j < N; ++j) a[i].e[j] = S::from_float(S::to_float(a[i].e[j]) + S::to_float(d[i].e[j]));
      stv<S>(resid + row + c, a[i]);
    }
#pragma unroll
    for (int j = 0; j < N; ++j) {
      const float f = S::to_float(a[i].e[j]);
      ss = fmaf(f, f, ss);
    }
  }
  if (!y) return;
  ss = wave_sum(ss);
  if (W == 4) {
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = ss;
    __syncthreads();
    ss = (part[0] + part[1]) + (part[2] + part[3]);
  }
  const float inv = 1.0f / sqrtf(ss / (float)H + eps);
#pragma unroll
  for (int i = 0; i < NV; ++i) {
    const int c = c0 + i * 64 * W * N;
    if (c >= H) break;
    Vec<S> o;
#pragma unroll
    for (int j = 0; j < N; ++j) o.e[j] = S::from_float(S::to_float(a[i].e[j]) * inv * S::to_float(g[i].e[j]));
    stv<S>(y + row + c, o);
  }
}

// Longer rows: one wave per token row, four rows per workgroup.  Pass 1 accumulates the sum of squares (and, with
// a delta, stores the rounded residual it is taken over); pass 2 re-reads the row (each lane the bytes
// it touched in pass 1: L1/L2 hits) and writes the normalised row.
template <typename S>
__global__ __launch_bounds__(256) void rmsnorm_long_kernel(const typename S::storage* x_in, typename S::storage* resid,
                                                      const typename S::storage* __restrict__ delta,
                                                      const typename S::storage* __restrict__ w,
                                                      typename S::storage* y, int T, int H, float eps) {
  typedef typename S::storage ST;
  constexpr int N = Vec<S>::N;
  const int row = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (row >= T) return;
  const ST* xr = (delta ? resid : x_in) + (int64_t)row * H;
  float ss = 0.f;
  for (int c = lane * N; c < H; c += 64 * N) {
    Vec<S> a = ldv<S>(xr + c);
    if (delta) {
      const Vec<S> d = ldv<S>(delta + (int64_t)row * H + c);
#pragma unroll
      for (int j = 0; j < N; ++j) a.e[j] = S::from_float(S::to_float(a.e[j]) + S::to_float(d.e[j]));
      stv<S>(resid + (int64_t)row * H + c, a);
    }
#pragma unroll
    for (int j = 0; j < N; ++j) {
      const float f = S::to_float(a.e[j]);
      ss = fmaf(f, f, ss);
    }
  }
  if (!y) return;
  ss = wave_sum(ss);
  const float inv = 1.0f / sqrtf(ss / (float)H + eps);
  for (int c = lane * N; c < H; c += 64 * N) {
    const Vec<S> a = ldv<S>(xr + c), g = ldv<S>(w + c);
    Vec<S> o;
#pragma unroll
    for (int j = 0; j < N; ++j) o.e[j] = S::from_float(S::to_float(a.e[j]) * inv * S::to_float(g.e[j]));
    stv<S>(y + (int64_t)row * H + c, o);
  }
}

// One workgroup per token.  The d/2 angles of the token are computed once in fp64 (position times
// theta^(-2i/d) reaches thousands of radians: fp32 would lose the fraction that matters), their sine and
// cosine kept in LDS as fp32, then every head's pairs are rotated, 16 bytes of each half per thread.
template <typename S, int D>
__global__ __launch_bounds__(256) void rope_kernel(typename S::storage* __restrict__ q, typename S::storage* __restrict__ k,
                                                   const int32_t* __restrict__ positions, int n_h, int n_kv,
                                                   double log2_theta) {
  typedef typename S::storage ST;
  constexpr int N = Vec<S>::N, HALF = D / 2, VPH = HALF / N;    // 16-byte vectors per half head
  __shared__ float cs[HALF], sn[HALF];
  const int t = blockIdx.x;
  if (threadIdx.x < HALF) {
    const double ang = (double)positions[t] * exp2(-2.0 * (double)threadIdx.x / (double)D * log2_theta);
    double s, c;
    sincos(ang, &s, &c);
    cs[threadIdx.x] = (float)c;
    sn[threadIdx.x] = (float)s;
  }
  __syncthreads();
  const int n_q_items = q ? n_h * VPH : 0, n_items = n_q_items + (k ? n_kv * VPH : 0);
  for (int it = threadIdx.x; it < n_items; it += 256) {
    const bool is_q = it < n_q_items;
    const int local = is_q ? it : it - n_q_items;
    const int head = local / VPH, i0 = (local % VPH) * N;
    ST* base = is_q ? q + ((int64_t)t * n_h + head) * D : k + ((int64_t)t * n_kv + head) * D;
    const Vec<S> a = ldv<S>(base + i0), b = ldv<S>(base + HALF + i0);
    Vec<S> oa, ob;
#pragma unroll
    for (int j = 0; j < N; ++j) {
      const float af = S::to_float(a.e[j]), bf = S::to_float(b.e[j]), c = cs[i0 + j], s = sn[i0 + j];
      oa.e[j] = S::from_float(af * c - bf * s);
      ob.e[j] = S::from_float(bf * c + af * s);
    }
    stv<S>(base + i0, oa);
    stv<S>(base + HALF + i0, ob);
  }
}

template <typename S>
__global__ __launch_bounds__(256) void silu_mul_kernel(const typename S::storage* __restrict__ gate, int64_t ld_g,
                                                       const typename S::storage* __restrict__ up, int64_t ld_u,
                                                       typename S::storage* __restrict__ out, int64_t ld_o, int64_t n_vec,
                                                       int vec_per_row) {
  constexpr int N = Vec<S>::N;
  const int64_t v = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (v >= n_vec) return;
  const int64_t row = v / vec_per_row;
  const int c = (int)(v - row * vec_per_row) * N;
  const Vec<S> g = ldv<S>(gate + row * ld_g + c), u = ldv<S>(up + row * ld_u + c);
  Vec<S> o;
#pragma unroll
  for (int j = 0; j < N; ++j) {
    const float gf = S::to_float(g.e[j]);
    o.e[j] = S::from_float(gf / (1.0f + expf(-gf)) * S::to_float(u.e[j]));
  }
  stv<S>(out + row * ld_o + c, o);
}

bool aligned16(const void* p) { return ((uintptr_t)p & 15) == 0; }
int elem_bytes(int dtype) { return dtype == FLP_F32 ? 4 : 2; }

#define FLL_BY_DTYPE(dtype, CALL)          \
  do {                                     \
    if (dtype == FLP_F32) {                \
      typedef F32 S_;                      \
      CALL;                                \
    } else if (dtype == FLP_F16) {         \
      typedef F16 S_;                      \
      CALL;                                \
    } else {                               \
      typedef BF16 S_;                     \
      CALL;                                \
    }                                      \
  } while (0)

flp_status norm_common(int32_t dtype, const void* x, void* resid, const void* delta, const void* w, void* y, int32_t T,
                       int32_t H, float eps, void* hip_stream, const char* who) {
  if (dtype < FLP_F32 || dtype > FLP_BF16 || T < 0 || H <= 0 || (y && !w) || !aligned16(x) || !aligned16(resid) ||
      !aligned16(delta) || !aligned16(w) || !aligned16(y)) {
    flp_set_error("%s: bad dtype / sizes or null / misaligned pointer", who);
    return FLP_EINVAL;
  }
  if ((int64_t)H * elem_bytes(dtype) % 16) {
    flp_set_error("%s: a row of %d elements is not a multiple of 16 bytes", who, H);
    return FLP_ENOTSUP;
  }
  if (T == 0) return FLP_OK;
  hipStream_t st = (hipStream_t)hip_stream;
  const int64_t vecs = (int64_t)H * elem_bytes(dtype) / 16;         // 16-byte vectors per row
  const auto launch = [&](auto vectors, auto waves) {
    constexpr int NV = decltype(vectors)::value, W = decltype(waves)::value;
    FLL_BY_DTYPE(dtype, hipLaunchKernelGGL((rmsnorm_kernel<S_, NV, W>), dim3(W == 4 ? T : (T + 3) / 4), dim3(256), 0, st,
                                           (const S_::storage*)x, (S_::storage*)resid, (const S_::storage*)delta,
                                           (const S_::storage*)w, (S_::storage*)y, T, H, eps));
  };
  typedef std::integral_constant<int, 1> one;
  typedef std::integral_constant<int, 2> two;
  typedef std::integral_constant<int, 4> four;
  if (vecs <= 64)
    launch(one{}, one{});
  else if (vecs <= 96)   // 10000 rows of 1024: norm 15.2 with one wave, 16.7 with four, with residual 25.2, 23.6 us; with and without
                         // a residual the sum of squares is taken in one order
    launch(two{}, one{});
  else if (vecs <= 512)
    launch(two{}, four{});
  else if (vecs <= 1024)
    launch(four{}, four{});
  else
    FLL_BY_DTYPE(dtype, hipLaunchKernelGGL(rmsnorm_long_kernel<S_>, dim3((T + 3) / 4), dim3(256), 0, st,
                                           (const S_::storage*)x, (S_::storage*)resid, (const S_::storage*)delta,
                                           (const S_::storage*)w, (S_::storage*)y, T, H, eps));
  FLP_TRY_HIP(hipGetLastError());
  return FLP_OK;
}

}  // namespace

extern "C" flp_status fll_rmsnorm(int32_t dtype, const void* x, const void* w, void* y, int32_t n_tokens, int32_t hidden,
                                  float eps, void* hip_stream) {
  if (!x || !w || !y) {
    flp_set_error("fll_rmsnorm: null pointer");
    return FLP_EINVAL;
  }
  return norm_common(dtype, x, nullptr, nullptr, w, y, n_tokens, hidden, eps, hip_stream, "fll_rmsnorm");
}

extern "C" flp_status fll_add_rmsnorm(int32_t dtype, void* resid, const void* delta, const void* w, void* y,
                                      int32_t n_tokens, int32_t hidden, float eps, void* hip_stream) {
  if (!resid || !delta) {
    flp_set_error("fll_add_rmsnorm: null pointer");
    return FLP_EINVAL;
  }
  return norm_common(dtype, nullptr, resid, delta, w, y, n_tokens, hidden, eps, hip_stream, "fll_add_rmsnorm");
}

extern "C" flp_status fll_rope(int32_t dtype, void* q, void* k, const int32_t* positions, int32_t n_tokens,
                               int32_t n_q_heads, int32_t n_kv_heads, int32_t head_dim, float theta, void* hip_stream) {
  if (dtype < FLP_F32 || dtype > FLP_BF16 || n_tokens < 0 || !positions || (q && n_q_heads <= 0) ||
      (k && n_kv_heads <= 0) || !(theta > 0) || !aligned16(q) || !aligned16(k)) {
    flp_set_error("fll_rope: bad dtype / sizes / theta or null / misaligned pointer");
    return FLP_EINVAL;
  }
  if (head_dim != 64 && head_dim != 128) {
    flp_set_error("fll_rope: head_dim %d not supported (64 or 128)", head_dim);
    return FLP_ENOTSUP;
  }
  if (n_tokens == 0 || (!q && !k)) return FLP_OK;
  hipStream_t st = (hipStream_t)hip_stream;
  const double l2t = std::log2((double)theta);
  if (head_dim == 64)
    FLL_BY_DTYPE(dtype, hipLaunchKernelGGL((rope_kernel<S_, 64>), dim3(n_tokens), dim3(256), 0, st, (S_::storage*)q,
                                           (S_::storage*)k, positions, n_q_heads, n_kv_heads, l2t));
  else
    FLL_BY_DTYPE(dtype, hipLaunchKernelGGL((rope_kernel<S_, 128>), dim3(n_tokens), dim3(256), 0, st, (S_::storage*)q,
                                           (S_::storage*)k, positions, n_q_heads, n_kv_heads, l2t));
  FLP_TRY_HIP(hipGetLastError());
  return FLP_OK;
}

extern "C" flp_status fll_silu_mul(int32_t dtype, const void* gate, int64_t ld_gate, const void* up, int64_t ld_up,
                                   void* out, int64_t ld_out, int32_t n_tokens, int32_t width, void* hip_stream) {
  if (dtype < FLP_F32 || dtype > FLP_BF16 || n_tokens < 0 || width <= 0 || !gate || !up || !out || ld_gate < width ||
      ld_up < width || ld_out < width || !aligned16(gate) || !aligned16(up) || !aligned16(out)) {
    flp_set_error("fll_silu_mul: bad dtype / sizes or null / misaligned pointer");
    return FLP_EINVAL;
  }
  const int eb = elem_bytes(dtype);
  if ((int64_t)width * eb % 16 || ld_gate * eb % 16 || ld_up * eb % 16 || ld_out * eb % 16) {
    flp_set_error("fll_silu_mul: width and leading dimensions must be multiples of 16 bytes");
    return FLP_ENOTSUP;
  }
  if (n_tokens == 0) return FLP_OK;
  const int vpr = width * eb / 16;
  const int64_t n_vec = (int64_t)n_tokens * vpr;
  hipStream_t st = (hipStream_t)hip_stream;
  FLL_BY_DTYPE(dtype, hipLaunchKernelGGL(silu_mul_kernel<S_>, dim3((unsigned)((n_vec + 255) / 256)), dim3(256), 0, st,
                                         (const S_::storage*)gate, ld_gate, (const S_::storage*)up, ld_up,
                                         (S_::storage*)out, ld_out, n_vec, vpr));
  FLP_TRY_HIP(hipGetLastError());
  return FLP_OK;
}

// ------------------------------------------------------------------------------- the layer
namespace {
struct Scratch {
  size_t n, q, k, v, attn, proj, gate, up, total;
};
Scratch layout(const flp_pool* p, const fll_layer_config* c, int64_t T) {
  const int64_t eb = p->elem_bytes, d = p->cfg.head_dim;
  auto al = [](int64_t b) { return (size_t)((b + 255) & ~(int64_t)255); };
  Scratch s{};
  size_t off = 0;
  auto take = [&](int64_t bytes) {
    const size_t o = off;
    off += al(bytes);
    return o;
  };
  s.n = take(T * c->hidden * eb);
  s.q = take(T * c->n_q_heads * d * eb);
  s.k = take(T * p->cfg.n_kv_heads * d * eb);
  s.v = take(T * p->cfg.n_kv_heads * d * eb);
  s.attn = take(T * c->n_q_heads * d * eb);
  s.proj = take(T * c->hidden * eb);
  s.gate = take(T * c->mlp_dim * eb);
  s.up = take(T * c->mlp_dim * eb);
  s.total = off;
  return s;
}
bool cfg_ok(const flp_pool* p, const fll_layer_config* c) {
  return p && c && c->hidden > 0 && c->n_q_heads > 0 && c->mlp_dim > 0 && c->n_q_heads % p->cfg.n_kv_heads == 0;
}

// How many of T tokens a large product takes in whole rounds of 256 x 256 tiles, one per CU; the rest, less than a round, follows
// in a launch (with LoRA: a call) of its own, on smaller tiles and in slices.  T where the planner sees no gain in that: the last
// round of a launch lasts two thirds of a full one however few tiles it has.  extra_us: what the second call costs beside its
// product.  Layers, one launch and two, us:
//   4400 tokens, 7B shapes     2059   1868      8300 tokens    3528   3201
//   2200 tokens, 34B shapes    3230   2960      4300 tokens    5665   5263
//   3300 tokens, 13B shapes    2326   2145      9874 tokens    6673   6454      5000 tokens    3496   3491 (one launch, mostly)
// Where the last tokens are single ones with an adapter each, the rest's own call spares the large product tiles with many adapters:
// 156 layers of 2100-8400 tokens, 60-250 of them such, ranks 16 and 64, 0.97 of the time without the cut (0.84 to 1.04).  (The price
// of a rest with LoRA is that of the small batches' steps, which it takes below 1024 tokens.)
constexpr double kRestUs = 4, kLoraRestUs = 30;        // a launch; the two launches of the branch and the base's way through memory
int32_t whole_rounds(int T, int K, int n, const int* N, bool lora, double extra_us) {
  int64_t f_tiles = 0;
  bool fits = K % 64 == 0;                              // widths that the LoRA branch's tiles divide: it runs inside the large product
  for (int i = 0; i < n; ++i) {
    f_tiles += (N[i] + 255) / 256;
    fits = fits && (!lora || N[i] % 64 == 0);
  }
  const int64_t rounds = f_tiles * ((T + 255) / 256) / 256;
  const int64_t first = rounds < 1 ? 0 : 256 * (256 * rounds / f_tiles), rest = T - first;
  if (!fits || first < 2048 || rest < 1 || rest > 1024) return T;
  const unsigned allow = lora ? FLP_GEMM_NO_SPLIT | FLP_GEMM_LARGE_ONLY : 0;
  const size_t room = kLayerSliceBytes;
  const double whole = flp_gemm_plan(T, K, n, N, allow, room).us;
  const double parts = flp_gemm_plan((int)first, K, n, N, allow, room).us + flp_gemm_plan((int)rest, K, n, N, 0, room).us + extra_us;
  return parts < 0.98 * whole ? (int32_t)first : T;
}

// Dense products of the T tokens from token `at` on, in one launch (and one that adds the slices).  Slices of a small batch's
// contraction live in the pool's workspace (stream order keeps them apart from the LoRA intermediates of the calls before and
// after).  Larger batches without LoRA needed no workspace before they were sliced, so calls on several streams owe each other no
// order: their slices, those of their last tokens among them, have a workspace of their own that one call hands to the next, for an
// event per product (products of 100 us and more; the small ones would notice it).
constexpr int kSharedWorkTokens = 1024;
// batch: the tokens of the whole call
flp_status dense_launch(flp_pool* p, const void* x, int d_in, int at, int T, int batch, int n, const FlpGemmOut* whole, const int* N,
                        bool gated, hipStream_t stream, void* resid, bool* added) {
  const void* const x_at = (const uint8_t*)x + (int64_t)at * d_in * p->elem_bytes;
  FlpGemmOut out[3];
  for (int i = 0; i < n; ++i) {
    out[i] = whole[i];
    out[i].y = (uint8_t*)whole[i].y + (int64_t)at * whole[i].ld_y * p->elem_bytes;
  }
  const FlpGemmPlan plan = flp_gemm_plan(T, d_in, n, N, 0, kLayerSliceBytes);
  const bool own = plan.splits > 1 && batch > kSharedWorkTokens;
  std::unique_lock<std::mutex> lk(p->mu, std::defer_lock);
  if (plan.splits > 1) {
    void* part = nullptr;
    lk.lock();
    if (own)
      FLP_TRY(flp_dense_workspace_acquire(p, flp_gemm_part_bytes(plan, T, n, N), stream, &part));
    else
      FLP_TRY(flp_workspace(p, flp_gemm_part_bytes(plan, T, n, N), &part));
    float* f = (float*)part;
    for (int i = 0; i < n; ++i) {
      out[i].part = f;
      f += (size_t)plan.splits * T * N[i];
    }
  }
  flp_status s = flp_launch_gemm(p->cfg.dtype, x_at, d_in, T, d_in, plan, n, out, gated, nullptr, stream);
  if (s == FLP_OK && plan.splits > 1) {
    if (resid) {
      out->y = resid;
      *added = true;
    }
    s = flp_launch_gemm_reduce(p->cfg.dtype, T, n, out, plan.splits, gated, resid ? FLP_REDUCE_ADD : FLP_REDUCE_PLAIN, stream);
  }
  if (own) {
    const flp_status r = flp_dense_workspace_release(p, stream);
    return s != FLP_OK ? s : r;
  }
  return s;
}

// Dense products alone (gated: the gated-SiLU pair as one output).  `resid`, one product: where its slices are added by a kernel,
// that kernel adds the rounded result to the residual stream instead of writing out->y, and *added says so.
flp_status dense_products(flp_pool* p, const void* x, int d_in, int T, int n, const FlpGemmOut* out, const int* N, bool gated,
                          hipStream_t stream, void* resid = nullptr, bool* added = nullptr) {
  if (p->elem_bytes == 4) {
    for (int i = 0; i < n; ++i)
      FLP_TRY(flp_launch_gemm_f32((const float*)x, d_in, (const float*)out[i].w, 1, (float*)out[i].y, out[i].ld_y, T, N[i], d_in,
                                  stream));
    return FLP_OK;
  }
  // Cut once: the planner, asked for the first part alone, may see a gain in cutting that as well (K 28672, N 35840: 2564 tokens,
  // 2560, 2304).
  const int32_t first = whole_rounds(T, d_in, n, N, false, kRestUs);
  if (first == T) return dense_launch(p, x, d_in, 0, T, T, n, out, N, gated, stream, resid, added);
  FLP_TRY(dense_launch(p, x, d_in, 0, first, T, n, out, N, gated, stream, nullptr, nullptr));
  return dense_launch(p, x, d_in, first, T - first, T, n, out, N, gated, stream, nullptr, nullptr);
}
}  // namespace

// whole_rounds for tests that state where a shape is cut
extern "C" int32_t flp_dense_first_tokens(int32_t T, int32_t K, int32_t n, const int32_t* N, int32_t lora) {
  return whole_rounds(T, K, n, N, lora != 0, lora ? kLoraRestUs : kRestUs);
}

extern "C" int64_t fll_layer_scratch_bytes(const flp_pool* pool, const fll_layer_config* cfg, int32_t n_tokens) {
  if (!cfg_ok(pool, cfg) || n_tokens < 0) return -1;
  return (int64_t)layout(pool, cfg, n_tokens).total;
}

extern "C" flp_status fll_layer_forward(flp_pool* p, const fll_layer_config* c, const fll_layer_weights* w,
                                        const fll_layer_batch* b, void* h, void* scratch, int64_t scratch_bytes,
                                        void* hip_stream) {
  if (!cfg_ok(p, c) || !w || !b || !h || !scratch || b->n_tokens < 0 || b->n_seqs < 0) {
    flp_set_error("fll_layer_forward: null argument or bad layer shape");
    return FLP_EINVAL;
  }
  if (!w->in_norm || !w->post_norm || !w->wq || !w->wk || !w->wv || !w->wo || !w->w_gate || !w->w_up || !w->w_down) {
    flp_set_error("fll_layer_forward: a weight pointer is null");
    return FLP_EINVAL;
  }
  const int32_t T = b->n_tokens;
  if (T == 0) return FLP_OK;
  // the direct global-to-LDS loads of the 16-bit products drop the low bits of a misaligned address without an error
  for (const void* m : {w->wq, w->wk, w->wv, w->wo, w->w_gate, w->w_up, w->w_down})
    if (p->elem_bytes == 2 && ((uintptr_t)m & 15)) {
      flp_set_error("fll_layer_forward: a weight matrix is not 16-byte aligned");
      return FLP_EINVAL;
    }
  const Scratch s = layout(p, c, T);
  if (((uintptr_t)scratch & 255) || scratch_bytes < (int64_t)s.total) {
    flp_set_error("fll_layer_forward: scratch misaligned or smaller than %lld bytes", (long long)s.total);
    return FLP_EINVAL;
  }
  const int dtype = p->cfg.dtype, d = p->cfg.head_dim, n_kv = p->cfg.n_kv_heads;
  const int Hq = c->n_q_heads * d, Hkv = n_kv * d, H = c->hidden, M = c->mlp_dim;
  const float eps = c->rms_eps > 0 ? c->rms_eps : 1e-5f, theta = c->rope_theta > 0 ? c->rope_theta : 10000.0f;
  uint8_t* sb = (uint8_t*)scratch;
  void *n = sb + s.n, *q = sb + s.q, *k = sb + s.k, *v = sb + s.v, *attn = sb + s.attn, *proj = sb + s.proj,
       *gate = sb + s.gate, *up = sb + s.up;

  // base GEMM + LoRA branch of up to three projections that share their input
  auto project = [&](const void* x, int d_in, int n_proj, const int* which, void* const* ys, const int* d_outs,
                     const void* const* ws, void* gated_out = nullptr, bool* added = nullptr) -> flp_status {
    flp_lora_batch lb{};
    lb.n_tokens = T;
    lb.d_in = d_in;
    lb.ld_x = d_in;
    lb.n_adapters = b->n_adapters;
    lb.max_rank = b->max_rank;
    lb.n_proj = n_proj;
    lb.x = x;
    lb.token_adapter = b->token_adapter;
    lb.rank = b->rank;
    lb.scale = b->scale;
    lb.block_tables = b->lora_tables;
    int n_lora = 0, n_dense = 0, dense_N[3];
    FlpGemmOut dense[3] = {};
    for (int i = 0; i < n_proj; ++i) {
      const fll_lora_place& pl = b->lora[which[i]];
      const int n_set = (pl.a_tab_off != nullptr) + (pl.a_row_base != nullptr) + (pl.b_tab_off != nullptr) +
                        (pl.b_row_base != nullptr);
      if (n_set == 0) {                               // no LoRA branch on this projection: the dense product alone
        if (p->elem_bytes == 2 && d_in % 64) {
          flp_set_error("fll_layer_forward: projection %d: d_in %d is not a multiple of 64", which[i], d_in);
          return FLP_ENOTSUP;
        }
        dense[n_dense].w = ws[i];
        dense[n_dense].y = ys[i];
        dense[n_dense].ld_y = d_outs[i];
        dense[n_dense].N = dense_N[n_dense] = d_outs[i];
        ++n_dense;
        continue;
      }
      if (n_set != 4) {
        flp_set_error("fll_layer_forward: projection %d has an incomplete LoRA placement", which[i]);
        return FLP_EINVAL;
      }
      flp_lora_proj& pr = lb.proj[n_lora++];
      pr.d_out = d_outs[i];
      pr.w_base_layout = 1;
      pr.ld_y = d_outs[i];
      pr.y = ys[i];
      pr.w_base = ws[i];
      pr.a_tab_off = pl.a_tab_off;
      pr.a_row_base = pl.a_row_base;
      pr.b_tab_off = pl.b_tab_off;
      pr.b_row_base = pl.b_row_base;
    }
    if (n_dense > 0)
      FLP_TRY(dense_products(p, x, d_in, T, n_dense, dense, dense_N, false, (hipStream_t)hip_stream,
                             added && n_proj == 1 ? h : nullptr, added));
    if (n_lora == 0) return FLP_OK;
    lb.n_proj = n_lora;
    if (gated_out) return flp_lora_apply_gated(p, &lb, FlpSequences{b->cu_new, b->n_seqs, 0}, gated_out, d_outs[0], hip_stream);
    int N[3];
    for (int i = 0; i < n_lora; ++i) N[i] = lb.proj[i].d_out;
    const int32_t first = p->elem_bytes == 2 ? whole_rounds(T, d_in, n_lora, N, true, kLoraRestUs) : T;
    lb.n_tokens = first;
    FLP_TRY(flp_lora_apply_layer(p, &lb, FlpSequences{b->cu_new, b->n_seqs, 0}, hip_stream));
    if (first == T) return FLP_OK;
    lb.n_tokens = T - first;
    lb.x = (const uint8_t*)x + (int64_t)first * d_in * p->elem_bytes;
    lb.token_adapter = b->token_adapter + first;
    for (int i = 0; i < n_lora; ++i) lb.proj[i].y = (uint8_t*)lb.proj[i].y + (int64_t)first * lb.proj[i].ld_y * p->elem_bytes;
    return flp_lora_apply_layer(p, &lb, FlpSequences{b->cu_new, b->n_seqs, first}, hip_stream);
  };

  FLP_TRY(fll_rmsnorm(dtype, h, w->in_norm, n, T, H, eps, hip_stream));
  {
    const int which[3] = {0, 1, 2}, d_outs[3] = {Hq, Hkv, Hkv};
    void* const ys[3] = {q, k, v};
    const void* const ws[3] = {w->wq, w->wk, w->wv};
    FLP_TRY(project(n, H, 3, which, ys, d_outs, ws));
  }
  FLP_TRY(fll_rope(dtype, q, k, b->positions, T, c->n_q_heads, n_kv, d, theta, hip_stream));
  {
    flp_attn_batch ab{};
    ab.n_seqs = b->n_seqs;
    ab.n_q_heads = c->n_q_heads;
    ab.max_blocks_per_seq = b->max_blocks_per_seq;
    ab.sm_scale = 0.f;
    ab.q = q;
    ab.k_new = k;
    ab.v_new = v;
    ab.out = attn;
    ab.cu_new = b->cu_new;
    ab.prefix_len = b->prefix_len;
    ab.block_tables = b->kv_tables;
    FLP_TRY(flp_paged_prefix_attention(p, &ab, hip_stream));
  }
  {
    const int which[1] = {3}, d_outs[1] = {H};
    void* const ys[1] = {proj};
    const void* const ws[1] = {w->wo};
    FLP_TRY(project(attn, Hq, 1, which, ys, d_outs, ws));
  }
  FLP_TRY(fll_add_rmsnorm(dtype, h, proj, w->post_norm, n, T, H, eps, hip_stream));
  {
    // without LoRA branches on gate and up the two products and the gate are one step that writes only silu(g) * u;
    // with branches on both that holds for large batches; otherwise two products and the element-wise step
    const auto no_lora = [&](int i) {
      const fll_lora_place& pl = b->lora[i];
      return !pl.a_tab_off && !pl.a_row_base && !pl.b_tab_off && !pl.b_row_base;
    };
    const auto full_lora = [&](int i) {
      const fll_lora_place& pl = b->lora[i];
      return pl.a_tab_off && pl.a_row_base && pl.b_tab_off && pl.b_row_base;
    };
    const int which[2] = {4, 5}, d_outs[2] = {M, M};
    void* const ys[2] = {gate, up};
    const void* const ws[2] = {w->w_gate, w->w_up};
    flp_status fused = FLP_ENOTSUP;
    if (no_lora(4) && no_lora(5) && p->elem_bytes == 2 && H % 64 == 0 && M % 32 == 0) {
      const int N[1] = {2 * M};
      FlpGemmOut o{};
      o.w = w->w_gate;
      o.w2 = w->w_up;
      o.y = gate;
      o.ld_y = M;
      o.N = N[0];
      fused = dense_products(p, n, H, T, 1, &o, N, true, (hipStream_t)hip_stream);
    }
    else if (full_lora(4) && full_lora(5))          // both with a LoRA branch: the branches are added inside the same pass
      fused = project(n, H, 2, which, ys, d_outs, ws, gate);
    if (fused == FLP_ENOTSUP) {
      FLP_TRY(project(n, H, 2, which, ys, d_outs, ws));
      FLP_TRY(fll_silu_mul(dtype, gate, M, up, M, gate, M, T, M, hip_stream));
    } else if (fused != FLP_OK) {
      return fused;
    }
  }
  {
    const int which[1] = {6}, d_outs[1] = {H};
    void* const ys[1] = {proj};
    const void* const ws[1] = {w->w_down};
    bool added = false;
    FLP_TRY(project(gate, M, 1, which, ys, d_outs, ws, nullptr, &added));
    if (added) return FLP_OK;
  }
  return fll_add_rmsnorm(dtype, h, proj, nullptr, nullptr, T, H, eps, hip_stream);
}
