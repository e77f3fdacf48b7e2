// One wave's share of paged attention of single new tokens: see attention_decode.hip, whose kernel launches nothing else, and
// attention_mfma.hip, whose mixed launches run such waves beside the tiles.
#pragma once
#include <hip/hip_runtime.h>

#include <type_traits>

#include "flp_internal.h"
#include "flp_types.h"

namespace flp_decode {

constexpr int D = 128;
constexpr int BT = 16;
constexpr int kChains = 4;                             // independent sums that hide a matrix instruction's latency

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef _Float16 h16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 b16x8 __attribute__((ext_vector_type(8)));

struct DF16 {
  typedef h16x8 vec;
  typedef _Float16 el;
  typedef F16 S;
  static constexpr float kScale = 32768.f, kStep = 2048.f;      // of the weights, and from one of their pieces to the next
  static __device__ __forceinline__ f32x4 mfma(vec a, vec b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ float widen(uint32_t two, int odd) {      // one of the two values of a word
    return F16::to_float((uint16_t)(odd ? two >> 16 : two));
  }
};
struct DBF16 {
  typedef b16x8 vec;
  typedef __bf16 el;
  typedef BF16 S;
  static constexpr float kScale = 65536.f, kStep = 1.f;
  static __device__ __forceinline__ f32x4 mfma(vec a, vec b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ float widen(uint32_t two, int odd) {
    return __uint_as_float(odd ? two & 0xffff0000u : two << 16);
  }
};

template <typename V>
__device__ __forceinline__ V as_vec(u32x4 r) {
  V v;
  __builtin_memcpy(&v, &r, 16);
  return v;
}

struct Tile {                    // K and V of 32 positions
  u32x4 k[2][4], v[8];
};

// One wave: the query heads of kv head g of one unit
template <typename M>
__device__ __forceinline__ void decode_unit(const FlpAttnArgs& a, const FlpAttnUnit u, int g) {
  typedef typename M::vec vec;
  const int lane = threadIdx.x & 63;
  const int lr = lane & 15, lh = lane >> 4;
  const int G = a.n_h / a.n_kv;
  const int t = u.t, ctx = u.ctx;                      // positions 0 .. ctx - 1 are visible
  const int g_lo = u.g_lo, g_hi = u.g_hi;              // this piece: groups [g_lo, g_hi) of 16 positions
  const int lim = BT * g_hi < ctx ? BT * g_hi : ctx;
  const int bt = a.bt, hsh = bt / BT - 1;              // a block holds 1 << hsh groups
  const int32_t* __restrict__ table = a.tables + (int64_t)u.seq * a.max_blocks;
  const uint16_t* __restrict__ pool = reinterpret_cast<const uint16_t*>(a.pool);
  const float c = a.scale_log2e;

  const int h = g * G + (lr < G ? lr : G - 1);         // this lane's query head
  const int64_t rowoff = ((int64_t)t * a.n_h + h) * D;
  vec qf[4];
#pragma unroll
  for (int kk = 0; kk < 4; ++kk)
    qf[kk] = as_vec<vec>(*reinterpret_cast<const u32x4*>(reinterpret_cast<const uint16_t*>(a.q) + rowoff + 32 * kk + 8 * lh));

  // K: lane row m = lr is key 8 (m / 4) + 4 t + m % 4, chunk lh of its channels; V^T: channel lr of a tile of 16, run
  // of positions 8 lh ... + 7
  const int ksel = lr >> 3, vsel = lh >> 1;            // which of the two groups the lane's K row / V run lies in
  const int krow = 8 * ((lr >> 2) & 1) + (lr & 3);
  const int64_t k_lane = ((int64_t)g * bt + krow) * D + 8 * lh;
  const int64_t v_lane = (int64_t)a.n_kv * bt * D + ((int64_t)g * D + lr) * bt + 8 * (lh & 1);
  auto group = [&](int tile, int sel) {                // clamped: an odd run's last tile reads its last group twice
    const int gi = g_lo + 2 * tile + sel;
    return gi < g_hi ? gi : g_hi - 1;
  };
  auto load = [&](Tile& T, int tile, int32_t idk, int32_t idv) {
    const uint16_t* kp = pool + (int64_t)idk * a.block_elems + k_lane + BT * (group(tile, ksel) & hsh) * D;
    const uint16_t* vp = pool + (int64_t)idv * a.block_elems + v_lane + BT * (group(tile, vsel) & hsh);
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) T.k[s][kk] = *reinterpret_cast<const u32x4*>(kp + 4 * s * D + 32 * kk);
#pragma unroll
    for (int ct = 0; ct < 8; ++ct) T.v[ct] = *reinterpret_cast<const u32x4*>(vp + (int64_t)16 * ct * bt);
  };

  f32x4 O[8];
  float m, l;                                          // m: running maximum; l: this lane's share of the sum

  auto multiply = [&](Tile& T, int tile, auto pieces) {
    constexpr bool PIECES = decltype(pieces)::value;
    f32x4 s[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      s[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) s[i] = M::mfma(as_vec<vec>(T.k[i][kk]), qf[kk], s[i]);
    }
    const int pos0 = BT * (g_lo + 2 * tile) + 8 * lh;
    float p[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) p[e] = s[e >> 2][e & 3] * c;
    if (BT * (g_lo + 2 * tile) + 32 > lim) {           // wave-uniform: only the last tile of a piece
      // slots past the context hold arbitrary bits: their scores and their V are replaced, never multiplied
#pragma unroll
      for (int e = 0; e < 8; ++e) p[e] = pos0 + e < lim ? p[e] : -INFINITY;
#pragma unroll
      for (int ct = 0; ct < 8; ++ct)
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          const uint32_t mask = (pos0 + 2 * w < lim ? 0xffffu : 0u) | (pos0 + 2 * w + 1 < lim ? 0xffff0000u : 0u);
          T.v[ct][w] &= mask;
        }
    }
    float mx = p[0];
#pragma unroll
    for (int e = 1; e < 8; ++e) mx = fmaxf(mx, p[e]);
    mx = fmaxf(mx, __shfl_xor(mx, 16));
    mx = fmaxf(mx, __shfl_xor(mx, 32));
    if (__builtin_amdgcn_ballot_w64(mx > m)) {         // some row's maximum grew
      const float mn = fmaxf(m, mx);
      const float alpha = exp2f(m - mn);               // 0 on the first tile (m = -inf)
      m = mn;
      l *= alpha;
#pragma unroll
      for (int ct = 0; ct < 8; ++ct)
#pragma unroll
        for (int i = 0; i < 4; ++i) O[ct][i] *= alpha;
    }
    // a tile's sums are taken by themselves, its small terms first, and then added: one rounding of the running sum per tile
    float w[8], lw = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      w[e] = exp2f(p[e] - m) * (PIECES ? M::kScale : 1.f);
      lw += w[e];
    }
    l += lw;
    vec piece[3];                                      // the weights are piece[0] + (piece[1] + piece[2] / kStep) / kStep
    if constexpr (PIECES)
#pragma unroll
      for (int e = 0; e < 8; ++e)
#pragma unroll
        for (int i = 0; i < 3; ++i) {
          piece[i][e] = (typename M::el)w[e];
          w[e] = (w[e] - (float)piece[i][e]) * M::kStep;
        }
#pragma unroll
    for (int ct0 = 0; ct0 < 8; ct0 += kChains) {
      f32x4 sum[kChains];
#pragma unroll
      for (int k = 0; k < kChains; ++k) sum[k] = f32x4{0.f, 0.f, 0.f, 0.f};
      if constexpr (PIECES) {
#pragma unroll
        for (int i = 2; i >= 0; --i)
#pragma unroll
          for (int k = 0; k < kChains; ++k) {
            sum[k] = M::mfma(as_vec<vec>(T.v[ct0 + k]), piece[i], sum[k]);
            if (i > 0 && M::kStep != 1.f)
#pragma unroll
              for (int j = 0; j < 4; ++j) sum[k][j] *= 1.f / M::kStep;
          }
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e)
#pragma unroll
          for (int k = 0; k < kChains; ++k) {
            const float v = M::widen(T.v[ct0 + k][e >> 1], e & 1);
            sum[k] = __builtin_amdgcn_mfma_f32_16x16x4f32(v, w[e], sum[k], 0, 0, 0);
          }
      }
#pragma unroll
      for (int k = 0; k < kChains; ++k)
#pragma unroll
        for (int i = 0; i < 4; ++i) O[ct0 + k][i] += sum[k][i];
    }
  };

  // Block ids are requested one tile ahead of the loads that use them, and before the loads of the tile in between, so
  // that waiting for them leaves those in flight.
  const int n_tiles = (g_hi - g_lo + 1) >> 1;
  auto id = [&](int tile, int sel) { return table[group(tile, sel) >> hsh]; };
  auto walk = [&](auto pieces) {
#pragma unroll
    for (int ct = 0; ct < 8; ++ct) O[ct] = f32x4{0.f, 0.f, 0.f, 0.f};
    m = -INFINITY;
    l = 0.f;
    int32_t idk = id(0, ksel), idv = id(0, vsel);
    int32_t idk1 = id(1, ksel), idv1 = id(1, vsel);
    Tile T0, T1;
    load(T0, 0, idk, idv);
    for (int tile = 0; tile < n_tiles; tile += 2) {
      idk = id(tile + 2, ksel);
      idv = id(tile + 2, vsel);
      load(T1, tile + 1, idk1, idv1);                  // past the end: the last group again (in cache), not used
      __builtin_amdgcn_sched_barrier(0);
      multiply(T0, tile, pieces);
      __builtin_amdgcn_sched_barrier(0);
      if (tile + 1 >= n_tiles) break;
      idk1 = id(tile + 3, ksel);
      idv1 = id(tile + 3, vsel);
      load(T0, tile + 2, idk, idv);
      __builtin_amdgcn_sched_barrier(0);
      multiply(T1, tile + 1, pieces);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  walk(std::true_type{});
  bool finite = true;                                  // an infinite V never leaves a finite sum: even 0 x inf is NaN
  l *= 1.f / M::kScale;
#pragma unroll
  for (int ct = 0; ct < 8; ++ct)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      finite = finite && fabsf(O[ct][i]) < INFINITY;
      O[ct][i] *= 1.f / M::kScale;
    }
  if (__builtin_amdgcn_ballot_w64(!finite)) walk(std::false_type{});

  l += __shfl_xor(l, 16);
  l += __shfl_xor(l, 32);
  if (lr >= G) return;
  // lane (row lr, quarter lh) holds channels 16 ct + 4 lh + (0..3)
  if (u.part >= 0) {
    float* pp = a.partials + ((int64_t)u.part * a.n_h + h) * (D + 2);
    if (lh == 0) *reinterpret_cast<float2*>(pp) = make_float2(m, l);
#pragma unroll
    for (int ct = 0; ct < 8; ++ct) {
      float2* o = reinterpret_cast<float2*>(pp + 2 + 16 * ct + 4 * lh);
      o[0] = make_float2(O[ct][0], O[ct][1]);
      o[1] = make_float2(O[ct][2], O[ct][3]);
    }
    return;
  }
  const float inv = 1.f / l;
  uint16_t* op = reinterpret_cast<uint16_t*>(a.out) + rowoff;
#pragma unroll
  for (int ct = 0; ct < 8; ++ct) {
    uint16_t o4[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) o4[i] = M::S::from_float(O[ct][i] * inv);
    uint2 w;
    __builtin_memcpy(&w, o4, 8);
    *reinterpret_cast<uint2*>(op + 16 * ct + 4 * lh) = w;
  }
}

}  // namespace flp_decode
