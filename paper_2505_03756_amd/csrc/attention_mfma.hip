// Paged prefix attention on the matrix cores, for 16-bit pools with head_dim 128.
//
// Same definition as the row-streaming kernel (paper sections 2.1 / 4.2: the new tokens of
// a query attend over the reused prefix KV and their own fresh KV, read through the block
// table), organised as a tiled online-softmax so that K and V are read once per tile of
// query rows instead of once per row.
//
// One workgroup (8 waves, one per CU) owns up to 256 query rows of one (sequence, kv head); row r
// is (new token r / G, query head g*G + r % G), so the G query heads that share a kv head
// sit in the same tile and K/V are read once for all of them.  It walks the context in
// tiles of 64 positions (4 pool blocks).
//
// The products are computed transposed, S^T = K Q^T and O^T = V^T P^T, with mfma_f32_16x16x32: a lane holds one query
// row (column l % 16) of each of the wave's two row tiles, and with the keys of a 32-key group fed in the order
// key(m) = 8 (m / 4) + 4 t + m % 4 for row m of key tile t it holds the weights of 8 consecutive positions, which is the
// B-operand layout of the second product and also its 16-byte run of the transposed V of a pool block.  The row maximum
// is only exchanged between lanes when it has to be raised.
//
// Long launches are bound by the power the chip may draw, so what counts is energy per tile: with 32x32x16 instructions,
// which read and write twice the accumulator registers per product, the same loop held a lower clock (64 sequences of
// 4096 + 512 positions, 64 / 8 heads, bf16: 4.36 ms, now 4.07; with all operands zero, where power does not limit, 3.56
// and 3.55 ms).  A software pipeline inside a wave (the scores of tile t + 1 between the exponentials of tile t, 244
// registers) was 3-8 % slower.  Batches of prefill, or prefill and decode, attention alone:
//   64 sequences, prefixes to 2 k, 128-512 new tokens, 32 / 32 heads, fp16       756 -> 716 us
//   128 sequences, prefixes to 4 k, 40 / 40 heads, fp16                          2984 -> 2836 us
//   512 sequences, contexts to 16 k, a quarter prefill, 64 / 8 heads, bf16       15.33 -> 14.61 ms
//
// K/V tiles travel from the pool to LDS with the direct global-to-LDS loads of gfx950
// (16 bytes per lane, landing at LDS base + 16 * lane): no registers and no LDS stores are
// spent on staging, and a ring of three tiles keeps two tiles in flight behind the one being
// multiplied.  The XOR swizzle of the LDS layout is applied on the global side: a lane
// fetches the 16-byte chunk that belongs at its fixed LDS slot.  A wave issues one
// instruction about every 4.5 cycles whatever its kind, and LDS reads take a few hundred
// cycles under load, so operand fragments are read two steps ahead of the products that use them (the steps of the scores are
// fenced: unfenced, the compiler moved every read of K down to its product; 64 sequences of 4096 + 512 positions zeroed 3540 ->
// 3465 us, drawn 4247 -> 4188), the next tile is
// requested from between the products of the scores, and the exponentials are spread between those of the second product
// (2.5 % of the batches above).
#include <hip/hip_runtime.h>

#include "attention_decode_wave.h"
#include "flp_internal.h"
#include "flp_types.h"

namespace {

constexpr int D = 128;
constexpr int BT = 16;
constexpr int BN = 64;                 // keys per tile
constexpr int kTile = BN * D * 2;      // bytes of one K (or V) tile: 16 KiB
constexpr int kStage = 2 * kTile;      // K tile followed by V tile
constexpr int kStages = 3;             // tiles in the LDS ring: one being multiplied, kStages - 1 in flight

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef _Float16 h16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 b16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 h16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 b16x2 __attribute__((ext_vector_type(2)));

struct MF16 {
  typedef h16x8 vec;
  typedef flp_decode::DF16 Single;
  static __device__ __forceinline__ f32x4 mfma(vec a, vec b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
  }
  // 8 weights -> 16 bit; adds their sum as seen after rounding
  static __device__ __forceinline__ vec pack(const float* p, float& sum) {
    vec v;
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = (_Float16)p[j];
    const h16x2 one = {(_Float16)1.f, (_Float16)1.f};
#pragma unroll
    for (int j = 0; j < 4; ++j) sum = __builtin_amdgcn_fdot2(h16x2{v[2 * j], v[2 * j + 1]}, one, sum, false);
    return v;
  }
  static __device__ __forceinline__ uint16_t out(float f) { return F16::from_float(f); }
};
struct MBF16 {
  typedef b16x8 vec;
  typedef flp_decode::DBF16 Single;
  static __device__ __forceinline__ f32x4 mfma(vec a, vec b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ vec pack(const float* p, float& sum) {
    vec v;
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = (__bf16)p[j];
    const b16x2 one = {(__bf16)1.f, (__bf16)1.f};
#pragma unroll
    for (int j = 0; j < 4; ++j) sum = __builtin_amdgcn_fdot2_f32_bf16(b16x2{v[2 * j], v[2 * j + 1]}, one, sum, false);
    return v;
  }
  static __device__ __forceinline__ uint16_t out(float f) { return BF16::from_float(f); }
};

template <typename V>
__device__ __forceinline__ V as_vec(u32x4 r) {
  V v;
  __builtin_memcpy(&v, &r, 16);
  return v;
}

// XOR term of the K row swizzle: the key's row of its A operand
__device__ __forceinline__ int k_swz(int key32) { return ((key32 >> 3) << 2) | (key32 & 3); }
__device__ __forceinline__ int v_swz(int d) { return ((d >> 2) & 1) ^ ((d >> 3) & 1); }

// s_waitcnt immediates (gfx9 encoding: vmcnt[3:0] + [15:14], expcnt[6:4], lgkmcnt[11:8]), other counters untouched
constexpr int kWaitTile = (4 * (kStages - 2)) | (7 << 4) | (15 << 8);   // all but the newest kStages - 2 tiles (4 loads each) have landed
constexpr int kScheduleAlu = 6;        // __builtin_amdgcn_sched_barrier: vector and scalar arithmetic may cross
constexpr int kWaitVm0 = 0 | (7 << 4) | (15 << 8);

// One direct global-to-LDS load: every lane fetches 16 bytes from base + voff and the wave's 64
// pieces land at LDS byte address lds .. lds + 1023 in lane order (base and lds wave-uniform).
// Written as inline assembly on purpose: the compiler does not see these loads, so it neither
// counts them in its own memory-counter waits nor makes every later LDS read wait for all of
// them; the kernel orders them against the LDS reads itself (s_waitcnt vmcnt + barrier).
// M0 is named as clobbered so that no pass keeps a value of its own alive in it across the statement; the
// compiler notes that it reserves the register, which is the point.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void load_to_lds16(const void* base, uint32_t voff, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(voff), "s"(base), "s"(lds)
               : "memory", "m0");
}
#pragma clang diagnostic pop
typedef __attribute__((address_space(3))) uint8_t lds_u8;

template <typename M>
__global__ __launch_bounds__(512, 2) void attn_mfma_kernel(FlpAttnArgs a, const FlpMfmaItem* __restrict__ items,
                                                               const FlpAttnUnit* __restrict__ units) {
  typedef typename M::vec vec;
  __shared__ __attribute__((aligned(16))) uint8_t smem[kStages * kStage];
  __shared__ int32_t tab_lds[kMfmaMaxBlocks];          // this sequence's block table

  const FlpMfmaItem it = items[blockIdx.x];
  if (it.n_rows == 0) return;
  const int tid = threadIdx.x, lane = tid & 63, lr = lane & 15, lh = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  if (it.n_rows < 0) {                                 // single tokens: (unit, kv head) pairs r0 .. r0 + 7 of `seq`
    const int pair = it.r0 + wave;
    if (pair < it.seq) flp_decode::decode_unit<typename M::Single>(a, units[pair / a.n_kv], pair % a.n_kv);
    return;                                            // waves share nothing
  }
  const int G = a.n_h / a.n_kv, g = it.g;
  const int P = a.prefix_len[it.seq];
  const int t0 = a.cu_new[it.seq];
  const int N = a.cu_new[it.seq + 1] - t0;
  const int L = P + N;
  const int bt = a.bt, hsh = bt / BT - 1;             // a block holds 1 << hsh groups of 16 positions
  const int ngrp_valid = (L + BT - 1) / BT;           // groups of 16 positions that hold keys of this sequence
  const int nblk_valid = (L + bt - 1) / bt;
  const int32_t* __restrict__ table = a.tables + (int64_t)it.seq * a.max_blocks;
  const uint16_t* __restrict__ pool = reinterpret_cast<const uint16_t*>(a.pool);
  const float c = a.scale_log2e;

  // ---- this wave's 32 query rows: rows wrow0 + 16 j + lr, j = 0, 1, of a lane
  const int row_end = it.r0 + it.n_rows;             // one past the tile's last valid row
  const int wrow0 = it.r0 + wave * 32;
  const bool wave_active = wrow0 < row_end;
  const int wrow_last = (wrow0 + 31 < row_end - 1) ? wrow0 + 31 : row_end - 1;
  const int wave_min_pos = P + wrow0 / G;
  const int n_tiles = (P + (row_end - 1) / G) / BN + 1;
  const int kt_last = wave_active ? (P + wrow_last / G) / BN : -1;   // last tile this wave has keys in

  int prow[2];                                        // positions of this lane's rows
  int64_t rowoff[2];
  vec qf[2][4];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int row = wrow0 + 16 * j + lr;
    const int rc = row < row_end ? row : row_end - 1;
    prow[j] = P + rc / G;
    rowoff[j] = ((int64_t)(t0 + rc / G) * a.n_h + (g * G + rc % G)) * D;
    const uint16_t* qp = reinterpret_cast<const uint16_t*>(a.q) + rowoff[j] + 8 * lh;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) qf[j][kk] = as_vec<vec>(*reinterpret_cast<const u32x4*>(qp + 32 * kk));
  }

  f32x4 O[8][2];
  float mrow[2] = {-INFINITY, -INFINITY}, lsum[2] = {0.f, 0.f};
#pragma unroll
  for (int ct = 0; ct < 8; ++ct)
#pragma unroll
    for (int j = 0; j < 2; ++j) O[ct][j] = f32x4{0.f, 0.f, 0.f, 0.f};

  // ---- staging: wave w moves group w/2 of every tile, quarters 2(w%2) and 2(w%2)+1 of its K rows
  //      and of its V^T runs (1 KiB per instruction).  LDS chunk ci (16 bytes) of a group's K part
  //      holds key ci/16, logical chunk (ci%16) ^ swizzle(key); chunk ci of its V part holds channel
  //      ci/2, positions 8*((ci%2) ^ swizzle(channel)) .. +7.
  const int sblk = wave >> 1;
  uint32_t kg[2], vg[2];                             // this lane's byte offsets inside a block
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int ci = (2 * (wave & 1) + j) * 64 + lane;
    const int key = ci >> 4;
    kg[j] = (uint32_t)(2 * (key * D + 8 * ((ci & 15) ^ k_swz(16 * (sblk & 1) + key))));
    const int vd = ci >> 1;
    vg[j] = (uint32_t)(2 * (vd * bt + 8 * ((ci & 1) ^ v_swz(vd))));     // channel vd's run of 16 slots inside its bt-slot row
  }
  const int64_t k_region = (int64_t)g * bt * D;
  const int64_t v_region = (int64_t)a.n_kv * bt * D + (int64_t)g * D * bt;
  const uint32_t lds_wave = (uint32_t)(uintptr_t)(lds_u8*)smem + sblk * 4096 + 2 * (wave & 1) * 1024;   // LDS address of this wave's first quarter in stage 0

  for (int i = tid; i < nblk_valid; i += 512) tab_lds[i] = table[i];
  __builtin_amdgcn_s_waitcnt(kWaitVm0);                // the query fragments are in: from here on only tile loads are in flight
  __syncthreads();
  // this wave's 16-position group of tile t (clamped: always valid) and its block's id
  auto group = [&](int t) {
    const int gi = 4 * t + sblk;
    return gi < ngrp_valid ? gi : ngrp_valid - 1;
  };
  auto issue_tile = [&](int t, int32_t id) {         // 4 direct loads: tile t -> stage t % kStages
    const int half = group(t) & hsh;
    const uint16_t* blk = pool + (int64_t)__builtin_amdgcn_readfirstlane(id) * a.block_elems;
    const uint32_t dst = lds_wave + (t % kStages) * kStage;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      load_to_lds16(blk + k_region + BT * half * D, kg[j], dst + j * 1024);
      load_to_lds16(blk + v_region + BT * half, vg[j], dst + kTile + j * 1024);
    }
  };
#pragma unroll
  for (int t = 0; t < kStages - 1; ++t) issue_tile(t, tab_lds[group(t) >> hsh]);
  int32_t id_next = tab_lds[group(kStages - 1) >> hsh];      // of the tile that is requested next

  // ---- operand fragments.  Row m of key tile 2 b + t is key 32 b + 8 (m / 4) + 4 t + m % 4, so that a lane ends up with
  //      the weights of 8 consecutive positions, which are also its 16-byte run of V^T
  const uint32_t kbase = (uint32_t)((8 * (lr >> 2) + (lr & 3)) * 256 + ((lh ^ lr) << 4));
  const uint32_t vbase = (uint32_t)(kTile + (lh >> 1) * 4096 + lr * 32 + (((lh & 1) ^ v_swz(lr)) << 4));
  f32x4 S[4][2];
  vec Pw[2][2];
  auto load_k = [&](vec(&kf)[2], const uint8_t* buf, int q) {      // step q: key tiles of group q / 4, channels 32 (q % 4) ..
#pragma unroll
    for (int i = 0; i < 2; ++i)
      kf[i] = *reinterpret_cast<const vec*>(buf + (kbase ^ (uint32_t)((q & 3) << 6)) + (q >> 2) * 8192 + i * 1024);
  };
  auto load_v = [&](vec(&vf)[2], const uint8_t* buf, int q) {      // step q: keys 32 (q / 4) .., channel tiles 2 (q % 4) ..
#pragma unroll
    for (int i = 0; i < 2; ++i)
      vf[i] = *reinterpret_cast<const vec*>(buf + vbase + (q >> 2) * 8192 + (2 * (q & 3) + i) * 512);
  };
  auto score = [&](const vec(&kf)[2], int q) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
        S[2 * (q >> 2) + i][j] = M::mfma(kf[i], qf[j][q & 3], q & 3 ? S[2 * (q >> 2) + i][j] : f32x4{0.f, 0.f, 0.f, 0.f});
  };
  auto mask = [&](int t) {                             // causal mask on the tiles that reach past the first row's position
    if (BN * t + BN - 1 > wave_min_pos) {
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int thr = prow[j] - (BN * t + 8 * lh);
#pragma unroll
        for (int k4 = 0; k4 < 4; ++k4)
#pragma unroll
          for (int i = 0; i < 4; ++i) S[k4][j][i] = 32 * (k4 >> 1) + 4 * (k4 & 1) + i <= thr ? S[k4][j][i] : -INFINITY;
      }
    }
  };
  // The running maximum is only raised when some row of the wave has outgrown it by more
  // than 2^8: until then the weights are taken relative to the old maximum (they stay below
  // 256, exact in fp32 and well inside the 16-bit range), which spares the rescaling of the
  // 64 accumulator registers and the exchange between lanes on almost every tile.
  auto raise = [&]() {
    float tm[2];                                       // over the lane's keys
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      tm[j] = S[0][j][0];
#pragma unroll
      for (int k4 = 0; k4 < 4; ++k4)
#pragma unroll
        for (int i = 0; i < 4; ++i) tm[j] = fmaxf(tm[j], S[k4][j][i]);
    }
    if (__builtin_amdgcn_ballot_w64((tm[0] - mrow[0]) * c > 8.f || (tm[1] - mrow[1]) * c > 8.f)) {
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        tm[j] = fmaxf(tm[j], __shfl_xor(tm[j], 16));
        tm[j] = fmaxf(tm[j], __shfl_xor(tm[j], 32));
        const float m_new = fmaxf(mrow[j], tm[j]);
        const float alpha = __builtin_amdgcn_exp2f((mrow[j] - m_new) * c);
        mrow[j] = m_new;
        lsum[j] *= alpha;
#pragma unroll
        for (int ct = 0; ct < 8; ++ct)
#pragma unroll
          for (int i = 0; i < 4; ++i) O[ct][j][i] *= alpha;
      }
    }
  };
  auto weights = [&](int j, int b, float mc) {
    float p[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) p[e] = __builtin_amdgcn_exp2f(fmaf(S[2 * b + (e >> 2)][j][e & 3], c, -mc));
    // the row sum is taken over the rounded weights, the ones the second product uses
    Pw[j][b] = M::pack(p, lsum[j]);
  };

  auto request = [&](int kt) {                         // the tile that takes the stage of tile kt - 1
    issue_tile(kt + kStages - 1, id_next);
    id_next = tab_lds[group(kt + kStages) >> hsh];
  };
  auto step = [&](int kt) {
    const uint8_t* buf = smem + (kt % kStages) * kStage;
    vec kf[3][2];
    load_k(kf[0], buf, 0);
    load_k(kf[1], buf, 1);
    __builtin_amdgcn_sched_barrier(kScheduleAlu);
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      if (q < 6) load_k(kf[(q + 2) % 3], buf, q + 2);
      score(kf[q % 3], q);
      if (q == 3) request(kt);
      __builtin_amdgcn_sched_barrier(kScheduleAlu);      // or the reads move down to their products
    }
    __builtin_amdgcn_sched_barrier(0);
    vec vf[3][2];                                      // on their way while the weights are computed
    load_v(vf[0], buf, 0);
    load_v(vf[1], buf, 1);
    __builtin_amdgcn_sched_barrier(0);
    mask(kt);
    raise();
    const float mc[2] = {mrow[0] * c, mrow[1] * c};
#pragma unroll
    for (int q = 0; q < 4; ++q) weights(q & 1, q >> 1, mc[q & 1]);
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      if (q < 6) load_v(vf[(q + 2) % 3], buf, q + 2);
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          O[2 * (q & 3) + i][j] = M::mfma(vf[q % 3][i], Pw[j][q >> 2], O[2 * (q & 3) + i][j]);
    }
    // the first weights, then three of the others' instructions between two products
    __builtin_amdgcn_sched_group_barrier(0x002, 40, 0);
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      if (q < 6) __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x002, 3, 0);
      }
    }
  };
  // slots at or past the sequence's length hold arbitrary bits: zero them so that a zero weight
  // times such a value cannot turn into NaN (only the last tile of a sequence needs it)
  auto clear_past_end = [&](int kt) {
    if (BN * kt + BN <= L) return;
    uint8_t* buf = smem + (kt % kStages) * kStage;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int ci = tid + 512 * j;
      const int u = ci >> 8, vd = (ci & 255) >> 1, vh = (ci & 1) ^ v_swz(vd);
      const int pos0 = BN * kt + BT * u + 8 * vh;
      if (pos0 + 8 > L) {
        u32x4* slot = reinterpret_cast<u32x4*>(buf + kTile + ci * 16);
        u32x4 v = *slot;
        uint16_t e[8];
        __builtin_memcpy(e, &v, 16);
#pragma unroll
        for (int s = 0; s < 8; ++s)
          if (pos0 + s >= L) e[s] = 0;
        __builtin_memcpy(&v, e, 16);
        *slot = v;
      }
    }
    __syncthreads();
  };

  // tile kt has landed (this wave's part: all but the 4 loads of tile kt + 1 are complete), and after
  // the barrier so has everybody's; everybody is also done with tile kt - 1, whose stage is refilled next
  auto enter = [&](int kt) {
    __builtin_amdgcn_s_waitcnt(kWaitTile);
    __syncthreads();
    clear_past_end(kt);
  };
  int kt = 0;
  for (; kt <= kt_last; ++kt) {
    enter(kt);
    step(kt);
  }
  for (; kt < n_tiles; ++kt) {                         // tiles that only the other waves have keys in
    enter(kt);
    request(kt);
  }
  __builtin_amdgcn_s_waitcnt(kWaitVm0);                // the look-ahead loads past the last tile must land before the LDS is released

  // ---- normalise and store: lane (row lr of tile j, quarter lh) holds channels 16 ct + 4 lh + (0..3)
  if (wave_active) {
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      float l = lsum[j];
      l += __shfl_xor(l, 16);
      l += __shfl_xor(l, 32);
      const float inv = 1.f / l;
      if (wrow0 + 16 * j + lr >= row_end) continue;
      uint16_t* op = reinterpret_cast<uint16_t*>(a.out) + rowoff[j] + 4 * lh;
#pragma unroll
      for (int ct = 0; ct < 8; ++ct) {
        uint16_t o4[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) o4[i] = M::out(O[ct][j][i] * inv);
        uint2 w;
        __builtin_memcpy(&w, o4, 8);
        *reinterpret_cast<uint2*>(op + 16 * ct) = w;
      }
    }
  }
}

}  // namespace

flp_status flp_launch_attn_mfma(int dtype, const FlpAttnArgs& a, const FlpMfmaItem* items_dev, int32_t n_items,
                                const FlpAttnUnit* units_dev, hipStream_t stream) {
  if (n_items <= 0) return FLP_OK;
  if (dtype == FLP_F16)
    hipLaunchKernelGGL((attn_mfma_kernel<MF16>), dim3(n_items), dim3(512), 0, stream, a, items_dev, units_dev);
  else if (dtype == FLP_BF16)
    hipLaunchKernelGGL((attn_mfma_kernel<MBF16>), dim3(n_items), dim3(512), 0, stream, a, items_dev, units_dev);
  else {
    flp_set_error("attention (matrix-core path): dtype %d not supported", dtype);
    return FLP_ENOTSUP;
  }
  FLP_TRY_HIP(hipGetLastError());
  return FLP_OK;
}
