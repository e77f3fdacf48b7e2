// Dense products of the layer step: the base projection y = x . W_base of flp_lora_apply_paged when the caller
// passes w_base (paper Eq. 1: W' = W + A B; this is the W term.  The paper keeps the base model outside the pool,
// and so does this library: w_base is an ordinary dense matrix, [d_in, d_out] or [d_out, d_in]), and the dense
// projections of fll_layer_forward.
//
// 16-bit pools: both operands are read along the contraction (a W given as [d_in, d_out] is first transposed into
// the pool's workspace), the projections that share an input go in one launch, and the contraction may be split into
// slices whose fp32 partial products a second kernel adds in slice order.
// fp32 pools: a matrix-core kernel of its own (the fp32 workload is tiny and bound by latency).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <type_traits>

#include "flp_internal.h"
#include "flp_types.h"

namespace {

typedef float f32x4g __attribute__((ext_vector_type(4)));
typedef _Float16 h16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 b16x8 __attribute__((ext_vector_type(8)));

struct GF16 {
  typedef h16x8 vec;
  typedef _Float16 elem;
  typedef F16 S;
  static __device__ __forceinline__ f32x4g mfma(vec a, vec b, f32x4g c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
  }
};
struct GBF16 {
  typedef b16x8 vec;
  typedef __bf16 elem;
  typedef BF16 S;
  static __device__ __forceinline__ f32x4g mfma(vec a, vec b, f32x4g c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
  }
};

// ---- W [K, N] -> Wt [N, K], 16-bit elements, 64 x 64 tiles through LDS
__global__ __launch_bounds__(256) void transpose16_kernel(const uint16_t* __restrict__ w, uint16_t* __restrict__ wt,
                                                          int K, int N) {
  __shared__ uint16_t tile[64][66];
  const int k0 = blockIdx.y * 64, n0 = blockIdx.x * 64;
  for (int i = threadIdx.x; i < 64 * 64; i += 256) {
    const int r = i >> 6, c = i & 63;
    tile[r][c] = (k0 + r < K && n0 + c < N) ? w[(int64_t)(k0 + r) * N + n0 + c] : (uint16_t)0;
  }
  __syncthreads();
  for (int i = threadIdx.x; i < 64 * 64; i += 256) {
    const int r = i >> 6, c = i & 63;      // r: n within tile, c: k within tile
    if (n0 + r < N && k0 + c < K) wt[(int64_t)(n0 + r) * K + k0 + c] = tile[c][r];
  }
}

// ------------------------------------------------------------------------------- the tiled kernel
// One workgroup computes a tile of FT features x MT tokens of one projection and one slice of the contraction, as
// the transposed product (A operand = rows of W, B operand = token rows) with mfma_f32_16x16x32.  Large products are
// bound by the power the chip may draw: M 16384, N = K = 4096 takes 402 us at 2.05 GHz (1.37 PFLOP/s); a four-wave kernel
// with 128 x 128 corners on 32x32x16 instructions took 429 us at 1.85 GHz.
//
// Operands travel in k tiles of 64 coefficients, so that a row of a tile is one whole 128-byte line, from memory to
// LDS with the direct loads of gfx950 (8 lines per instruction; inline assembly with its own s_waitcnt vmcnt) into a
// ring of ST stages.  LDS position rho of a row inside a tile: chunk c (16 bytes) sits in slot c ^ ((rho >> 1) & 7) of
// the row's 128 bytes; the 16 rows of an operand fragment are 16 neighbouring positions, so the 16 lanes that read one
// chunk hit 16 different slots of a 256-byte window.  Which feature a position holds is free (the lane that loads
// it fetches any row): positions 16 tau + m of a 64-feature group hold feature 4 m + tau, so that a lane's four
// accumulators of one token are 16 consecutive features and results leave in 32-byte (fp32: 64-byte) pieces.
//
// Two loops:
//   ring (ST >= 3)   every wave reads the fragments of the next k step while it multiplies the current one; one barrier
//                    per stage, ahead of the stage's last k step; ST - 1 stages in flight.  Small batches live on loads
//                    in flight, so their tiles are narrow in tokens and the ring is deep.
//   ping-pong (PP)   256 x 256 tiles, two stages of 64 KiB, eight waves in two groups of four (one wave of each group
//                    per SIMD) that take turns: while one group reads its fragments and requests the stage after next,
//                    the other multiplies; they change places at every barrier.  (M 20000, N = K = 4096: 525 us, with
//                    256 x 128 tiles in the ring form 574 us.)
//
// GATED: the gated-SiLU pair of an MLP in one pass.  The features are those of both matrices interleaved in groups
// of 64 (32 gate rows, the same 32 up rows: positions 16 tau + m hold feature 2 m + (tau & 1) of matrix tau >> 1), so a
// lane holds gate and up of the same 8 features and stores silu(g) * u, both rounded to the element type first as
// two separate products and an element-wise kernel would have stored and re-read them.
//
// LORA: the expand step of the projections' LoRA branches as an epilogue.  For every adapter among a wave's tokens
// (tokens of a sequence are neighbours, so one or two) it adds B^T (64 features x ranks) times the tokens' scaled v,
// 16 ranks per step: v enters as a 16-bit high part (k slots 0 .. 15) plus remainder (16 .. 31) against the same
// coefficients: 16 bits of it in bf16; in fp16 22 from 0.25 on, fewer below (the remainder's spacing ends at 2^-24), and
// it has to stay below 65504, scaled.  The look-ups are made before the loop and v is laid out in LDS once
// per workgroup; chains of dependent loads per adapter, token tile and slice of v had cost a fifth of the launch.  The coefficients come from the adapter's pages eight bytes (four
// features) per lane and rank and are turned into the four tiles' fragments in registers.  The sum is rounded once.
constexpr int GK = 64;
constexpr int vmcnt_imm(int n) { return (n & 15) | ((n >> 4) << 14) | (7 << 4) | (15 << 8); }   // s_waitcnt vmcnt(n) only
constexpr int kWaitLgkm0 = 15 | (3 << 14) | (7 << 4);                                           // lgkmcnt(0) only
constexpr int kWaitAll0 = 7 << 4;                                                               // vmcnt(0) and lgkmcnt(0)

// M0 is named as clobbered so that no pass keeps a value of its own alive in it across the statement; the
// compiler notes that it reserves the register, which is the point.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void gload_lds16(const void* base, uint32_t voff, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(voff), "s"(base), "s"(lds)
               : "memory", "m0");
}
#pragma clang diagnostic pop
typedef __attribute__((address_space(3))) uint8_t g_lds_u8;

__device__ __forceinline__ int gswz(int rho) { return (rho >> 1) & 7; }

struct GemmLoraArgs {
  FlpGemmLora p[FLP_MAX_PROJ];     // per projection; gated: gate, up
};
struct NoLora {};

// What the LoRA epilogue needs to know about a tile's tokens, looked up while the first stages of the tile are on
// their way: which adapter (slot of the current round) and row of v a token has, and the page rows of the slots'
// coefficients.  Without it every adapter costs the epilogue five dependent trips to memory.  A tile with more than
// kLoraSlots adapters takes them in rounds.
constexpr int kLoraSlots = 8;
struct GemmLoraLds {
  uint64_t row[2][kLoraSlots][64];  // address of rank row rho of a slot's B; [1]: the up matrix of a gated pair
  int32_t ad[256];                  // adapter of a token of the tile, -1: none
  int32_t vrow[256];                // row of v of the token
  int32_t index[256];               // position of the token's adapter in `list`, -1: none
  int32_t list[256];                // the tile's adapters
  int32_t n, rank[kLoraSlots];
};

// the tables of the adapters list[first .. first + kLoraSlots)
template <bool GATED, int NTHR>
__device__ __forceinline__ void lora_round(const FlpGemmLora* lp0, const FlpGemmLora* lp1, int N, int first, GemmLoraLds& t) {
  const int rpb = (int)(lp0->block_elems / N);
  const int n = t.n - first < kLoraSlots ? t.n - first : kLoraSlots;
  for (int e = threadIdx.x; e < n * 64; e += NTHR) {
    const int s = e >> 6, rho = e & 63, ad = t.list[first + s];
    const int r = lp0->rank[ad] < lp0->max_rank ? lp0->rank[ad] : lp0->max_rank;
    if (rho == 0) t.rank[s] = r;
#pragma unroll
    for (int g = 0; g < (GATED ? 2 : 1); ++g) {
      const FlpGemmLora& lp = g ? *lp1 : *lp0;
      if (r > 0) {
        const int row = lp.b_row_base[ad] + (rho < r ? rho : 0);
        const uint16_t* a = reinterpret_cast<const uint16_t*>(lp.pool) +
                            (int64_t)lp.tables[lp.b_tab_off[ad] + row / rpb] * lp.block_elems + (int64_t)(row % rpb) * N;
        t.row[g][s][rho] = (uint64_t)(uintptr_t)a;
      }
    }
  }
}

template <bool GATED, int MT, int NTHR>
__device__ __forceinline__ void lora_setup(const FlpGemmLora* lp0, const FlpGemmLora* lp1, int N, int m0, int M, GemmLoraLds& t) {
  static_assert(MT <= NTHR && MT <= 256, "a thread looks up one token");
  const int tid = threadIdx.x;
  if (tid < MT) {
    const int m = m0 + tid;
    int ad = m < M ? lp0->token_adapter[m] : -1;
    if (ad >= lp0->n_adapters) ad = -1;
    t.ad[tid] = ad;
    t.vrow[tid] = ad >= 0 ? lp0->vrow_base[ad] + lp0->inv_perm[m] : 0;
    t.index[tid] = -1;
  }
  __syncthreads();
  if (tid < 64) {                                         // one wave lists the adapters
    int mine[MT / 64], n = 0;
#pragma unroll
    for (int k = 0; k < MT / 64; ++k) mine[k] = t.ad[64 * k + tid];
    for (;;) {
      int cand = -1;
#pragma unroll
      for (int k = 0; k < MT / 64; ++k) cand = mine[k] >= 0 ? mine[k] : cand;
      const uint64_t todo = __ballot(cand >= 0);
      if (!todo) break;
      const int ad = __builtin_amdgcn_readlane(cand, __ffsll((long long)todo) - 1);
#pragma unroll
      for (int k = 0; k < MT / 64; ++k)
        if (mine[k] == ad) {
          t.index[64 * k + tid] = n;
          mine[k] = -1;
        }
      if (tid == 0) t.list[n] = ad;
      ++n;
    }
    if (tid == 0) t.n = n;
  }
  __syncthreads();
  lora_round<GATED, NTHR>(lp0, lp1, N, 0, t);
}

// The scaled v of the tile's tokens as B operands, in the LDS that the ring leaves: block (token tile, rank tile) of 1 KiB
// holds the 64 lanes' fragments, ranks 8 kq .. 8 kq + 7 as a 16-bit high part (lanes 16 kq ..) and remainder
// (lanes 32 + 16 kq ..).  Once per workgroup: its waves share the tokens, and the sums over the shrink step's slices
// are all in flight together.
template <typename G, int MT, int NTHR>
__device__ __forceinline__ void lora_stage_v(const FlpGemmLora& lp, const GemmLoraLds& t, uint8_t* smem) {
  typedef typename G::elem elem;
  const int n_g8 = lp.rp / 8;                             // groups of 8 ranks: 2, 4 or 8
  const int64_t step = (int64_t)lp.v_rows * lp.n_proj * lp.rp;
#pragma unroll 2
  for (int e = threadIdx.x; e < MT * n_g8; e += NTHR) {
    const int tok = e / n_g8, g8 = e - tok * n_g8;
    const int ad = t.ad[tok];
    f32x4g x0 = {0.f, 0.f, 0.f, 0.f}, x1 = x0;
    if (ad >= 0) {
      const float* vp = lp.v + ((int64_t)t.vrow[tok] * lp.n_proj + lp.p) * lp.rp + 8 * g8;
      for (int ks = 0; ks < lp.k_splits; ++ks, vp += step) {
        x0 += *reinterpret_cast<const f32x4g*>(vp);
        x1 += *reinterpret_cast<const f32x4g*>(vp + 4);
      }
      const float sc = lp.scale[ad];
      x0 *= sc;
      x1 *= sc;
    }
    elem hi[8], lo[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const float v = q < 4 ? x0[q & 3] : x1[q & 3];
      hi[q] = (elem)v;
      lo[q] = (elem)(v - (float)hi[q]);
    }
    uint8_t* blk = smem + ((tok >> 4) * (n_g8 / 2) + (g8 >> 1)) * 1024 + ((tok & 15) + 16 * (g8 & 1)) * 16;
    u32x4 raw;
    __builtin_memcpy(&raw, hi, 16);
    *reinterpret_cast<u32x4*>(blk) = raw;
    __builtin_memcpy(&raw, lo, 16);
    *reinterpret_cast<u32x4*>(blk + 512) = raw;
  }
}

// adds one projection's LoRA branch of one slot to NTAU feature tiles (acc[TAU0 .. TAU0 + NTAU - 1][.]) of a wave; the
// lane's tile row m of tile TAU0 + q is feature f0 + NTAU * m + q; v: the wave's first token tile's fragments.
// own: the lanes whose token of tile j has the slot's adapter.  A lane's accumulators belong to one token (the products'
// columns are independent), so each lane keeps or drops its sums and another adapter's coefficients, infinities and NaN
// among them, never reach a token; tiles without a token of the adapter are skipped.  (13B layer, 9900 tokens: 6597 us
// against 6570 with v zeroed for other adapters' tokens, which lets 0 x inf through.  A further branch for tiles of one
// adapter costs registers that the 256 x 256 tile does not have: 208 bytes of scratch and 26.8 ms.)
template <typename G, int TAU0, int NTAU, int AT>
__device__ __forceinline__ void add_lora(const uint64_t* rows, int r, int n_nt, const uint64_t (&own)[AT],
                                         const uint8_t* v, int f0, int N, f32x4g (&acc)[4][AT]) {
  typedef typename G::vec vec;
  const int lane = threadIdx.x & 63, m16 = lane & 15, kg = lane >> 4, kq = kg & 1;
  int fc = f0 + NTAU * m16;                               // N is a multiple of 8 and f0 of 32: a lane's features are all in or all out
  const bool fvalid = fc < N;
  fc = fvalid ? fc : 0;
  // A operand: B[rho, feature] for the lane's 8 ranks and its NTAU neighbouring features, one rank tile ahead
  uint32_t g[8][NTAU / 2];
  auto fetch = [&](int nt) {
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const uint32_t* rp = reinterpret_cast<const uint32_t*>((uintptr_t)rows[16 * nt + 8 * kq + q] + 2 * fc);
#pragma unroll
      for (int h = 0; h < NTAU / 2; ++h) g[q][h] = rp[h];
    }
  };
  fetch(0);
  for (int nt = 0; 16 * nt < r; ++nt) {
#pragma unroll
    for (int q = 0; q < 8; ++q)
#pragma unroll
      for (int h = 0; h < NTAU / 2; ++h) g[q][h] = 16 * nt + 8 * kq + q < r && fvalid ? g[q][h] : 0u;
    vec af[NTAU];
#pragma unroll
    for (int t = 0; t < NTAU; ++t) {
      u32x4 e;
#pragma unroll
      for (int q = 0; q < 4; ++q)                         // ranks 2 q, 2 q + 1 of feature t: its half of the two words
        e[q] = __builtin_amdgcn_perm(g[2 * q + 1][t / 2], g[2 * q][t / 2], t & 1 ? 0x07060302u : 0x05040100u);
      __builtin_memcpy(&af[t], &e, 16);
    }
    if (16 * (nt + 1) < r) fetch(nt + 1);
#pragma unroll
    for (int j = 0; j < AT; ++j) {
      if (!own[j]) continue;
      const vec b = *reinterpret_cast<const vec*>(v + (j * n_nt + nt) * 1024 + lane * 16);
      const bool mine = (own[j] >> lane) & 1;
#pragma unroll
      for (int t = 0; t < NTAU; ++t) {
        const f32x4g sum = G::mfma(af[t], b, acc[TAU0 + t][j]);
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[TAU0 + t][j][i] = mine ? sum[i] : acc[TAU0 + t][j][i];
      }
    }
  }
}

// Workgroup -> (feature tile, slice) unit u and token tile tm.  Blocks of gf units x the token tiles of a band run next to each other
// on one XCD (workgroups are placed on the 8 XCDs in turn), so that an operand tile crosses from memory into one L2 once.  The
// tiles, in the order of their blocks, are dealt out 256 at a time, 32 to an XCD and the last ones in eighths.  (Whole blocks dealt to
// the XCDs in turn left some with one more than the others: 240 tiles of 256 x 256, 30 for each XCD, took two rounds.  An eighth of
// all tiles to each XCD keeps them apart, and the operands cross from memory more often: layer of 9874 tokens, 13B shapes, 6660 ->
// 6917 us.)  The bands are of equal height: with eight tiles in each but the last, a last one of a single token tile put up to 32 of
// its tiles on one XCD and none on others, and where that tile holds the batch's single tokens, with an adapter each, its tiles take
// several times as long (2048 tokens of prompts and 200 single ones, 7B shapes, LoRA of rank 64 on all seven: layer 4690 us, with equal
// bands 3844).
__host__ __device__ inline bool tile_of_block(int block, int n_units, int m_tiles, int gf, int bands, int* u, int* tm) {
  const int n_tiles = n_units * m_tiles, xcd = block & 7;
  const int first = block >> 8 << 8, part = n_tiles - first < 256 ? n_tiles - first : 256;
  int at = (part * xcd >> 3) + ((block & 255) >> 3);
  if (at >= part * (xcd + 1) >> 3) return false;
  at += first;
  const int low = m_tiles / bands, n_high = m_tiles % bands;         // the first n_high bands have one token tile more
  const int t = at / n_units, in_high = n_high * (low + 1);
  const int rows = t < in_high ? low + 1 : low;
  const int m0 = t < in_high ? t / rows * rows : in_high + (t - in_high) / rows * rows;
  at -= m0 * n_units;
  const int ub = at / (gf * rows), cols = n_units - ub * gf < gf ? n_units - ub * gf : gf;
  at -= ub * gf * rows;
  *u = ub * gf + at % cols;
  *tm = m0 + at / cols;
  return true;
}
// with more than eight token tiles, blocks of about 4 x 8: the workgroups that run together fetch 12 operand panels, not 33
inline void tile_blocks(int m_tiles, int* gf, int* bands) {
  *gf = m_tiles > 8 ? 4 : 1;
  *bands = (m_tiles + 7) / 8;
}

// WF x WT waves of 64 features x 16 AT tokens each
template <typename G, int WF, int WT, int AT, int ST, bool PP, bool GATED, bool LORA>
__global__ __launch_bounds__(64 * WF * WT, (WF * WT + 3) / 4)
    void gemm_kernel(FlpGemmArgs a, std::conditional_t<LORA, GemmLoraArgs, NoLora> la) {
  typedef typename G::vec vec;
  typedef typename G::S S;
  constexpr int FT = 64 * WF, MT = 16 * WT * AT, NW = WF * WT;
  constexpr int NF = FT / 8 / NW;                       // loads of W rows of a wave per stage (8 rows each)
  constexpr int NPER = (FT + MT) / 8 / NW;              // all loads of a wave per stage
  constexpr int kStage = (FT + MT) * 128;
  static_assert(FT / 8 % NW == 0 && MT / 8 % NW == 0, "the waves share the loads of a stage evenly");
  static_assert(!PP || (ST == 2 && WT == 2 && WF == 4), "ping-pong: two groups of four waves, two stages");
  extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];
  const int tid = threadIdx.x, lane = tid & 63, m16 = lane & 15, kg = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wf = wave % WF, wt = wave / WF;

  int u, tm;
  if (!tile_of_block((int)blockIdx.x, a.f_tiles * a.splits, a.m_tiles, a.gf, a.bands, &u, &tm)) return;
  const int z = u / a.f_tiles;
  int ft = u - z * a.f_tiles;
  int p = 0;
  while (p + 1 < a.n_proj && ft >= a.proj[p + 1].tile0) ++p;
  const FlpGemmProj& pr = a.proj[p];
  ft -= pr.tile0;
  const int N = pr.N;                                   // GATED: rows of both matrices together
  const int n0 = ft * FT, m0 = tm * MT, K = a.K;
  const int nk_all = K / GK;
  const int kt0 = (int)((int64_t)nk_all * z / a.splits), nk = (int)((int64_t)nk_all * (z + 1) / a.splits) - kt0;

  // ---- loads: instruction j of a stage covers LDS rows 8 j .. 8 j + 7 (W rows first, then tokens); wave w issues
  //      j = w, w + NW, ...; offsets are relative to the tile's first row, so 32 bits always do.  Rows past the end
  //      repeat the last one and are never stored.
  uint32_t voff[NPER];
#pragma unroll
  for (int q = 0; q < NPER; ++q) {
    const int rl = 8 * (wave + NW * q) + (lane >> 3);
    if (q < NF) {
      const int g64 = rl & ~63, tau = (rl >> 4) & 3, m = rl & 15;
      int row;
      if (GATED) {
        row = (g64 >> 1) + 2 * m + (tau & 1);
        row = n0 / 2 + row < N / 2 ? row : N / 2 - 1 - n0 / 2;
      } else {
        row = g64 + 4 * m + tau;
        row = n0 + row < N ? row : N - 1 - n0;
      }
      voff[q] = (uint32_t)row * (uint32_t)(K * 2) + 16u * ((lane & 7) ^ gswz(rl));
    } else {
      const int r = rl - FT;
      const int row = m0 + r < a.M ? r : a.M - 1 - m0;
      voff[q] = (uint32_t)row * (uint32_t)(a.ld_x * 2) + 16u * ((lane & 7) ^ gswz(rl));
    }
  }
  const uint32_t lds_wave = (uint32_t)(uintptr_t)(g_lds_u8*)smem + 1024u * (uint32_t)wave;
  const uint16_t* const xk = a.x + (int64_t)m0 * a.ld_x + (int64_t)kt0 * GK;
  const uint16_t* const wk = pr.w + (int64_t)(GATED ? n0 / 2 : n0) * K + (int64_t)kt0 * GK;
  const uint16_t* const wk2 = GATED ? pr.w2 + (int64_t)(n0 / 2) * K + (int64_t)kt0 * GK : nullptr;
  auto issue_load = [&](int t, int st, int q) {         // load q of k tile t into stage st
    const uint32_t dst = lds_wave + (uint32_t)(st * kStage + 1024 * NW * q);
    if (q < NF) {
      const bool up = GATED && ((wave + NW * q) & 4);    // rows 32 .. 63 of a group of 64
      gload_lds16((up ? wk2 : wk) + (int64_t)t * GK, voff[q], dst);
    } else {
      gload_lds16(xk + (int64_t)t * GK, voff[q], dst);
    }
  };

  // ---- fragments: chunk 4 kk + kg of the row
  const uint32_t offa = (uint32_t)((64 * wf + m16) * 128 + ((kg ^ gswz(m16)) << 4));             // + 2048 per tile
  const uint32_t offb = (uint32_t)((FT + 16 * wt * AT + m16) * 128 + ((kg ^ gswz(m16)) << 4));
  f32x4g acc[4][AT];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < AT; ++j) acc[i][j] = f32x4g{0.f, 0.f, 0.f, 0.f};
  auto read_frags = [&](vec(&fa)[4], vec(&fb)[AT], int st, int kk) {
    const uint8_t* base = smem + st * kStage;
#pragma unroll
    for (int j = 0; j < AT; ++j) fb[j] = *reinterpret_cast<const vec*>(base + ((offb ^ (kk << 6)) + 2048 * j));
#pragma unroll
    for (int i = 0; i < 4; ++i) fa[i] = *reinterpret_cast<const vec*>(base + ((offa ^ (kk << 6)) + 2048 * i));
  };
  auto products = [&](const vec(&fa)[4], const vec(&fb)[AT]) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < AT; ++j) acc[i][j] = G::mfma(fa[i], fb[j], acc[i][j]);
  };

  const FlpGemmLora *lp0 = nullptr, *lp1 = nullptr;
  __shared__ std::conditional_t<LORA, GemmLoraLds, NoLora> lds;
  if constexpr (LORA) {
    lp0 = &la.p[GATED ? 0 : p];
    lp1 = &la.p[GATED ? 1 : p];
  }
  if constexpr (PP) {
    vec fa[4], fb[AT];
    auto bar = [&]() {
      __builtin_amdgcn_sched_barrier(0);
      asm volatile("s_barrier" ::: "memory");
      __builtin_amdgcn_sched_barrier(0);
    };
#pragma unroll
    for (int q = 0; q < NPER; ++q) issue_load(0, 0, q);
    if (nk > 1) {
#pragma unroll
      for (int q = 0; q < NPER; ++q) issue_load(1, 1, q);
    }
    if constexpr (LORA) lora_setup<GATED, MT, 64 * NW>(lp0, lp1, GATED ? N / 2 : N, m0, a.M, lds);
    if (nk > 1 && !LORA)
      __builtin_amdgcn_s_waitcnt(vmcnt_imm(NPER));
    else
      __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
    __syncthreads();
    // Intervals between barriers: group 0 reads k step s (two per stage) in interval 2 s and multiplies in 2 s + 1,
    // group 1 one interval later.  The last reads of stage t end with interval 4 t + 3; its buffer is refilled from
    // interval 4 t + 4 on, and what arrives there is first read in interval 4 t + 8: every wave waits for its own loads
    // before the barrier that ends interval 4 t + 7 (group 0 after a product, group 1 after a read).  Every wave passes
    // 4 nk + 1 barriers.
    if (wt) bar();
    for (int kt = 0; kt < nk; ++kt) {
      const int st = kt & 1;
      if (kt > 0 && kt + 1 < nk) {
#pragma unroll
        for (int q = 0; q < NPER; ++q) issue_load(kt + 1, st ^ 1, q);
      }
      read_frags(fa, fb, st, 0);
      __builtin_amdgcn_s_waitcnt(kWaitLgkm0);
      bar();
      products(fa, fb);
      bar();
      read_frags(fa, fb, st, 1);
      if (wt)
        __builtin_amdgcn_s_waitcnt(kWaitAll0);
      else
        __builtin_amdgcn_s_waitcnt(kWaitLgkm0);
      bar();
      products(fa, fb);
      if (!wt) __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
      bar();
    }
    if (!wt) bar();
  } else {
    // prologue: stages 0 .. ST - 2 requested, stage 0 complete
    vec a0[4], b0[AT], a1[4], b1[AT];
#pragma unroll
    for (int t = 0; t < ST - 1; ++t)
      if (t < nk) {
#pragma unroll
        for (int q = 0; q < NPER; ++q) issue_load(t, t, q);
      }
    if constexpr (LORA) lora_setup<GATED, MT, 64 * NW>(lp0, lp1, GATED ? N / 2 : N, m0, a.M, lds);
    if (ST - 1 <= nk && !LORA)
      __builtin_amdgcn_s_waitcnt(vmcnt_imm((ST - 2) * NPER));
    else
      __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));           // the set-up's own loads are the newest
    __syncthreads();
    read_frags(a0, b0, 0, 0);
    int st = 0, st_load = ST - 1;                       // stage of k tile kt; stage that takes k tile kt + ST - 1
    for (int kt = 0; kt < nk; ++kt) {
      // the buffer of k tile kt - 1 is free: everybody read its last fragments before the previous barrier
      const bool more = kt + ST - 1 < nk;
      if (more) {
#pragma unroll
        for (int q = 0; q < NPER; ++q) issue_load(kt + ST - 1, st_load, q);
      }
      read_frags(a1, b1, st, 1);
      products(a0, b0);
      __builtin_amdgcn_sched_barrier(0);
      st = st + 1 == ST ? 0 : st + 1;
      st_load = st_load + 1 == ST ? 0 : st_load + 1;
      // k tile kt + 1 has landed when at most ST - 2 later ones are outstanding
      if (more)
        __builtin_amdgcn_s_waitcnt(vmcnt_imm((ST - 2) * NPER));
      else
        __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
      __syncthreads();
      if (kt + 1 < nk) read_frags(a0, b0, st, 0);
      products(a1, b1);
      __builtin_amdgcn_sched_barrier(0);
    }
  }

  const int m_first = m0 + 16 * wt * AT;                // the wave's first token
  if constexpr (LORA) {
    const int32_t* const index = lds.index + 16 * wt * AT;
    const int n_nt = lp0->rp / 16;
    const int v_bytes = MT / 16 * n_nt * 1024;            // at most 64 KiB, twice for a gated pair: the ring holds it
    __syncthreads();                                      // nobody reads the ring any more
    lora_stage_v<G, MT, 64 * NW>(*lp0, lds, smem);
    if constexpr (GATED) lora_stage_v<G, MT, 64 * NW>(*lp1, lds, smem + v_bytes);
    __syncthreads();
    const uint8_t* const v0 = smem + wt * AT * n_nt * 1024;
    for (int first = 0; first < lds.n; first += kLoraSlots) {
      if (first > 0) {
        __syncthreads();                                // the previous round's tables are no longer read
        lora_round<GATED, 64 * NW>(lp0, lp1, GATED ? N / 2 : N, first, lds);
        __syncthreads();
      }
      for (int s = 0; s < kLoraSlots && first + s < lds.n; ++s) {
        uint64_t own[AT], any = 0;
#pragma unroll
        for (int j = 0; j < AT; ++j) {
          own[j] = __ballot(index[16 * j + m16] == first + s);
          any |= own[j];
        }
        const int r = lds.rank[s];
        if (!any || r <= 0) continue;
        if constexpr (GATED) {
          add_lora<G, 0, 2, AT>(lds.row[0][s], r, n_nt, own, v0, n0 / 2 + 32 * wf, N / 2, acc);
          add_lora<G, 2, 2, AT>(lds.row[1][s], r, n_nt, own, v0 + v_bytes, n0 / 2 + 32 * wf, N / 2, acc);
        } else {
          add_lora<G, 0, 4, AT>(lds.row[0][s], r, n_nt, own, v0, n0 + 64 * wf, N, acc);
        }
      }
    }
  }

  // ---- lane (token m16 of tile j, group kg): tile row 4 kg + i of tile tau is feature 16 kg + 4 i + tau of the 64
#pragma unroll
  for (int j = 0; j < AT; ++j) {
    const int m = m_first + 16 * j + m16;
    if (m >= a.M) continue;
    if constexpr (GATED) {
      if (pr.y) {
        const int n = n0 / 2 + 32 * wf + 8 * kg;        // the MLP width is a multiple of 32: all 8 features are in
        if (n >= N / 2) continue;
        uint16_t o[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float g = S::to_float(S::from_float(acc[e & 1][j][e >> 1]));
          const float up = S::to_float(S::from_float(acc[2 + (e & 1)][j][e >> 1]));
          o[e] = S::from_float(g / (1.0f + expf(-g)) * up);
        }
        u32x4 raw;
        __builtin_memcpy(&raw, o, 16);
        *reinterpret_cast<u32x4*>(pr.y + (int64_t)m * pr.ld_y + n) = raw;
      } else {
        // slices keep the two products apart: [gate | up] of width N / 2 each
        const int n = n0 / 2 + 32 * wf + 8 * kg;
        if (n >= N / 2) continue;
        float* yp = pr.part + ((int64_t)z * a.M + m) * N + n;
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int q = 0; q < 2; ++q)
            *reinterpret_cast<f32x4g*>(yp + h * (N / 2) + 4 * q) =
                f32x4g{acc[2 * h][j][2 * q], acc[2 * h + 1][j][2 * q], acc[2 * h][j][2 * q + 1], acc[2 * h + 1][j][2 * q + 1]};
      }
    } else {
      const int n = n0 + 64 * wf + 16 * kg;
      if (n >= N) continue;
      float v[16];
#pragma unroll
      for (int e = 0; e < 16; ++e) v[e] = acc[e & 3][j][e >> 2];
      if (pr.part) {
        float* yp = pr.part + ((int64_t)z * a.M + m) * N + n;
        if (n + 16 <= N && (N & 3) == 0) {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            reinterpret_cast<f32x4g*>(yp)[e] = f32x4g{v[4 * e], v[4 * e + 1], v[4 * e + 2], v[4 * e + 3]};
        } else {
#pragma unroll
          for (int e = 0; e < 16; ++e)
            if (n + e < N) yp[e] = v[e];
        }
      }
      if (pr.y) {
        uint16_t o[16];
#pragma unroll
        for (int e = 0; e < 16; ++e) o[e] = S::from_float(v[e]);
        uint16_t* yp = pr.y + (int64_t)m * pr.ld_y + n;
        if (n + 16 <= N) {
          u32x4 raw[2];
          __builtin_memcpy(raw, o, 32);
          reinterpret_cast<u32x4*>(yp)[0] = raw[0];
          reinterpret_cast<u32x4*>(yp)[1] = raw[1];
        } else {
#pragma unroll
          for (int e = 0; e < 16; ++e)
            if (n + e < N) yp[e] = o[e];
        }
      }
    }
  }
}

// ---- sum of the slices, in slice order, four features per thread.  GATED: the slices hold [gate | up]; the result is
//      silu(g) * u with both rounded first.  FLP_REDUCE_KEEP: the unrounded sum goes back into slice 0.  FLP_REDUCE_ADD: y is a residual
//      stream that the rounded sum is added to.
template <typename G, bool GATED>
__global__ __launch_bounds__(256) void gemm_reduce_kernel(FlpGemmArgs a, int mode) {
  typedef typename G::S S;
  const FlpGemmProj& pr = a.proj[blockIdx.y];
  const int n_out = GATED ? pr.N / 2 : pr.N, n4 = n_out / 4;
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= (int64_t)a.M * n4) return;
  const int m = (int)(i / n4), n = (int)(i - (int64_t)m * n4) * 4;
  float* pp = pr.part + (int64_t)m * pr.N + n;
  const int64_t step = (int64_t)a.M * pr.N;
  f32x4g s = *reinterpret_cast<const f32x4g*>(pp), s2 = {0.f, 0.f, 0.f, 0.f};
  if (GATED) s2 = *reinterpret_cast<const f32x4g*>(pp + n_out);
  for (int z = 1; z < a.splits; ++z) {
    s += *reinterpret_cast<const f32x4g*>(pp + z * step);
    if (GATED) s2 += *reinterpret_cast<const f32x4g*>(pp + z * step + n_out);
  }
  uint16_t o[4];
  uint2 raw;
  uint2* const yp = reinterpret_cast<uint2*>(pr.y + (int64_t)m * pr.ld_y + n);
  if (mode == FLP_REDUCE_ADD) {
    raw = *yp;
    __builtin_memcpy(o, &raw, 8);
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    if (GATED) {
      const float g = S::to_float(S::from_float(s[e])), up = S::to_float(S::from_float(s2[e]));
      o[e] = S::from_float(g / (1.0f + expf(-g)) * up);
    } else {
      const uint16_t sum = S::from_float(s[e]);
      o[e] = mode == FLP_REDUCE_ADD ? S::from_float(S::to_float(o[e]) + S::to_float(sum)) : sum;
    }
  }
  __builtin_memcpy(&raw, o, 8);
  *yp = raw;
  if (mode == FLP_REDUCE_KEEP) *reinterpret_cast<f32x4g*>(pp) = s;
}

// ---- fp32: y = x . W^T, one 16 x 16 tile per workgroup with mfma_f32_16x16x4 (fp32 products and sums).  Bound by
//      latency, not by rate: the four waves take every fourth piece of 16 coefficients, operands come straight from
//      global memory (16 bytes per lane along the contraction; each of a piece's four instructions contracts one of
//      the lane's four coefficients), and the waves' sums meet in LDS in wave order.  20 tokens x 256 x 256: 33 us
//      with one thread per output.
template <bool KMAJOR>                                    // W stored [N, K]; otherwise [K, N]
__global__ __launch_bounds__(256) void gemm_f32_kernel(const float* __restrict__ x, int64_t ld_x,
                                                       const float* __restrict__ w, float* __restrict__ y, int64_t ld_y,
                                                       int M, int N, int K) {
  __shared__ f32x4g red[4][64];
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, r16 = lane & 15, kg = lane >> 4;
  const int n0 = blockIdx.x * 16, m0 = blockIdx.y * 16;
  const int n = n0 + r16 < N ? n0 + r16 : N - 1, m = m0 + r16 < M ? m0 + r16 : M - 1;     // clamped rows are never stored
  const float* xr = x + (int64_t)m * ld_x;
  f32x4g acc = {0.f, 0.f, 0.f, 0.f};
  const bool vec4 = (K & 3) == 0 && (ld_x & 3) == 0;
  for (int k0 = 16 * wave; k0 < K; k0 += 64) {
    const int k = k0 + 4 * kg;
    f32x4g xv = {0.f, 0.f, 0.f, 0.f}, wv = {0.f, 0.f, 0.f, 0.f};
    if (vec4 && k < K) {
      xv = *reinterpret_cast<const f32x4g*>(xr + k);
    } else {
#pragma unroll
      for (int c = 0; c < 4; ++c)
        if (k + c < K) xv[c] = xr[k + c];
    }
    if (KMAJOR && vec4 && k < K) {
      wv = *reinterpret_cast<const f32x4g*>(w + (int64_t)n * K + k);
    } else {
#pragma unroll
      for (int c = 0; c < 4; ++c)
        if (k + c < K) wv[c] = KMAJOR ? w[(int64_t)n * K + k + c] : w[(int64_t)(k + c) * N + n];
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(xv[c], wv[c], acc, 0, 0, 0);
  }
  red[wave][lane] = acc;
  __syncthreads();
  if (wave == 0) {
    const f32x4g s = ((red[0][lane] + red[1][lane]) + red[2][lane]) + red[3][lane];
#pragma unroll
    for (int i = 0; i < 4; ++i) {                         // row (token) 4 kg + i, column (feature) r16
      const int mm = m0 + 4 * kg + i;
      if (mm < M && n0 + r16 < N) y[(int64_t)mm * ld_y + n0 + r16] = s[i];
    }
  }
}

}  // namespace

namespace {

struct GemmCfg {
  int ft, mt, waves, lds;
  int per_cu;            // workgroups that fit a CU
  float step_us;         // time of one k tile when every CU runs its workgroups (products and loads)
  float fill_us;         // start-up and epilogue of a workgroup
  float part;            // time of a round that is nearly empty, as a share of a full one
};
constexpr int stage_bytes(int ft, int mt) { return (ft + mt) * 128; }
// kinds of tile, FLP_GEMM_*.  The times are what the planner adds up, fitted to launches on MI355X.  Against all kinds and
// numbers of slices at 96 shapes (1 .. 2000 tokens, the matrices of the 7B, 13B and 34B shapes; 3720 timings with operands
// from memory) the plan it picks is 2.4 % slower than the best one on average and 23 % at worst (34B gate and up at 33 tokens;
// one shape in six is more than 5 % off).
const GemmCfg kCfg[FLP_GEMM_KINDS] = {
    {64, 32, 2, 4 * stage_bytes(64, 32), 3, 0.488f, 4.44f, 0.53f},
    {128, 64, 4, 3 * stage_bytes(128, 64), 2, 0.949f, 4.69f, 0.63f},
    {128, 128, 4, 4 * stage_bytes(128, 128), 1, 0.609f, 4.66f, 1.0f},
    {256, 128, 8, 3 * stage_bytes(256, 128), 1, 0.797f, 4.38f, 0.94f},
    {256, 256, 8, 2 * stage_bytes(256, 256), 1, 1.442f, 8.53f, 0.70f},
};

template <typename G, bool GATED, bool LORA>
const void* gemm_fn(int kind) {
  if constexpr (LORA) {
    return kind == FLP_GEMM_256x128 ? (const void*)gemm_kernel<G, 4, 2, 4, 3, false, GATED, true>
                                    : (const void*)gemm_kernel<G, 4, 2, 8, 2, true, GATED, true>;
  } else {
    switch (kind) {
      case FLP_GEMM_64x32: return (const void*)gemm_kernel<G, 1, 2, 1, 4, false, GATED, false>;
      case FLP_GEMM_128x64: return (const void*)gemm_kernel<G, 2, 2, 2, 3, false, GATED, false>;
      case FLP_GEMM_128x128: return (const void*)gemm_kernel<G, 2, 2, 4, 4, false, GATED, false>;
      case FLP_GEMM_256x128: return (const void*)gemm_kernel<G, 4, 2, 4, 3, false, GATED, false>;
      default: return (const void*)gemm_kernel<G, 4, 2, 8, 2, true, GATED, false>;
    }
  }
}

const void* gemm_entry(int dtype, int kind, bool gated, bool lora) {
  const auto pick = [&](auto g) -> const void* {
    using G = decltype(g);
    return gated ? (lora ? gemm_fn<G, true, true>(kind) : gemm_fn<G, true, false>(kind))
                 : (lora ? gemm_fn<G, false, true>(kind) : gemm_fn<G, false, false>(kind));
  };
  return dtype == FLP_F16 ? pick(GF16{}) : pick(GBF16{});
}

// the kernels that use more than 64 KiB of LDS have to say so once (pools on different threads share it)
flp_status gemm_attrs() {
  static std::atomic<bool> done{false};
  if (done.load(std::memory_order_acquire)) return FLP_OK;
  for (int dtype : {FLP_F16, FLP_BF16})
    for (int kind = 0; kind < FLP_GEMM_KINDS; ++kind)
      for (int gated = 0; gated < 2; ++gated)
        for (int lora = 0; lora < 2; ++lora)
          if (!lora || kind >= FLP_GEMM_256x128)
            FLP_TRY_HIP(hipFuncSetAttribute(gemm_entry(dtype, kind, gated, lora), hipFuncAttributeMaxDynamicSharedMemorySize,
                                            kCfg[kind].lds));
  done.store(true, std::memory_order_release);
  return FLP_OK;
}

}  // namespace

size_t flp_gemm_part_bytes(const FlpGemmPlan& plan, int M, int n_proj, const int* N) {
  size_t n = 0;
  for (int p = 0; p < n_proj; ++p) n += (size_t)N[p];
  return (size_t)plan.splits * M * n * 4;
}

// The plan with the least estimated time: rounds of workgroups x (k tiles of a slice x time per k tile + start-up),
// at least the time the matrices take from memory, plus the slices' way through memory and the kernel that adds them.
FlpGemmPlan flp_gemm_plan(int M, int K, int n_proj, const int* N, unsigned allow, size_t max_part_bytes) {
  FlpGemmPlan best{FLP_GEMM_128x128, 1, 0.f};
  double best_us = 1e30, n_all = 0;
  bool split_ok = !(allow & FLP_GEMM_NO_SPLIT);
  for (int p = 0; p < n_proj; ++p) {
    n_all += N[p];
    split_ok = split_ok && N[p] % 4 == 0;
  }
  const int nk = K / GK;
  for (int kind = (allow & FLP_GEMM_LARGE_ONLY) ? FLP_GEMM_256x128 : 0; kind < FLP_GEMM_KINDS; ++kind) {
    const GemmCfg& c = kCfg[kind];
    int64_t f_tiles = 0;
    for (int p = 0; p < n_proj; ++p) f_tiles += (N[p] + c.ft - 1) / c.ft;
    const int64_t m_tiles = (M + c.mt - 1) / c.mt, tiles = f_tiles * m_tiles;
    for (int s = 1; s <= 16; s = s < 4 ? s + 1 : s < 8 ? s + 2 : s + 4) {
      if (s > 1 && (!split_ok || nk / s < 4 || (double)s * M * n_all * 4 > (double)max_part_bytes)) break;
      const double wgs = (double)tiles * s, slots = 256.0 * c.per_cu;
      const double full = std::floor(wgs / slots), rest = wgs - full * slots;
      const double share = rest <= 0 ? 0 : c.per_cu == 1 ? c.part + (1 - c.part) * rest / 256
                                                         : std::max((double)c.part, std::ceil(rest / 256) / c.per_cu);
      double us = (full + share) * ((double)nk / s * c.step_us + c.fill_us);
      us = std::max(us, n_all * K * 2 / 8.36e6 + 3.3);
      // slices written and read, and the launch that adds them (also where the LoRA expand step of a small batch does: the
      // constants were fitted with that launch, and its share of the expand step has not been told apart)
      if (s > 1) us += (double)s * M * n_all * 8 / 4.64e6 + 3.5;
      if (us < best_us) {
        best_us = us;
        best = FlpGemmPlan{kind, s, (float)us};
      }
    }
  }
  return best;
}

bool flp_gemm_offsets_fit(int kind, int M, int64_t ld_x) {
  return ld_x <= (int64_t)UINT32_MAX / 2 / std::min(kCfg[kind].mt, M);
}

extern "C" void flp_dense_plan(int32_t M, int32_t K, int32_t n_proj, const int32_t* N, int32_t large_only, int64_t room,
                               int32_t* kind, int32_t* splits) {
  const FlpGemmPlan p = flp_gemm_plan(M, K, n_proj, N, large_only ? FLP_GEMM_NO_SPLIT | FLP_GEMM_LARGE_ONLY : 0,
                                      room < 0 ? kLayerSliceBytes : (size_t)room);
  *kind = p.kind;
  *splits = p.splits;
}

extern "C" int32_t flp_dense_tile(int32_t block, int32_t n_units, int32_t m_tiles, int32_t* u, int32_t* tm) {
  int gf, bands;
  tile_blocks(m_tiles, &gf, &bands);
  return tile_of_block(block, n_units, m_tiles, gf, bands, u, tm);
}

flp_status flp_launch_gemm(int dtype, const void* x, int64_t ld_x, int M, int K, const FlpGemmPlan& plan, int n_proj,
                           const FlpGemmOut* out, bool gated, const FlpGemmLora* lora, hipStream_t stream) {
  if (M <= 0 || K <= 0 || n_proj <= 0) return FLP_OK;
  if (K % GK != 0) {
    flp_set_error("dense product: d_in %d is not a multiple of %d", K, GK);
    return FLP_ENOTSUP;
  }
  // a tile's token rows are addressed with 32-bit byte offsets from its first one: rows too far apart for that take the
  // narrowest tile (32 tokens that span 4 GiB are refused)
  const int kind = !lora && !flp_gemm_offsets_fit(plan.kind, M, ld_x) ? FLP_GEMM_64x32 : plan.kind;
  if (!flp_gemm_offsets_fit(kind, M, ld_x)) {
    flp_set_error("dense product: rows of the input are %lld elements apart", (long long)ld_x);
    return FLP_ENOTSUP;
  }
  const GemmCfg& c = kCfg[kind];
  if (lora && (plan.kind < FLP_GEMM_256x128 || plan.splits != 1)) {
    flp_set_error("dense product: the LoRA epilogue needs whole contractions on the large tiles");
    return FLP_ENOTSUP;
  }
  FLP_TRY(gemm_attrs());
  FlpGemmArgs a{};
  a.x = (const uint16_t*)x;
  a.ld_x = ld_x;
  a.M = M;
  a.K = K;
  a.n_proj = n_proj;
  a.splits = plan.splits;
  a.m_tiles = (M + c.mt - 1) / c.mt;
  for (int p = 0; p < n_proj; ++p) {
    FlpGemmProj& pr = a.proj[p];
    pr.w = (const uint16_t*)out[p].w;
    pr.w2 = (const uint16_t*)out[p].w2;
    pr.y = (uint16_t*)out[p].y;
    pr.ld_y = out[p].ld_y;
    pr.part = out[p].part;
    pr.N = out[p].N;
    pr.tile0 = a.f_tiles;
    a.f_tiles += (pr.N + c.ft - 1) / c.ft;
    if (plan.splits > 1) pr.y = nullptr;                 // whoever adds the slices writes it: gemm_reduce, or the LoRA expand step
  }
  tile_blocks(a.m_tiles, &a.gf, &a.bands);
  const int64_t n_tiles = (int64_t)a.f_tiles * a.splits * a.m_tiles, grid = (n_tiles + 7) / 8 * 8;    // 256s, then eighths rounded up
  if (grid > INT32_MAX) {
    flp_set_error("dense product: %lld workgroups, too many for one launch", (long long)grid);
    return FLP_ENOTSUP;
  }
  GemmLoraArgs la{};
  if (lora)
    for (int p = 0; p < (gated ? 2 : n_proj); ++p) la.p[p] = lora[p];
  NoLora none;
  void* args[2] = {&a, lora ? (void*)&la : (void*)&none};
  FLP_TRY_HIP(hipLaunchKernel(gemm_entry(dtype, kind, gated, lora != nullptr), dim3((unsigned)grid), dim3(64 * c.waves),
                              args, (size_t)c.lds, stream));
  return FLP_OK;
}

flp_status flp_launch_gemm_reduce(int dtype, int M, int n_proj, const FlpGemmOut* out, int splits, bool gated, int mode,
                                  hipStream_t stream) {
  FlpGemmArgs a{};
  a.M = M;
  a.n_proj = n_proj;
  a.splits = splits;
  int64_t most = 0;
  for (int p = 0; p < n_proj; ++p) {
    FlpGemmProj& pr = a.proj[p];
    pr.y = (uint16_t*)out[p].y;
    pr.ld_y = out[p].ld_y;
    pr.part = out[p].part;
    pr.N = out[p].N;
    most = std::max(most, (int64_t)M * (gated ? pr.N / 2 : pr.N) / 4);
  }
  const dim3 grid((unsigned)((most + 255) / 256), (unsigned)n_proj);
  if (dtype == FLP_F16 && gated)
    hipLaunchKernelGGL((gemm_reduce_kernel<GF16, true>), grid, dim3(256), 0, stream, a, mode);
  else if (dtype == FLP_F16)
    hipLaunchKernelGGL((gemm_reduce_kernel<GF16, false>), grid, dim3(256), 0, stream, a, mode);
  else if (gated)
    hipLaunchKernelGGL((gemm_reduce_kernel<GBF16, true>), grid, dim3(256), 0, stream, a, mode);
  else
    hipLaunchKernelGGL((gemm_reduce_kernel<GBF16, false>), grid, dim3(256), 0, stream, a, mode);
  FLP_TRY_HIP(hipGetLastError());
  return FLP_OK;
}

flp_status flp_launch_transpose16(const void* w, void* wt, int K, int N, hipStream_t stream) {
  hipLaunchKernelGGL(transpose16_kernel, dim3((N + 63) / 64, (K + 63) / 64), dim3(256), 0, stream, (const uint16_t*)w,
                     (uint16_t*)wt, K, N);
  FLP_TRY_HIP(hipGetLastError());
  return FLP_OK;
}

flp_status flp_launch_gemm_f32(const float* x, int64_t ld_x, const float* w, int w_layout, float* y, int64_t ld_y, int M, int N,
                               int K, hipStream_t stream) {
  const dim3 grid((unsigned)((N + 15) / 16), (unsigned)((M + 15) / 16));
  if (w_layout)
    hipLaunchKernelGGL(gemm_f32_kernel<true>, grid, dim3(256), 0, stream, x, ld_x, w, y, ld_y, M, N, K);
  else
    hipLaunchKernelGGL(gemm_f32_kernel<false>, grid, dim3(256), 0, stream, x, ld_x, w, y, ld_y, M, N, K);
  FLP_TRY_HIP(hipGetLastError());
  return FLP_OK;
}
