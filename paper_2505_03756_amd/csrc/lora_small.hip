// Batched heterogeneous LoRA of up to kLoraSmallTokens tokens, 16-bit pools (paper Eq. 1 / Eq. 2 in row-vector form,
// y = base + s (x A^T) B; section 2.1: tokens of different adapters share one batch; section 4.3: adapters live in pool
// blocks as rank rows).
//
// In a decode batch a few tokens share each adapter and the adapters' pages are the traffic; in a single prompt all tokens
// share one.  Either way the tokens of an adapter are taken in token order, sixteen at a time, as the sixteen columns of a
// matrix instruction, so that a page is read once for all of them.  Who belongs together is found by every wave itself from
// the batch's adapter ids (ballots over all of them): that costs a microsecond, a launch that sorts them costs eight.  Bound
// by latency: a workgroup is one wave, which meets no barrier, has its loads in flight together and gives its place back at
// once where it has nothing to do (with four waves to a workgroup the idle ones held theirs: 30 % longer at 256 tokens).
//
//   shrink  one wave per (sixteen tokens, projection, slice of d_in, 32 ranks): v^T = A x^T with mfma_f32_16x16x32.  The
//           slices' sums stay apart, the expand step adds them in order.
//   expand  one wave per (sixteen tokens, projection, 128 columns): y^T += s B^T v^T with fp32 instructions, so that v
//           keeps its 32 bits.  16x16x4: column 8 m + tau of the chunk is row m of tile tau (a lane reads 8 neighbouring
//           columns of a page row and ends up with 32 neighbouring columns of one token), rank 4 k + i of a rank tile is slot k
//           of step i.  Groups of up to four tokens take 4x4x1 instructions, a quarter of the time in the matrix pipe.  In a
//           layer any eight tokens of which belong to one or two sequences a wave looks after eight neighbouring ones: with one each, a
//           499-token prompt launches 48 000 waves of which one in sixteen has something to do, and the launch takes longer than
//           the work.  (For decode batches the form costs registers, and groups in turn: 300 single tokens 165 -> 200 us.)
//
// Both steps add in short chains: four chunks of d_in at a time, then those sums; a rank tile at a time (4x4x1: half a tile), then
// the tiles.  Error of the branch against 64 bits (fp16, widths 4096 to 8192, 2-norm over 2-norm, 8 to 1000 tokens):
//   rank 64    1.6e-7 with the vector kernels, 2.1e-7 with one chain over the ranks and eight chunks at a time, 1.5e-7 with these
//   rank 16    1.8e-7 to 2.1e-7, 5 % more, 1 % less (2 % more where 4096 coefficients are in two slices; two running sums per
//              slice mend that for 1 to 7 % of the time)
//
// What keeps a batch of many adapters of high rank fast is how much of their pages is in flight: 64 ranks of one token are two
// waves with a 20 KiB ring each (one wave with 30 KiB: shrink step 207 against 198 us for 300 tokens of 64 x 8 heads); groups of
// up to eight tokens fetch eight rows of x instead of sixteen, which leaves room for a fourth stage.  Above 512 tokens the waves
// with nothing to do are so many that one wave takes all 64 ranks (500 + 500 tokens, rank 64: 109 against 113 us).  The expand
// step's grid holds the column chunks that there are, projection by projection (64 x 8 heads: three times the chunks of q had
// two thirds of the waves leave at once: 85 -> 67 us).
//
// Measured on MI355X with the adapters' pages out of the caches, us: the per-token vector kernels / these
//                                                             q,k,v           o
//   32 / 32 heads    256 tokens, 92 adapters of ranks 8-64    93.6 / 73.5     43.9 / 40.2
//   bf16             200 tokens, 100 adapters of ranks 8-64   75.7 / 71.5     41.4 / 35.9
//                    8 tokens of rank 16                      19.7 / 17.5     18.3 / 15.2
//                    499 tokens of one adapter of rank 16     64.1 / 37.8     33.8 / 26.5   (a wave per token)
//                    64 tokens, 500 adapters of rank 64       84.2 / 88.2     40.0 / 40.5
//   40 / 40 heads    1000 tokens of 2 sequences, rank 32       416 / 102       157 / 49.4
//   64 / 8 heads     1000 tokens of 2 sequences, rank 64       652 / 142       321 / 81.5
//   bf16             200 tokens, 100 adapters of rank 64       154 / 153      93.7 / 94.0
//                    128 tokens, 500 adapters of rank 64       159 / 165       102 / 103
//                    300 tokens, 500 adapters of rank 64       247 / 262       156 / 163
//                    300 tokens, 500 adapters of rank 16       115 / 114      68.5 / 64.2
// Where nearly every token has an adapter of rank 64 of its own the vector kernels stay 3 to 6 % ahead (their workgroups read
// whole KiB of a page row); which batches those are is only known on the device.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "flp_internal.h"
#include "flp_types.h"

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef _Float16 h16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 b16x8 __attribute__((ext_vector_type(8)));

struct SF16 {
  typedef h16x8 vec;
  typedef F16 S;
  static __device__ __forceinline__ f32x4 mfma(vec a, vec b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
  }
};
struct SBF16 {
  typedef b16x8 vec;
  typedef BF16 S;
  static __device__ __forceinline__ f32x4 mfma(vec a, vec b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
  }
};

// For token t of adapter ad (>= 0): the batch's tokens with the same adapter, in token order, are taken sixteen at a time and
// the first of each sixteen works for all of them.  Returns how many tokens t works for (0: t is not a first); lane l gets
// the index of token l % 16 of them in `tok` (t past the last one).  Wave-uniform; T <= kLoraSmallTokens.
__device__ __forceinline__ int sixteen(const int32_t* __restrict__ token_adapter, int T, int t, int ad, int* tok) {
  const int lane = threadIdx.x;
  constexpr int W = kLoraSmallTokens / 64;
  int ids[W];
#pragma unroll
  for (int w = 0; w < W; ++w) ids[w] = 64 * w + lane < T ? token_adapter[64 * w + lane] : -1;
  uint64_t mask[W];
  int before = 0;
#pragma unroll
  for (int w = 0; w < W; ++w) {
    mask[w] = __ballot(ids[w] == ad);
    if (64 * w <= t) before += __popcll(t >= 64 * w + 63 ? mask[w] : mask[w] & ((1ull << (t & 63)) - 1));
  }
  if (t % 64 == 63) before -= 1;                       // the word's whole popcount holds t itself
  *tok = t;
  if (before % 16) return 0;
  int n = 0;
#pragma unroll
  for (int w = 0; w < W; ++w) {
    uint64_t m = 64 * w + 63 < t ? 0 : 64 * w <= t ? mask[w] & ~((1ull << (t & 63)) - 1) : mask[w];
    while (m && n < 16) {
      const int i = 64 * w + __ffsll((long long)m) - 1;
      if ((lane & 15) == n) *tok = i;
      m &= m - 1;
      ++n;
    }
  }
  return n;
}

// M0 is named as clobbered so that no pass keeps a value of its own alive in it across the statement; the
// compiler notes that it reserves the register, which is the point.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void sload_lds16(uint64_t addr, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(addr), "s"(lds) : "memory", "m0");
}
#pragma clang diagnostic pop
typedef __attribute__((address_space(3))) uint8_t s_lds_u8;

template <typename T>
__device__ __forceinline__ T load_global(uint64_t addr) {
  return *reinterpret_cast<const __attribute__((address_space(1))) T*>(addr);
}

// lane rho's address (of a page row), as seen by the lane that asks for rank `from`
__device__ __forceinline__ uint64_t address_of(const uint16_t* mine, int from) {
  const uint64_t ad = (uint64_t)(uintptr_t)mine;
  return (uint64_t)(uint32_t)__shfl((int)(uint32_t)ad, from) | (uint64_t)(uint32_t)__shfl((int)(ad >> 32), from) << 32;
}

// v of one group of up to 8 NX tokens for NB tiles of 16 ranks over the chunks [c0, c1) of 64 coefficients.  The rows of x and of A travel as whole
// 128-byte lines (8 rows per instruction) into a ring in LDS that belongs to this wave alone, so its own waits are all
// the order it needs.  Piece j (16 bytes) of row r sits in slot j ^ ((r >> 1) & 7).  (Straight from global memory in operand
// layout, 64 bytes of 16 rows per instruction, rows that are a multiple of 8 KiB apart met in one cache set.)
template <typename L, int NB, int NX, int kLds>
__device__ __forceinline__ void shrink_group(uint8_t* smem, const uint16_t* xrow, const uint16_t* arow, int tok, int64_t ld_x, int r,
                                             int c0, int c1, int rotate, f32x4 (&v)[NB]) {
  typedef typename L::vec vec;
  constexpr int NPER = NX + 2 * NB, kStage = 1024 * NPER, ST = kLds / kStage < 6 ? kLds / kStage : 6;
  static_assert(ST >= 3, "two chunks in flight behind the one that is multiplied");
  const int lane = threadIdx.x, m16 = lane & 15, kg = lane >> 4;
  uint64_t addr[NPER];
#pragma unroll
  for (int i = 0; i < NPER; ++i) {
    const int row = 8 * (i < NX ? i : (i - NX) & 1) + (lane >> 3), piece = (lane & 7) ^ ((row >> 1) & 7);
    if (i < NX) {
      addr[i] = (uint64_t)(uintptr_t)(xrow + (int64_t)__shfl(tok, row) * ld_x + 8 * piece);
    } else {
      const int rho = 16 * ((i - NX) / 2) + row;         // ranks past the adapter's read its first row, their v is zeroed
      addr[i] = address_of(arow, rho < r ? rho : 0) + 16 * piece;
    }
  }
  const uint32_t lds0 = (uint32_t)(uintptr_t)(s_lds_u8*)smem;
  const int n = c1 - c0;
  // rows are often a power of two bytes apart: waves start at different chunks and wrap around, so that they do not all ask
  // the same memory channels at the same time
  const int start = rotate % n;
  auto issue = [&](int c, int st) {                    // past the end: the last chunk again, into a free stage
    int cc = (c < n ? c : n - 1) + start;
    cc = c0 + (cc < n ? cc : cc - n);
#pragma unroll
    for (int i = 0; i < NPER; ++i) sload_lds16(addr[i] + (uint64_t)cc * 128, lds0 + (uint32_t)(st * kStage + 1024 * i));
  };
  f32x4 acc[NB][2];
#pragma unroll
  for (int i = 0; i < NB; ++i) v[i] = acc[i][0] = acc[i][1] = f32x4{0.f, 0.f, 0.f, 0.f};
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");      // only chunk loads are in flight below
#pragma unroll
  for (int c = 0; c < ST - 1; ++c) issue(c, c);
  const int off = m16 * 128 + ((kg ^ (m16 >> 1)) << 4);  // k step 0; step 1 is slot + 4: offset ^ 64
  const int xm = NX == 1 ? m16 & 7 : m16, xoff = xm * 128 + ((kg ^ (xm >> 1)) << 4);     // NX == 1: columns past the eighth repeat
  int st = 0, st_load = ST - 1;
  for (int c = 0; c < n; ++c) {
    // chunk c has landed, and the reads of chunk c - 1, whose stage is filled next, are done
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((ST - 2) * NPER) : "memory");
    issue(c + ST - 1, st_load);
    const uint8_t* buf = smem + st * kStage;
#pragma unroll
    for (int k2 = 0; k2 < 2; ++k2) {
      const vec xf = *reinterpret_cast<const vec*>(buf + (xoff ^ (k2 << 6)));
#pragma unroll
      for (int i = 0; i < NB; ++i)
        acc[i][k2] = L::mfma(*reinterpret_cast<const vec*>(buf + 1024 * (NX + 2 * i) + (off ^ (k2 << 6))), xf, acc[i][k2]);
    }
    st = st + 1 == ST ? 0 : st + 1;
    st_load = st_load + 1 == ST ? 0 : st_load + 1;
    if ((c & 3) == 3 || c + 1 == n) {                  // sums of four chunks, then of those: shorter chains of roundings
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        v[i] += acc[i][0] + acc[i][1];
        acc[i][0] = acc[i][1] = f32x4{0.f, 0.f, 0.f, 0.f};
      }
    }
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");     // the look-ahead loads must land before the LDS is released
}

// NT: tiles of 16 ranks the launch allows for; NB: those that a wave takes (NT == 4: two, by two waves, or all four)
template <typename L, int NT, int NB>
__global__ __launch_bounds__(64) void lora_small_shrink_kernel(FlpLoraArgs a, FlpLoraSmall c) {
  constexpr int kLds = NB == 4 ? 30 * 1024 : NT == 4 ? 20 * 1024 : 24 * 1024;
  __shared__ __attribute__((aligned(1024))) uint8_t smem[kLds];
  const int lane = threadIdx.x, m16 = lane & 15, kg = lane >> 4;
  const int t = blockIdx.x;
  const int ks = blockIdx.y % c.k_splits, p = blockIdx.y / c.k_splits;
  FlpLoraGroup* rec = c.groups + t;
  const bool writes = blockIdx.y + blockIdx.z == 0;    // one of the token's waves leaves the record for the expand step
  const int ad = __builtin_amdgcn_readfirstlane(a.token_adapter[t]);
  int r = 0, tok = t, n = 0;
  if (ad >= 0 && ad < a.n_adapters) {
    r = __builtin_amdgcn_readfirstlane(a.rank[ad]);
    r = r < a.max_rank ? r : a.max_rank;
    n = sixteen(a.token_adapter, a.T, t, ad, &tok);
    if (r <= 0) n = 0;
  }
  const bool lone = n == 0 && (r <= 0 || ad < 0 || ad >= a.n_adapters);     // no branch: only slices of its base to be added
  if (writes) {
    if (lane < 16) rec->tok[lane] = tok;
    if (lane == 0) {
      rec->n = lone ? 1 : n;
      rec->r = lone ? 0 : r;
      rec->scale = n ? a.scale[ad] : 0.f;
    }
    if (lone && lane == 0) rec->tok[0] = t;
    if (n && lane < a.n_proj) {
      rec->tab[lane] = a.proj[lane].b_tab_off[ad];
      rec->row[lane] = a.proj[lane].b_row_base[ad];
    }
  }
  const int rank0 = NB < NT ? 16 * NB * (int)blockIdx.z : 0;   // the wave's first rank
  if (n == 0 || rank0 >= r) return;
  r -= rank0;
  const flp_lora_proj& pr = a.proj[p];
  const int rpb = (int)(a.block_elems / a.d_in);
  const int row = pr.a_row_base[ad] + rank0 + (lane < r ? lane : 0);       // lane rho looks up the page row of rank rank0 + rho
  const uint16_t* const arow = reinterpret_cast<const uint16_t*>(a.pool) +
                               (int64_t)a.tables[pr.a_tab_off[ad] + row / rpb] * a.block_elems + (int64_t)(row % rpb) * a.d_in;
  const uint16_t* const x = reinterpret_cast<const uint16_t*>(a.x);
  const int chunks = a.d_in / 64, c0 = chunks * ks / c.k_splits, c1 = chunks * (ks + 1) / c.k_splits;
  // lane (token m16, ranks 4 kg .. 4 kg + 3 of a tile)
  float* const vp = a.v + (((int64_t)ks * a.T + tok) * a.n_proj + p) * (16 * NT) + rank0 + 4 * kg;
  auto run = [&](auto tiles, auto x_loads) {
    constexpr int B = decltype(tiles)::value, NX = decltype(x_loads)::value;
    f32x4 v[B];
    shrink_group<L, B, NX, kLds>(smem, x, arow, tok, a.ld_x, r, c0, c1, t + t / 16 + p, v);
#pragma unroll
    for (int nt = 0; nt < B; ++nt) {
#pragma unroll
      for (int i = 0; i < 4; ++i) v[nt][i] = 16 * nt + 4 * kg + i < r ? v[nt][i] : 0.f;
      if (m16 < n) *reinterpret_cast<f32x4*>(vp + 16 * nt) = v[nt];
    }
  };
  const auto by_tokens = [&](auto tiles) {
    if (n <= 8)
      run(tiles, std::integral_constant<int, 1>{});
    else
      run(tiles, std::integral_constant<int, 2>{});
  };
  if (NB == 1 || r <= 16)
    by_tokens(std::integral_constant<int, 1>{});
  else if (NB == 2 || r <= 32)
    by_tokens(std::integral_constant<int, NB < 2 ? 1 : 2>{});
  else
    by_tokens(std::integral_constant<int, NB>{});
}

// the slices' sums in order, B of them requested together
template <int B>
__device__ __forceinline__ f32x4 sum_slices(const float* vp, int64_t slice, int n) {
  f32x4 v = {0.f, 0.f, 0.f, 0.f};
  for (int k = 0; k < n; k += B) {
    f32x4 q[B];
#pragma unroll
    for (int i = 0; i < B; ++i) q[i] = *reinterpret_cast<const f32x4*>(vp + (k + i < n ? k + i : n - 1) * slice);
#pragma unroll
    for (int i = 0; i < B; ++i)
      if (k + i < n) v = k + i ? v + q[i] : q[i];
  }
  return v;
}

// Adds s * delta to 8 NP columns of a token: to the unrounded base (four columns of it, base(i)), or to y itself.  One function for
// all forms of the kernel, also for the sake of the last bit: the compiler turns some of these products and their rounding to fp16
// into one instruction that rounds once, and some into two.
template <typename S, int NP, typename B, typename F>
__device__ __forceinline__ void add_to_y(uint16_t* yp, bool has_base, B base, const u32x4 (&yraw)[NP], int left, float sc, F delta) {
#pragma unroll
  for (int i = 0; i < NP; ++i) {
    if (8 * i >= left) break;
    uint16_t y8[8];
    if (has_base) {
      const f32x4 lo = base(2 * i), hi = base(2 * i + 1);
#pragma unroll
      for (int q = 0; q < 8; ++q) y8[q] = S::from_float(fmaf(sc, delta(i, q), q < 4 ? lo[q & 3] : hi[q & 3]));
    } else {
      __builtin_memcpy(y8, &yraw[i], 16);
#pragma unroll
      for (int q = 0; q < 8; ++q) y8[q] = S::from_float(fmaf(sc, delta(i, q), S::to_float(y8[q])));
    }
    u32x4 raw;
    __builtin_memcpy(&raw, y8, 16);
    *reinterpret_cast<u32x4*>(yp + 8 * i) = raw;
  }
}

// The group of n tokens of rank r that token t works for, 128 columns.  NT: tiles of 16 ranks the launch allows for; v_lds: [token
// (of 4)][four ranks]
template <typename L, int NT, bool LONG>
__device__ __forceinline__ void expand_group(const FlpLoraArgs& a, const FlpLoraSmall& c, int p, int t, int n, int r, int col0,
                                             f32x4* v_lds) {
  typedef typename L::S S;
  const int lane = threadIdx.x, m16 = lane & 15, kg = lane >> 4;
  const flp_lora_proj& pr = a.proj[p];
  const FlpLoraGroup* __restrict__ rec = c.groups + t;
  const int64_t base_slice = (int64_t)a.T * pr.d_out;
  const int slices = a.base_slices[p];
  const auto base_at = [&](const float* bp) {
    return [=](int i) { return sum_slices<4>(bp + 4 * i, base_slice, slices); };
  };
  if (r == 0) {                                        // a token without a branch: its product has only to be added up
    const int f0 = col0 + 8 * lane;
    if (slices <= 1 || lane >= 16 || f0 >= pr.d_out) return;
    const u32x4 none[1] = {u32x4{0u, 0u, 0u, 0u}};
    add_to_y<S, 1>(reinterpret_cast<uint16_t*>(pr.y) + (int64_t)t * pr.ld_y + f0, true,
                   base_at(a.base32[p] + (int64_t)t * pr.d_out + f0), none, pr.d_out - f0, 0.f, [](int, int) { return 0.f; });
    return;
  }
  const int rpb = (int)(a.block_elems / pr.d_out);
  constexpr int RP = 16 * NT;
  // lane rho looks up the page row of rank rho
  const int row = rec->row[p] + (lane < r ? lane : 0);
  const uint16_t* const mine = reinterpret_cast<const uint16_t*>(a.pool) +
                               (int64_t)a.tables[rec->tab[p] + row / rpb] * a.block_elems + (int64_t)(row % rpb) * pr.d_out;
  const float sc = rec->scale;
  const int64_t slice = (int64_t)a.T * a.n_proj * RP;
  const auto v_of = [&](int tok) { return a.v + ((int64_t)tok * a.n_proj + p) * RP; };

  if (n <= 4) {
    // up to four tokens: 4x4x1 instructions, 64 columns x 4 tokens of one rank each; row l of tile q is column 2 l + q of
    // the chunk, and a lane ends up with 8 neighbouring columns of token l % 4
    const int tok = rec->tok[lane & 3];
    const int f0 = col0 + 8 * (lane >> 2), fb = col0 + 2 * lane < pr.d_out ? col0 + 2 * lane : 0;
    uint16_t* const yp = reinterpret_cast<uint16_t*>(pr.y) + (int64_t)tok * pr.ld_y + f0;
    const float* const bp = a.base32[p] ? a.base32[p] + (int64_t)tok * pr.d_out + f0 : nullptr;
    u32x4 yraw[1] = {u32x4{0u, 0u, 0u, 0u}};
    if (!bp && f0 < pr.d_out) yraw[0] = *reinterpret_cast<const u32x4*>(yp);
    if (lane < RP) {
      const float* vp = v_of(rec->tok[lane / (RP / 4)]) + 4 * (lane % (RP / 4));
      f32x4 v = {0.f, 0.f, 0.f, 0.f};
      if (4 * (lane % (RP / 4)) < ((r + 15) & ~15)) v = sum_slices<8>(vp, slice, c.k_splits);
      v_lds[lane] = v;
    }
    __syncthreads();                                   // one wave: order only
    f32x4 acc[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
    uint32_t b[NT][16];                                // all ranks' coefficients in flight together
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
      if (16 * nt < r) {
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const uint64_t ad = (uint64_t)(uintptr_t)mine;
          const uint64_t base = (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)ad, 16 * nt + e) |
                                (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(ad >> 32), 16 * nt + e) << 32;
          b[nt][e] = load_global<uint32_t>(base + 2 * fb);
        }
      }
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      if (16 * nt >= r) break;
      f32x4 part[2][2];                                // ranks 8 h .. 8 h + 7 of the tile
#pragma unroll
      for (int h = 0; h < 2; ++h) part[h][0] = part[h][1] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int e4 = 0; e4 < 4; ++e4) {
        const f32x4 v = v_lds[(lane & 3) * (RP / 4) + 4 * nt + e4];
        f32x4(&to)[2] = part[e4 >> 1];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int e = 4 * e4 + i;
          const uint32_t w = 16 * nt + e < r ? b[nt][e] : 0u;
          to[0] = __builtin_amdgcn_mfma_f32_4x4x1f32(S::to_float((uint16_t)w), v[i], to[0], 0, 0, 0);
          to[1] = __builtin_amdgcn_mfma_f32_4x4x1f32(S::to_float((uint16_t)(w >> 16)), v[i], to[1], 0, 0, 0);
        }
      }
      acc[0] += part[0][0] + part[1][0];
      acc[1] += part[0][1] + part[1][1];
    }
    if ((lane & 3) < n) add_to_y<S, 1>(yp, bp, base_at(bp), yraw, pr.d_out - f0, sc, [&](int, int q) { return acc[q & 1][q >> 1]; });
    return;
  }

  const int tok = rec->tok[m16];
  const float* const vp = v_of(tok) + 4 * kg;
  f32x4 v[NT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    v[nt] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (16 * nt < r) v[nt] = sum_slices<4>(vp + 16 * nt, slice, c.k_splits);
  }
  const int fb = col0 + 8 * m16 < pr.d_out ? col0 + 8 * m16 : 0;    // widths are multiples of 8: a lane's columns are all in or all out
  const int f0 = col0 + 32 * kg;
  uint16_t* const yp = reinterpret_cast<uint16_t*>(pr.y) + (int64_t)tok * pr.ld_y + f0;
  const float* const bp = a.base32[p] ? a.base32[p] + (int64_t)tok * pr.d_out + f0 : nullptr;
  u32x4 yraw[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) yraw[i] = !bp && f0 + 8 * i < pr.d_out ? *reinterpret_cast<const u32x4*>(yp + 8 * i) : u32x4{0u, 0u, 0u, 0u};
  f32x4 acc[8];
  u32x4 b[NT][4];                                      // ranks 16 nt + 4 kg + i of the lane's 8 columns
#pragma unroll
  for (int nt = 0; nt < NT; ++nt)
    if (16 * nt < r) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
        b[nt][i] = load_global<u32x4>(address_of(mine, 16 * nt + 4 * kg + i) + 2 * fb);
    }
  f32x4 base[LONG ? 8 : 1];                            // LONG: an unrounded base is on its way beside the pages
  if constexpr (LONG)
    if (bp) {
#pragma unroll
      for (int i = 0; i < 8; ++i)
        if (f0 + 4 * i < pr.d_out)
          base[i] = slices == 1 ? *reinterpret_cast<const f32x4*>(bp + 4 * i) : sum_slices<4>(bp + 4 * i, base_slice, slices);
    }
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    if (16 * nt >= r) break;
    f32x4 part[8];                                     // of this rank tile: chains of 16 roundings
#pragma unroll
    for (int q = 0; q < 8; ++q) part[q] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const bool live = 16 * nt + 4 * kg + i < r;
      uint16_t e[8];
      __builtin_memcpy(e, &b[nt][i], 16);
#pragma unroll
      for (int q = 0; q < 8; ++q)
        part[q] = __builtin_amdgcn_mfma_f32_16x16x4f32(live ? S::to_float(e[q]) : 0.f, v[nt][i], part[q], 0, 0, 0);
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) acc[q] = nt ? acc[q] + part[q] : part[q];
  }
  if (m16 >= n) return;
  // lane (token m16, kg): element i of tile q is column 32 kg + 8 i + q of the chunk
  const auto delta = [&](int i, int q) { return acc[q][i]; };
  if constexpr (LONG)
    add_to_y<S, 4>(yp, bp, [&](int i) { return base[i]; }, yraw, pr.d_out - f0, sc, delta);
  else
    add_to_y<S, 4>(yp, bp, base_at(bp), yraw, pr.d_out - f0, sc, delta);
}

// LONG: a wave looks after kLoraLongBlock neighbouring tokens.  Waves per SIMD are asked for with LONG and with four rank tiles: there
// the compiler by itself spreads the accumulators over both register files and loses one or two waves.
template <typename L, int NT, bool LONG>
__global__ __launch_bounds__(64, LONG ? 2 : NT == 4 ? 3 : 1) void lora_small_expand_kernel(FlpLoraArgs a, FlpLoraSmall c) {
  __shared__ f32x4 v_lds[64 * NT / 4];
  const int lane = threadIdx.x;
  // the projections one after the other; columns vary fastest: rows are often a power of two bytes apart
  const unsigned blocks = LONG ? (unsigned)(a.T + kLoraLongBlock - 1) / kLoraLongBlock : (unsigned)a.T;
  int p = 0;
  unsigned unit = blockIdx.x, chunks = (unsigned)(a.proj[0].d_out + 127) / 128;
  while (unit >= chunks * blocks) {
    unit -= chunks * blocks;
    chunks = (unsigned)(a.proj[++p].d_out + 127) / 128;
  }
  const int t0 = (int)(unit / chunks) * (LONG ? kLoraLongBlock : 1), col0 = (int)(unit % chunks) * 128;
  if constexpr (LONG) {
    // lane i: how many tokens token t0 + i works for, and the rank
    const FlpLoraGroup* rec = c.groups + (t0 + lane < a.T ? t0 + lane : t0);
    const int n = rec->n, r = rec->r;
    for (uint64_t todo = __ballot(lane < kLoraLongBlock && t0 + lane < a.T && n > 0); todo; todo &= todo - 1) {
      const int i = __ffsll((long long)todo) - 1;
      __syncthreads();                                 // one wave: the last group's reads of v_lds stay before this one's writes
      expand_group<L, NT, LONG>(a, c, p, t0 + i, __builtin_amdgcn_readlane(n, i), __builtin_amdgcn_readlane(r, i), col0, v_lds);
    }
  } else {
    const int n = __builtin_amdgcn_readfirstlane(c.groups[t0].n);
    if (n > 0) expand_group<L, NT, LONG>(a, c, p, t0, n, __builtin_amdgcn_readfirstlane(c.groups[t0].r), col0, v_lds);
  }
}

template <typename L, int NT>
void launch(const FlpLoraArgs& a, const FlpLoraSmall& c, hipStream_t stream) {
  unsigned chunks = 0;
  for (int p = 0; p < a.n_proj; ++p) chunks += (unsigned)(a.proj[p].d_out + 127) / 128;
  dim3 gs((unsigned)a.T, (unsigned)(a.n_proj * c.k_splits));
  if (NT == 4 && a.T <= 512) {
    gs.z = 2;
    hipLaunchKernelGGL((lora_small_shrink_kernel<L, NT, NT == 4 ? 2 : NT>), gs, dim3(64), 0, stream, a, c);
  } else {
    hipLaunchKernelGGL((lora_small_shrink_kernel<L, NT, NT>), gs, dim3(64), 0, stream, a, c);
  }
  if constexpr (NT <= 2) {
    if (c.long_runs) {
      const dim3 gl(chunks * (unsigned)((a.T + kLoraLongBlock - 1) / kLoraLongBlock));
      hipLaunchKernelGGL((lora_small_expand_kernel<L, NT, true>), gl, dim3(64), 0, stream, a, c);
      return;
    }
  }
  hipLaunchKernelGGL((lora_small_expand_kernel<L, NT, false>), dim3(chunks * (unsigned)a.T), dim3(64), 0, stream, a, c);
}
template <typename L>
void launch(const FlpLoraArgs& a, const FlpLoraSmall& c, hipStream_t stream) {
  if (c.n_tiles == 1)
    launch<L, 1>(a, c, stream);
  else if (c.n_tiles == 2)
    launch<L, 2>(a, c, stream);
  else
    launch<L, 4>(a, c, stream);
}

}  // namespace

flp_status flp_launch_lora_small(int dtype, const FlpLoraArgs& a, const FlpLoraSmall& c, hipStream_t stream) {
  if (dtype == FLP_F32 || a.T > kLoraSmallTokens || a.d_in % 64) {
    flp_set_error("LoRA (small batches): dtype %d, %d tokens or d_in %d not supported", dtype, a.T, a.d_in);
    return FLP_ENOTSUP;
  }
  if (dtype == FLP_F16)
    launch<SF16>(a, c, stream);
  else
    launch<SBF16>(a, c, stream);
  FLP_TRY_HIP(hipGetLastError());
  return FLP_OK;
}
