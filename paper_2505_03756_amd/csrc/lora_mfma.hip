// Batched heterogeneous LoRA on the matrix cores, for 16-bit pools (paper Eq. 1 / Eq. 2 in
// row-vector form, y = base + s (x A^T) B; section 2.1: tokens of different adapters share
// one batch; section 4.3: adapters live in pool blocks as rank rows).
//
// Tokens are first grouped by adapter (lora.hip); a tile is up to 16*MT consecutive tokens of one adapter.  The
// rank-major page rows make 8 consecutive coefficients of one rank one 16-byte run, which is exactly a lane's share of a
// 16x16x32 operand of the shrink step.
//
//   shrink  v[t, rho] = sum_c x[t,c] A[rho,c]     M = tokens, N = ranks, K = d_in.  K is
//           split over the 4 waves of a workgroup (summed in LDS in a fixed order) and over
//           KS workgroups (partial sums in global memory, added in order by the expand
//           kernel), so that enough waves are in flight to stream x at HBM rate.
//   expand  y[t, o] += s sum_rho v[t,rho] B[rho,o]   M = tokens, N = columns, K = ranks.  v stays fp32: it is
//           split into a 16-bit high part and a 16-bit remainder that occupy the two halves of the K = 32
//           contraction (the B coefficients are fed to both halves).
#include <atomic>
#include <hip/hip_runtime.h>

#include "flp_internal.h"
#include "flp_types.h"

namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef _Float16 h16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 b16x8 __attribute__((ext_vector_type(8)));

struct LF16 {
  typedef h16x8 vec;
  typedef F16 S;
  static __device__ __forceinline__ f32x4 mfma(vec a, vec b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ void split(float v, _Float16* hi, _Float16* lo) {
    *hi = (_Float16)v;
    *lo = (_Float16)(v - (float)*hi);
  }
  typedef _Float16 elem;
};
struct LBF16 {
  typedef b16x8 vec;
  typedef BF16 S;
  static __device__ __forceinline__ f32x4 mfma(vec a, vec b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ void split(float v, __bf16* hi, __bf16* lo) {
    *hi = (__bf16)v;
    *lo = (__bf16)(v - (float)*hi);
  }
  typedef __bf16 elem;
};

template <typename V>
__device__ __forceinline__ V vec_from(u32x4 r) {
  V v;
  __builtin_memcpy(&v, &r, 16);
  return v;
}

// tile -> segment: largest s with tile_start[s] <= tile (tile < tile_start[n_seg])
__device__ __forceinline__ int find_segment(const int32_t* __restrict__ tile_start, int n_seg, int tile) {
  int lo = 0, hi = n_seg;   // invariant: tile_start[lo] <= tile < tile_start[hi]
  while (hi - lo > 1) {
    int mid = (lo + hi) >> 1;
    if (tile_start[mid] <= tile) lo = mid; else hi = mid;
  }
  return lo;
}

// ------------------------------------------------------------------------------- shrink
// ONEP: a workgroup takes ONE projection of its tile (the grid grows by the number of projections): with
// rank tiles NT >= 2 the accumulators and operand fragments of three projections at once leave one
// wave per SIMD, and the kernel, which lives on loads in flight, then runs at a fraction of HBM rate; x is
// re-read per projection, from L2.
template <typename L, int MT, int NT, bool ONEP>
__global__ __launch_bounds__(256) void lora_shrink_mfma_kernel(FlpLoraArgs a, FlpLoraMfma c) {
  typedef typename L::vec vec;
  constexpr int NPJ = ONEP ? 1 : FLP_MAX_PROJ;         // projections held by this workgroup
  extern __shared__ float red[];                       // [4 waves][n_acc][64 lanes]
  // Each XCD (workgroups are placed on the 8 XCDs round-robin by their linear id) takes a contiguous
  // eighth of the tiles with all their k splits: tiles of one adapter are neighbours, so its A pages
  // are fetched into one L2 instead of eight.  The launch covers gridDim.x / (8 k_splits) tiles per XCD
  // in one pass; with more segments than the host allowed for, a workgroup takes several tiles in turn.
  const int n_seg = *a.n_seg;
  const int n_tiles = a.tile_start[n_seg];
  const int per_xcd = (n_tiles + 7) / 8;
  const int per_tile = c.k_splits * (ONEP ? a.n_proj : 1);          // workgroups per tile
  const int ks = ((blockIdx.x >> 3) % per_tile) / (ONEP ? a.n_proj : 1);
  const int p_first = ONEP ? ((blockIdx.x >> 3) % per_tile) % a.n_proj : 0;   // local projection q is p_first + q
  const int n_pl = ONEP ? 1 : a.n_proj;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, row = lane & 15, kg = lane >> 4;
  const uint16_t* __restrict__ pool = reinterpret_cast<const uint16_t*>(a.pool);
  const int rpb = (int)(a.block_elems / a.d_in);
  for (int lt = (blockIdx.x >> 3) / per_tile; lt < per_xcd; lt += (gridDim.x >> 3) / per_tile) {
  const int tile = (blockIdx.x & 7) * per_xcd + lt;
  if (tile >= n_tiles) break;
  const int s = find_segment(a.tile_start, n_seg, tile);
  const int ad = a.seg_adapter[s];
  const int r = a.rank[ad] < a.max_rank ? a.rank[ad] : a.max_rank;
  const int TM = 16 * MT;
  const int pos0 = a.seg_start[s] + (tile - a.tile_start[s]) * TM;
  const int pos_end = a.seg_start[s + 1];

  const uint16_t* xp[MT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    int pos = pos0 + 16 * mt + row;
    pos = pos < pos_end ? pos : pos_end - 1;           // padding rows repeat the last token
    xp[mt] = reinterpret_cast<const uint16_t*>(a.x) + (int64_t)a.perm[pos] * a.ld_x + 8 * kg;
  }
  const uint16_t* ap[NPJ][NT];
  bool avalid[NT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) avalid[nt] = 16 * nt + row < r;
#pragma unroll
  for (int p = 0; p < NPJ; ++p)
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      ap[p][nt] = pool;
      if (p < n_pl && r > 0) {
        const flp_lora_proj& pr = a.proj[p_first + p];
        const int i = pr.a_row_base[ad] + (avalid[nt] ? 16 * nt + row : 0);
        ap[p][nt] = pool + (int64_t)a.tables[pr.a_tab_off[ad] + i / rpb] * a.block_elems +
                    (int64_t)(i % rpb) * a.d_in + 8 * kg;
      }
    }

  f32x4 acc[MT][NPJ][NT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int p = 0; p < NPJ; ++p)
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) acc[mt][p][nt] = f32x4{0.f, 0.f, 0.f, 0.f};

  const int kbeg = ks * c.k_per_split;
  const int kend = kbeg + c.k_per_split < a.d_in ? kbeg + c.k_per_split : a.d_in;
  const u32x4 zero4 = {0u, 0u, 0u, 0u};
  for (int c0 = kbeg + 32 * wave; c0 < kend; c0 += 128) {
    vec xf[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) xf[mt] = vec_from<vec>(*reinterpret_cast<const u32x4*>(xp[mt] + c0));
#pragma unroll
    for (int p = 0; p < NPJ; ++p) {
      if (p < n_pl) {
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
          if (16 * nt < r) {
            u32x4 raw = avalid[nt] ? *reinterpret_cast<const u32x4*>(ap[p][nt] + c0) : zero4;
            vec af = vec_from<vec>(raw);
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) acc[mt][p][nt] = L::mfma(xf[mt], af, acc[mt][p][nt]);
          }
        }
      }
    }
  }

  // ---- sum the four waves' partial tiles in a fixed order, then store
  const int n_acc = MT * n_pl * NT * 4;
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int p = 0; p < NPJ; ++p)
      if (p < n_pl)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
          for (int i = 0; i < 4; ++i)
            red[(wave * n_acc + ((mt * n_pl + p) * NT + nt) * 4 + i) * 64 + lane] = acc[mt][p][nt][i];
  __syncthreads();
  const int RP = 16 * NT;
  float* __restrict__ vout = a.v + ((int64_t)ks * c.v_rows + (int64_t)tile * TM) * a.n_proj * RP;
  for (int e = tid; e < n_acc * 64; e += 256) {
    const float sum = ((red[e] + red[n_acc * 64 + e]) + red[2 * n_acc * 64 + e]) + red[3 * n_acc * 64 + e];
    const int ln = e & 63, q = e >> 6;
    const int i = q & 3, nt = (q >> 2) % NT, p = ((q >> 2) / NT) % n_pl, mt = (q >> 2) / (NT * n_pl);
    const int trow = 16 * mt + (ln >> 4) * 4 + i, rho = 16 * nt + (ln & 15);
    vout[((int64_t)trow * a.n_proj + p_first + p) * RP + rho] = sum;
  }
  __syncthreads();                                     // the next tile reuses the reduction buffer
  }
}

// ------------------------------------------------------------------------------- shrink, ranks above 16
// The kernel above reads its operands straight from global memory in MFMA layout: 64-byte pieces of 16 rows
// per instruction.  With 2 or 4 rank tiles per token tile that is mostly A traffic from L2 in 64-byte
// requests, and the kernel runs far below the rate of the x stream.  Here a workgroup of four waves owns one
// (32-token tile, projection, k split) and walks its k range in chunks of 64 coefficients: the chunk's x
// rows (32 x 128 bytes) and A rows (16 NT x 128 bytes) travel as whole 128-byte lines into a ring of four LDS
// stages with direct global-to-LDS loads (inline assembly, own s_waitcnt vmcnt; three chunks ahead), slots
// XOR-swizzled by the row on the global side, and the waves split the (token tile, rank tile) pairs, so
// no reduction across waves is needed.  Ranks past the adapter's rank read the adapter's first row: their v
// entries are finite and meet zero coefficients in the expand kernel.
typedef __attribute__((address_space(3))) uint8_t l_lds_u8;
// M0 is named as clobbered so that no pass keeps a value of its own alive in it across the statement; the
// compiler notes that it reserves the register, which is the point.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void lload_lds16(uint64_t addr, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(addr), "s"(lds) : "memory", "m0");
}
#pragma clang diagnostic pop
constexpr int lvmcnt(int n) { return (n & 15) | ((n >> 4) << 14) | (7 << 4) | (15 << 8); }   // s_waitcnt vmcnt(n) only

template <typename L, int NT, int NPJ>
__global__ __launch_bounds__(256) void lora_shrink_lds_kernel(FlpLoraArgs a, FlpLoraMfma c) {
  typedef typename L::vec vec;
  // From rank 33 on a workgroup takes TWO neighbouring 32-token tiles of a segment (the first of each pair does
  // the work, the second exits): the adapter's A rows, which at rank 64 are twice the bytes of a 32-token x tile,
  // are then fetched once per 64 tokens (34B shapes: q,k,v call 1.47 -> 1.25 ms; at rank 32 it does not pay).
  // NPJ = 2, 3 (used with two rank tiles): the projections of the call are fused (their A rows sit behind each
  // other in a stage, x is fetched once for all of them); NPJ = 1: one projection per workgroup, taken from the
  // grid.
  constexpr int XT = NT >= 4 ? 4 : 2;                  // 16-token tiles per workgroup
  constexpr int kS = 4;                                // ring stages
  constexpr int kXB = 2048 * XT;                       // bytes of the x rows of a stage
  constexpr int kAB = 2048 * NT;                       // bytes of one projection's A rows
  constexpr int kStageB = kXB + NPJ * kAB;             // x rows, then A rows, 128 bytes each
  constexpr int NINS = 2 * XT + 2 * NT * NPJ;          // 1 KiB load instructions per chunk (8 rows each)
  static_assert(NINS % 4 == 0, "the waves share the load instructions of a chunk evenly");
  constexpr int NPER = NINS / 4;                       // of which each wave issues this many
  constexpr int NP = XT * NT * NPJ / 4;                // (projection, 16-token tile, rank tile) triples per wave
  static_assert(kS * kStageB <= 65536, "the ring fits the LDS of a static array");
  __shared__ __attribute__((aligned(1024))) uint8_t smem[kS * kStageB];
  const int n_seg = *a.n_seg;
  const int n_tiles = a.tile_start[n_seg];
  const int per_xcd = (n_tiles + 7) / 8;
  const int per_tile = c.k_splits * (NPJ == 1 ? a.n_proj : 1);
  const int ks = NPJ == 1 ? ((blockIdx.x >> 3) % per_tile) / a.n_proj : (blockIdx.x >> 3) % per_tile;
  const int p0 = NPJ == 1 ? ((blockIdx.x >> 3) % per_tile) % a.n_proj : 0;       // first (only) projection of this workgroup
  const int tid = threadIdx.x, lane = tid & 63, row16 = lane & 15, kg = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint16_t* __restrict__ pool = reinterpret_cast<const uint16_t*>(a.pool);
  const int rpb = (int)(a.block_elems / a.d_in);
  const uint32_t lds0 = (uint32_t)(uintptr_t)(l_lds_u8*)smem;
  for (int lt = (blockIdx.x >> 3) / per_tile; lt < per_xcd; lt += (gridDim.x >> 3) / per_tile) {
    const int tile = (blockIdx.x & 7) * per_xcd + lt;
    if (tile >= n_tiles) break;
    const int s = find_segment(a.tile_start, n_seg, tile);
    if (XT == 4 && ((tile - a.tile_start[s]) & 1)) continue;     // the second tile of a pair: its neighbour does it
    const bool second = XT == 4 && tile + 1 < a.tile_start[s + 1];  // the pair is complete
    const int ad = a.seg_adapter[s];
    const int r = a.rank[ad] < a.max_rank ? a.rank[ad] : a.max_rank;
    const int pos0 = a.seg_start[s] + (tile - a.tile_start[s]) * 32;
    const int pos_end = a.seg_start[s + 1];
    const int kbeg = ks * c.k_per_split;
    const int kend = kbeg + c.k_per_split < a.d_in ? kbeg + c.k_per_split : a.d_in;
    const int n_chunks = r > 0 ? (kend - kbeg) / 64 : 0;

    // ---- this lane's rows of the load instructions it issues: instruction j = wave + 4 i covers rows
    //      8 j .. 8 j + 7 of the x rows (j < 2 XT) or, for jj = j - 2 XT, rows 8 (jj % 2 NT) .. of the A tile of
    //      projection jj / 2 NT; lane l holds row l / 8, LDS slot l % 8, i.e. the row's logical 16-byte piece
    //      (l % 8) ^ (row % 8)
    uint64_t gaddr[NPER];
    uint32_t ldst[NPER];
#pragma unroll
    for (int i = 0; i < NPER; ++i) {
      const int j = wave + 4 * i, rl = lane >> 3;
      const uint16_t* rowp;
      int rowi;
      if (j < 2 * XT) {
        rowi = 8 * j + rl;
        int pos = pos0 + rowi;
        pos = pos < pos_end ? pos : pos_end - 1;       // padding rows repeat the last token
        rowp = reinterpret_cast<const uint16_t*>(a.x) + (int64_t)a.perm[pos] * a.ld_x;
        ldst[i] = 1024u * j;
      } else {
        const int jj = j - 2 * XT, pj = jj / (2 * NT), jr = jj % (2 * NT);
        const flp_lora_proj& pr = a.proj[p0 + pj];
        rowi = 8 * jr + rl;
        rowp = pool;
        if (r > 0) {
          const int ii = pr.a_row_base[ad] + (rowi < r ? rowi : 0);
          rowp = pool + (int64_t)a.tables[pr.a_tab_off[ad] + ii / rpb] * a.block_elems + (int64_t)(ii % rpb) * a.d_in;
        }
        ldst[i] = (uint32_t)(kXB + pj * kAB) + 1024u * jr;
      }
      gaddr[i] = (uint64_t)(uintptr_t)(rowp + kbeg + 8 * ((lane & 7) ^ (rowi & 7)));
    }
    auto issue_chunk = [&](int t) {
      const int tc = t < n_chunks ? t : n_chunks - 1;   // past the end: the last chunk again, into a free stage
      const uint32_t dst = lds0 + (uint32_t)(t & (kS - 1)) * kStageB;
#pragma unroll
      for (int i = 0; i < NPER; ++i) lload_lds16(gaddr[i] + (uint64_t)tc * 128, dst + ldst[i]);
    };

    f32x4 acc[NP];
    int offx[NP], offa[NP];
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
      const int pi = wave + 4 * i, pj = pi / (XT * NT), mt = (pi % (XT * NT)) / NT, nt = pi % NT;
      const int xr = 16 * mt + row16, ar = 16 * nt + row16;
      offx[i] = xr * 128 + ((kg ^ (xr & 7)) << 4);                 // k step 0; step 1 is slot + 4: offset ^ 64
      offa[i] = kXB + pj * kAB + ar * 128 + ((kg ^ (ar & 7)) << 4);
    }

    __builtin_amdgcn_s_waitcnt(lvmcnt(0));             // the loads above are in: only chunk loads are in flight below
    __syncthreads();                                   // the previous item's stages are no longer read
    if (n_chunks > 0) {
#pragma unroll
      for (int t = 0; t < kS - 1; ++t) issue_chunk(t);
    }
    for (int kt = 0; kt < n_chunks; ++kt) {
      __builtin_amdgcn_s_waitcnt(lvmcnt(2 * NPER));    // chunk kt has landed (kt + 1 and kt + 2 may be in flight)
      __syncthreads();
      issue_chunk(kt + kS - 1);
      const uint8_t* buf = smem + (kt & (kS - 1)) * kStageB;
#pragma unroll
      for (int k2 = 0; k2 < 2; ++k2)
#pragma unroll
        for (int i = 0; i < NP; ++i) {
          const vec xf = *reinterpret_cast<const vec*>(buf + (offx[i] ^ (k2 << 6)));
          const vec af = *reinterpret_cast<const vec*>(buf + (offa[i] ^ (k2 << 6)));
          acc[i] = L::mfma(xf, af, acc[i]);
        }
    }
    __builtin_amdgcn_s_waitcnt(lvmcnt(0));             // look-ahead loads past the last chunk must land before the ring is reused

    // lane (rank column n = lane % 16, token rows 4 kg .. 4 kg + 3) of each triple; the rows of the pair's second
    // tile follow the first one's in v
    const int RP = 16 * NT;
    float* __restrict__ vout = a.v + ((int64_t)ks * c.v_rows + (int64_t)tile * 32) * a.n_proj * RP;
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      const int pi = wave + 4 * i, pj = pi / (XT * NT), mt = (pi % (XT * NT)) / NT, nt = pi % NT;
      if (mt >= 2 && !second) continue;
#pragma unroll
      for (int e = 0; e < 4; ++e)
        vout[((int64_t)(16 * mt + 4 * kg + e) * a.n_proj + p0 + pj) * RP + 16 * nt + row16] = acc[i][e];
    }
  }
}

// The same staging for ranks up to 16, where the projections of a call are fused: the A rows of all NPJ
// projections (16 rank rows each) sit behind the 32 x rows of a chunk, x is fetched once for all of them,
// and the waves split the (token tile, projection) pairs.  When the load instructions of a chunk do not
// divide by four, a wave repeats one of its own loads, so that every wave has the same number in flight.
template <typename L, int NPJ>
__global__ __launch_bounds__(256) void lora_shrink_lds16_kernel(FlpLoraArgs a, FlpLoraMfma c) {
  typedef typename L::vec vec;
  constexpr int kS = 4;
  constexpr int kStageB = 4096 + 2048 * NPJ;
  constexpr int NINS = 4 + 2 * NPJ;
  constexpr int NPER = (NINS + 3) / 4;
  constexpr int NP = (2 * NPJ + 3) / 4;
  __shared__ __attribute__((aligned(1024))) uint8_t smem[kS * kStageB];
  const int n_seg = *a.n_seg;
  const int n_tiles = a.tile_start[n_seg];
  const int per_xcd = (n_tiles + 7) / 8;
  const int ks = (blockIdx.x >> 3) % c.k_splits;
  const int tid = threadIdx.x, lane = tid & 63, row16 = lane & 15, kg = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint16_t* __restrict__ pool = reinterpret_cast<const uint16_t*>(a.pool);
  const int rpb = (int)(a.block_elems / a.d_in);
  const uint32_t lds0 = (uint32_t)(uintptr_t)(l_lds_u8*)smem;
  for (int lt = (blockIdx.x >> 3) / c.k_splits; lt < per_xcd; lt += (gridDim.x >> 3) / c.k_splits) {
    const int tile = (blockIdx.x & 7) * per_xcd + lt;
    if (tile >= n_tiles) break;
    const int s = find_segment(a.tile_start, n_seg, tile);
    const int ad = a.seg_adapter[s];
    const int r = a.rank[ad] < a.max_rank ? a.rank[ad] : a.max_rank;
    const int pos0 = a.seg_start[s] + (tile - a.tile_start[s]) * 32;
    const int pos_end = a.seg_start[s + 1];
    const int kbeg = ks * c.k_per_split;
    const int kend = kbeg + c.k_per_split < a.d_in ? kbeg + c.k_per_split : a.d_in;
    const int n_chunks = r > 0 ? (kend - kbeg) / 64 : 0;

    uint64_t gaddr[NPER];
    uint32_t ldst[NPER];
#pragma unroll
    for (int i = 0; i < NPER; ++i) {
      int j = wave + 4 * i;
      if (j >= NINS) j -= 4;                           // no such instruction: this wave's previous one again
      const int rl = lane >> 3;
      const uint16_t* rowp;
      int rowi;
      if (j < 4) {
        rowi = 8 * j + rl;
        int pos = pos0 + rowi;
        pos = pos < pos_end ? pos : pos_end - 1;       // padding rows repeat the last token
        rowp = reinterpret_cast<const uint16_t*>(a.x) + (int64_t)a.perm[pos] * a.ld_x;
        ldst[i] = 1024u * j;
      } else {
        const int pj = (j - 4) >> 1;                   // projection whose A rows this instruction moves
        rowi = 8 * ((j - 4) & 1) + rl;                 // rank row
        rowp = pool;
        if (r > 0) {
          const flp_lora_proj& pr = a.proj[pj];
          const int ii = pr.a_row_base[ad] + (rowi < r ? rowi : 0);
          rowp = pool + (int64_t)a.tables[pr.a_tab_off[ad] + ii / rpb] * a.block_elems + (int64_t)(ii % rpb) * a.d_in;
        }
        ldst[i] = 4096u + 1024u * (j - 4);
      }
      gaddr[i] = (uint64_t)(uintptr_t)(rowp + kbeg + 8 * ((lane & 7) ^ (rowi & 7)));
    }
    auto issue_chunk = [&](int t) {
      const int tc = t < n_chunks ? t : n_chunks - 1;
      const uint32_t dst = lds0 + (uint32_t)(t & (kS - 1)) * kStageB;
#pragma unroll
      for (int i = 0; i < NPER; ++i) lload_lds16(gaddr[i] + (uint64_t)tc * 128, dst + ldst[i]);
    };

    f32x4 acc[NP];
    int offx[NP], offa[NP];
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
      int pi = wave + 4 * i;
      pi = pi < 2 * NPJ ? pi : 0;                      // no such pair: pair 0 again, not stored
      const int mt = pi / NPJ, pj = pi % NPJ;
      const int xr = 16 * mt + row16, ar = 16 * pj + row16;
      offx[i] = xr * 128 + ((kg ^ (xr & 7)) << 4);
      offa[i] = 4096 + ar * 128 + ((kg ^ (ar & 7)) << 4);
    }

    __builtin_amdgcn_s_waitcnt(lvmcnt(0));
    __syncthreads();
    if (n_chunks > 0) {
#pragma unroll
      for (int t = 0; t < kS - 1; ++t) issue_chunk(t);
    }
    for (int kt = 0; kt < n_chunks; ++kt) {
      __builtin_amdgcn_s_waitcnt(lvmcnt(2 * NPER));
      __syncthreads();
      issue_chunk(kt + kS - 1);
      const uint8_t* buf = smem + (kt & (kS - 1)) * kStageB;
#pragma unroll
      for (int k2 = 0; k2 < 2; ++k2)
#pragma unroll
        for (int i = 0; i < NP; ++i) {
          const vec xf = *reinterpret_cast<const vec*>(buf + (offx[i] ^ (k2 << 6)));
          const vec af = *reinterpret_cast<const vec*>(buf + (offa[i] ^ (k2 << 6)));
          acc[i] = L::mfma(xf, af, acc[i]);
        }
    }
    __builtin_amdgcn_s_waitcnt(lvmcnt(0));

    float* __restrict__ vout = a.v + ((int64_t)ks * c.v_rows + (int64_t)tile * 32) * a.n_proj * 16;
#pragma unroll
    for (int i = 0; i < NP; ++i) {
      const int pi = wave + 4 * i;
      if (pi < 2 * NPJ) {
        const int mt = pi / NPJ, pj = pi % NPJ;
#pragma unroll
        for (int e = 0; e < 4; ++e) vout[((int64_t)(16 * mt + 4 * kg + e) * a.n_proj + pj) * 16 + row16] = acc[i][e];
      }
    }
  }
}

// ------------------------------------------------------------------------------- expand
// y is updated in place, so this is the y stream with two thin products beside it, and what counts is how y is
// accessed.  A workgroup of four waves owns one (tile group, 256-column slab, projection); each wave takes every fourth
// 16-token sub-tile.
//
// The product is y = v B with the tokens as rows.  Column n of the eight column tiles of a 128-column half is column 8 n + tau,
// so a lane holds eight neighbouring columns of a token, sixteen lanes 256 contiguous bytes of its row, and one access
// covers whole lines of four rows.  Only such accesses gain from the non-temporal hint, loads and stores both.  (Transposed, with
// 32 bytes of one row per lane in two accesses, every access touches half of each line; hint or not, that is slower.)
// y is requested half a slab ahead, v a sub-tile ahead; v is summed over its slices, split and scaled once per 256 columns.
//
// Where an adapter has few tokens (up to sixteen: decode batches) three of the four waves would have nothing to do, and finding a
// group's adapter and pages takes longer than its work.  With ranks up to 16 such a group's workgroup takes four slabs, one per wave,
// and those of the other three slabs leave; the slab that a workgroup begins with moves on from group to group and from turn to
// turn, so that those with work are spread over the CUs.  (A workgroup per slab, and a wave per slab as before this kernel, q,k,v /
// o call of 1500 single tokens, up to 2000 adapters of rank 16, 32 heads: 754 / 299, 586 / 278 us; now 505 / 231.  Higher ranks are
// ahead without it, 0.6 to 0.8 of the former kernel, and their fragments would leave LDS for one workgroup less.)
//
// B of the slab lies in LDS as operand fragments, sixteen ranks times eight columns per thread: eight 16-byte loads along
// the page rows, turned in registers (ranks 2 j, 2 j + 1 of a column make a word).  v takes k-slots 0 .. 15 with its high part and
// 16 .. 31 with the remainder against the same coefficients, so lanes 32 apart read the same fragment.
//
// Measured, whole calls (segmentation, shrink, expand), against fragments gathered in registers (ranks up to 16) and
// transposed through LDS two bytes at a time (above), both with the transposed product; us:
//   21629 tokens, 32 heads, fp16, rank 16        q,k,v 370 -> 270      o 159 -> 122     (expand alone 4.05 -> 5.35 TB/s)
//   40961 tokens, 40 heads, fp16, rank 32        q,k,v 837 -> 709      gate,up 1288 -> 1078      down 530 -> 458
//   49712 tokens, 64 / 8 heads, bf16, rank 64    q,k,v 1411 -> 1246    o 966 -> 815
//   1801 tokens of up to 100 adapters, 64 / 8 heads, rank 64   q,k,v 612 -> 251   o 412 -> 145
template <typename L, int NT>
__global__ __launch_bounds__(256, 2) void lora_expand_stream_kernel(FlpLoraArgs a, FlpLoraMfma c) {
  typedef typename L::vec vec;
  typedef typename L::elem elem;
  typedef typename L::S S;
  // groups of up to sixteen tokens: a slab per wave (not with more rank tiles: they would leave too little LDS for a second workgroup)
  constexpr int kAlone = NT == 1 ? 4 : 1;
  __shared__ u32x4 frag[kAlone][2][NT][8][32];
  const int per_group = c.slabs * a.n_proj;
  const int n_seg = *a.n_seg;
  const int n_groups = a.group_start[n_seg];
  const int q_total = (n_groups + 7) / 8 * per_group;
  const int xcd = blockIdx.x & 7;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int n = lane & 15, kg = lane >> 4, kq = kg & 1, lo_half = kg >> 1;
  const uint16_t* __restrict__ pool = reinterpret_cast<const uint16_t*>(a.pool);
  for (int q = blockIdx.x >> 3, turn = 0; q < q_total; q += gridDim.x >> 3, ++turn) {
    const int group = (q / per_group) * 8 + xcd, p = (q % per_group) % a.n_proj;
    const int gi = q / per_group, slab = ((q % per_group) / a.n_proj + gi + gi / 4 + turn) % c.slabs;
    if (group >= n_groups) continue;
    const flp_lora_proj& pr = a.proj[p];
    if (slab * 256 >= pr.d_out) continue;
    const int s = find_segment(a.group_start, n_seg, group);
    const int ad = a.seg_adapter[s];
    const int r = a.rank[ad] < a.max_rank ? a.rank[ad] : a.max_rank;
    if (r <= 0) continue;
    const float sc = a.scale[ad];
    const int RP = 16 * NT, TM = 16 * c.mt;
    const int off0 = (group - a.group_start[s]) * c.group_tokens;
    const int pos0 = a.seg_start[s] + off0;
    const int pos_end = a.seg_start[s + 1];
    const int pos_stop = pos0 + c.group_tokens < pos_end ? pos0 + c.group_tokens : pos_end;
    const int64_t vrow0 = (int64_t)a.tile_start[s] * TM + off0;
    const int rpb = (int)(a.block_elems / pr.d_out);
    const bool alone = kAlone > 1 && pos_stop - pos0 <= 16;
    if (alone && slab % 4) continue;                   // with the slab before it
    const int slab_begin = 256 * (slab + (alone ? wave : 0));
    const int n_half = pr.d_out - slab_begin > 128 ? 2 : 1;
    u32x4(&mine)[2][NT][8][32] = frag[alone ? wave : 0];

    __syncthreads();                                   // the previous item's fragments are no longer read
    if (alone || tid < 64 * NT) {
      const int bn = tid & 15, h = (tid >> 4) & 1, bq = (tid >> 5) & 1, nt = alone ? 0 : tid >> 6;
      const int col = slab_begin + 128 * h + 8 * bn;
      u32x4 g[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int rho = 16 * nt + 8 * bq + j;
        const int i = pr.b_row_base[ad] + (rho < r ? rho : 0);
        g[j] = *reinterpret_cast<const u32x4*>(pool + (int64_t)a.tables[pr.b_tab_off[ad] + i / rpb] * a.block_elems +
                                               (int64_t)(i % rpb) * pr.d_out + (col < pr.d_out ? col : 0));
      }
#pragma unroll
      for (int j = 0; j < 8; ++j)
        if (!(16 * nt + 8 * bq + j < r && col < pr.d_out)) g[j] = u32x4{0u, 0u, 0u, 0u};
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        u32x4 e;
#pragma unroll
        for (int j = 0; j < 4; ++j)                    // ranks 2 j, 2 j + 1 of column t: its half of the two words
          e[j] = __builtin_amdgcn_perm(g[2 * j + 1][t / 2], g[2 * j][t / 2], t & 1 ? 0x07060302u : 0x05040100u);
        mine[h][nt][t][16 * bq + bn] = e;
      }
    }
    __syncthreads();
    if (slab_begin >= pr.d_out) continue;

    const bool from_y = !a.base32[p];
    uint16_t* const ybase = reinterpret_cast<uint16_t*>(pr.y) + slab_begin + 8 * n;
    const int h1 = slab_begin + 128 + 8 * n < pr.d_out ? 128 : 0;       // columns past the last one: the first ones again, not stored
    const int h0 = slab_begin + 8 * n < pr.d_out ? 0 : -8 * n;
    auto rows = [&](int32_t (&tok)[4], int pos_t) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int pos = pos_t + 4 * kg + i;
        tok[i] = a.perm[pos < pos_stop ? pos : pos_stop - 1];
      }
    };
    auto load_y = [&](u32x4 (&y)[4], const int32_t (&tok)[4], int off) {
      if (from_y)
#pragma unroll
        for (int i = 0; i < 4; ++i) y[i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(ybase + (int64_t)tok[i] * pr.ld_y + off));
    };
    auto v_row = [&](int pos_t, int ks) {
      const int pos = pos_t + n < pos_stop ? pos_t + n : pos_stop - 1;
      return a.v + (((int64_t)ks * c.v_rows + vrow0 + (pos - pos0)) * a.n_proj + p) * RP + 8 * kq;
    };
    auto load_v = [&](f32x4 (&v)[NT][2], int pos_t) {
      const float* vp = v_row(pos_t, 0);
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) {
        v[nt][0] = *reinterpret_cast<const f32x4*>(vp + 16 * nt);
        v[nt][1] = *reinterpret_cast<const f32x4*>(vp + 16 * nt + 4);
      }
    };
    int pos_t = pos0 + (alone ? 0 : 16 * wave);
    if (pos_t >= pos_stop) continue;
    int32_t tok[4];
    u32x4 y[2][4];
    f32x4 v[NT][2];
    vec vb[NT];
    rows(tok, pos_t);
    load_y(y[0], tok, h0);
    load_v(v, pos_t);
    auto update = [&](int h, const u32x4 (&yh)[4]) __attribute__((always_inline)) {
      f32x4 acc[8];
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
          if (16 * nt < r) acc[t] = L::mfma(vb[nt], vec_from<vec>(mine[h][nt][t][16 * kq + n]), acc[t]);
        if (t == 3) __builtin_amdgcn_sched_barrier(0);
      }
      const int col = slab_begin + 128 * h + 8 * n;
      if (col >= pr.d_out) return;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (pos_t + 4 * kg + i >= pos_stop) continue;
        uint16_t ys[8];
        if (from_y) {
          __builtin_memcpy(ys, &yh[i], 16);
#pragma unroll
          for (int t = 0; t < 8; ++t) ys[t] = S::from_float(S::to_float(ys[t]) + acc[t][i]);
        } else {                                       // unrounded base from the dense projection
          const float* brow = a.base32[p] + (int64_t)tok[i] * pr.d_out + col;
#pragma unroll
          for (int t = 0; t < 8; ++t) ys[t] = S::from_float(brow[t] + acc[t][i]);
        }
        u32x4 raw;
        __builtin_memcpy(&raw, ys, 16);
        __builtin_nontemporal_store(raw, reinterpret_cast<u32x4*>(ybase + (int64_t)tok[i] * pr.ld_y + 128 * h));
      }
    };
    for (; pos_t < pos_stop; pos_t += 64) {
      if (n_half > 1) load_y(y[1], tok, h1);
      // ---- A operand: this token's scaled v, high part in k-slots 0..15, remainder in 16..31
#pragma unroll
      for (int nt = 0; nt < NT; ++nt) {
        for (int ks = 1; ks < c.k_splits; ++ks) {
          const float* vp = v_row(pos_t, ks) + 16 * nt;
          v[nt][0] += *reinterpret_cast<const f32x4*>(vp);
          v[nt][1] += *reinterpret_cast<const f32x4*>(vp + 4);
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          elem hi, lo;
          L::split((16 * nt < r ? v[nt][j >> 2][j & 3] : 0.f) * sc, &hi, &lo);
          vb[nt][j] = lo_half ? lo : hi;
        }
      }
      int32_t tok_n[4];
      rows(tok_n, pos_t + 64);
      load_v(v, pos_t + 64);
      __builtin_amdgcn_sched_barrier(0);
      update(0, y[0]);
      __builtin_amdgcn_sched_barrier(0);
      load_y(y[0], tok_n, h0);
      __builtin_amdgcn_sched_barrier(0);
      if (n_half > 1) update(1, y[1]);
#pragma unroll
      for (int i = 0; i < 4; ++i) tok[i] = tok_n[i];
    }
  }
}

template <typename L, int MT, int NT>
flp_status launch_pair(const FlpLoraArgs& a, const FlpLoraMfma& c, hipStream_t stream) {
  constexpr bool ONEP = NT >= 2;                       // one projection per workgroup from rank 17 on
  const int n_pl = ONEP ? 1 : a.n_proj;
  const size_t smem = (size_t)4 * MT * n_pl * NT * 4 * 64 * sizeof(float);
  static std::atomic<bool> attr_set{false};   // pools on different threads share it
  if (!attr_set.load(std::memory_order_acquire)) {
    FLP_TRY_HIP(hipFuncSetAttribute((const void*)lora_shrink_mfma_kernel<L, MT, NT, ONEP>,
                                    hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024));
    attr_set.store(true, std::memory_order_release);
  }
  bool staged = false;
  if constexpr (NT >= 2 && MT == 2) {
    if (a.d_in % 64 == 0) {
      // two rank tiles: the projections of a call with two or three of them are fused (13B shapes, q,k,v call:
      // 0.89 -> 0.86 ms); with four rank tiles the fused stages leave one workgroup per CU and the call takes
      // twice as long (34B shapes: 1.25 -> 2.35 ms; the same with a ring of four stages in 128 KiB of dynamic LDS: 1.35 ->
      // 2.38 ms), so there a workgroup keeps to one projection
      constexpr int NPJ2 = NT == 2 ? 2 : 1, NPJ3 = NT == 2 ? 3 : 1;
      const dim3 gf((unsigned)(c.tiles_grid * c.k_splits));
      if (NT == 2 && a.n_proj == 2)
        hipLaunchKernelGGL((lora_shrink_lds_kernel<L, NT, NPJ2>), gf, dim3(256), 0, stream, a, c);
      else if (NT == 2 && a.n_proj == 3)
        hipLaunchKernelGGL((lora_shrink_lds_kernel<L, NT, NPJ3>), gf, dim3(256), 0, stream, a, c);
      else
        hipLaunchKernelGGL((lora_shrink_lds_kernel<L, NT, 1>), dim3((unsigned)(c.tiles_grid * c.k_splits * a.n_proj)),
                           dim3(256), 0, stream, a, c);
      staged = true;
    }
  }
  if constexpr (NT == 1 && MT == 2) {
    if (a.d_in % 64 == 0) {
      const dim3 g16((unsigned)(c.tiles_grid * c.k_splits));
      switch (a.n_proj) {
        case 1: hipLaunchKernelGGL((lora_shrink_lds16_kernel<L, 1>), g16, dim3(256), 0, stream, a, c); break;
        case 2: hipLaunchKernelGGL((lora_shrink_lds16_kernel<L, 2>), g16, dim3(256), 0, stream, a, c); break;
        case 3: hipLaunchKernelGGL((lora_shrink_lds16_kernel<L, 3>), g16, dim3(256), 0, stream, a, c); break;
        default: hipLaunchKernelGGL((lora_shrink_lds16_kernel<L, 4>), g16, dim3(256), 0, stream, a, c); break;
      }
      staged = true;
    }
  }
  if (!staged)
    hipLaunchKernelGGL((lora_shrink_mfma_kernel<L, MT, NT, ONEP>),
                       dim3((unsigned)(c.tiles_grid * c.k_splits * (ONEP ? a.n_proj : 1))), dim3(256), smem, stream, a, c);
  FLP_TRY_HIP(hipGetLastError());
  if (c.shrink_only) return FLP_OK;                     // the expand step is the dense product's epilogue
  int max_dout = 0;
  for (int p = 0; p < a.n_proj; ++p) max_dout = a.proj[p].d_out > max_dout ? a.proj[p].d_out : max_dout;
  FlpLoraMfma ce = c;
  ce.slabs = (max_dout + 255) / 256;
  const int64_t n_wg = (int64_t)c.groups_grid * ce.slabs * a.n_proj;
  if (n_wg > INT32_MAX) {
    flp_set_error("LoRA (matrix-core path): %lld workgroups, too many for one launch", (long long)n_wg);
    return FLP_ENOTSUP;
  }
  hipLaunchKernelGGL((lora_expand_stream_kernel<L, NT>), dim3((unsigned)n_wg), dim3(256), 0, stream, a, ce);
  FLP_TRY_HIP(hipGetLastError());
  return FLP_OK;
}

template <typename L>
flp_status launch_dtype(const FlpLoraArgs& a, const FlpLoraMfma& c, hipStream_t stream) {
  const int nt = (a.max_rank + 15) / 16;
  if (c.mt == 2) {
    if (nt <= 1) return launch_pair<L, 2, 1>(a, c, stream);
    if (nt == 2) return launch_pair<L, 2, 2>(a, c, stream);
    return launch_pair<L, 2, 4>(a, c, stream);
  }
  if (nt <= 1) return launch_pair<L, 1, 1>(a, c, stream);
  if (nt == 2) return launch_pair<L, 1, 2>(a, c, stream);
  return launch_pair<L, 1, 4>(a, c, stream);
}

}  // namespace

flp_status flp_launch_lora_mfma(int dtype, const FlpLoraArgs& a, const FlpLoraMfma& c, hipStream_t stream) {
  if (dtype == FLP_F16) return launch_dtype<LF16>(a, c, stream);
  if (dtype == FLP_BF16) return launch_dtype<LBF16>(a, c, stream);
  flp_set_error("LoRA (matrix-core path): dtype %d not supported", dtype);
  return FLP_ENOTSUP;
}
