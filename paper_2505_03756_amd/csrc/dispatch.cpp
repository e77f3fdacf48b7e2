// Host-side dispatch of the compute entry points: argument checks, the work lists built
// from the host-resident sequence lengths, and the launches.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <numeric>

#include "flp_internal.h"

namespace {

bool aligned16(const void* p) { return ((uintptr_t)p & 15) == 0; }

flp_status check_attn_batch(const flp_pool* p, const flp_attn_batch* b, bool need_qo, bool need_kv, const char* who) {
  if (!p || !b) {
    flp_set_error("%s: null pool or batch", who);
    return FLP_EINVAL;
  }
  if (b->n_seqs < 0 || b->max_blocks_per_seq < 0 || (b->n_seqs > 0 && (!b->cu_new || !b->prefix_len || !b->block_tables))) {
    flp_set_error("%s: bad sequence arrays", who);
    return FLP_EINVAL;
  }
  if ((p->cfg.block_tokens != 16 && p->cfg.block_tokens != 32) || (p->cfg.head_dim != 64 && p->cfg.head_dim != 128)) {
    flp_set_error("%s: kernels support block_tokens 16 or 32 and head_dim 64/128 (pool has %d / %d)", who,
                  p->cfg.block_tokens, p->cfg.head_dim);
    return FLP_ENOTSUP;
  }
  if (need_qo) {
    if (b->n_q_heads <= 0 || b->n_q_heads % p->cfg.n_kv_heads) {
      flp_set_error("%s: n_q_heads %d is not a multiple of n_kv_heads %d", who, b->n_q_heads, p->cfg.n_kv_heads);
      return FLP_EINVAL;
    }
  }
  if (b->n_seqs > 0 && b->cu_new[0] != 0) {
    flp_set_error("%s: cu_new[0] must be 0", who);
    return FLP_EINVAL;
  }
  const int64_t cap = (int64_t)b->max_blocks_per_seq * p->cfg.block_tokens;
  for (int32_t i = 0; i < b->n_seqs; ++i) {
    int64_t n = (int64_t)b->cu_new[i + 1] - b->cu_new[i];
    if (n < 0 || b->prefix_len[i] < 0) {
      flp_set_error("%s: sequence %d has negative length", who, i);
      return FLP_EINVAL;
    }
    if (b->prefix_len[i] + n > cap) {
      flp_set_error("%s: sequence %d needs %lld positions, its block table covers %lld", who, i,
                    (long long)(b->prefix_len[i] + n), (long long)cap);
      return FLP_ERANGE;
    }
  }
  const int32_t T = b->n_seqs > 0 ? b->cu_new[b->n_seqs] : 0;
  if (T > 0) {
    if (need_qo && (!b->q || !b->out || !aligned16(b->q) || !aligned16(b->out))) {
      flp_set_error("%s: q/out must be non-null and 16-byte aligned", who);
      return FLP_EINVAL;
    }
    if (need_kv && (!b->k_new || !b->v_new || !aligned16(b->k_new) || !aligned16(b->v_new))) {
      flp_set_error("%s: k_new/v_new must be non-null and 16-byte aligned", who);
      return FLP_EINVAL;
    }
  }
  return FLP_OK;
}

FlpAttnArgs make_args(const flp_pool* p, const flp_attn_batch* b) {
  FlpAttnArgs a{};
  a.pool = p->dev_base;
  a.block_elems = p->block_elems;
  a.tables = b->block_tables;
  a.max_blocks = b->max_blocks_per_seq;
  a.n_h = b->n_q_heads;
  a.n_kv = p->cfg.n_kv_heads;
  a.bt = p->cfg.block_tokens;
  a.q = b->q;
  a.out = b->out;
  a.k_new = b->k_new;
  a.v_new = b->v_new;
  float sc = b->sm_scale > 0.f ? b->sm_scale : 1.0f / std::sqrt((float)p->cfg.head_dim);
  a.scale_log2e = sc * 1.4426950408889634f;
  return a;
}

// the append step of a batch, a unit per 16-position group that gets new slots
std::vector<FlpAppendUnit> append_units(const flp_attn_batch* b) {
  const int bt = 16;                                 // the kernel's unit is a group of 16 positions, whatever the block size
  std::vector<FlpAppendUnit> units;
  for (int32_t i = 0; i < b->n_seqs; ++i) {
    const int32_t P = b->prefix_len[i], n = b->cu_new[i + 1] - b->cu_new[i];
    int32_t pos = P;
    while (pos < P + n) {
      FlpAppendUnit u{};
      u.seq = i;
      u.blk_idx = pos / bt;
      u.s0 = pos % bt;
      u.s1 = std::min<int32_t>(bt, u.s0 + (P + n - pos));
      u.t_first = b->cu_new[i] + (pos - P);
      units.push_back(u);
      pos += u.s1 - u.s0;
    }
  }
  return units;
}

// Whether the append launch reads its units where they were staged, in pinned host memory, or from a copy that a launch of its
// own makes first.  Up to as many workgroups as the chip holds at once (two per CU) all reads are under way together, and
// sparing the copy is worth 3 us (400 workgroups: 16 -> 13 us).  More of them read in turns, and now and then such a launch has
// taken a microsecond or so for every workgroup instead: 20 sequences of 2000 tokens, 5040 workgroups, 254 us or 4.1 ms, the mean of
// sixty calls 252 to 990 us; 257 us each with the copy.
bool append_reads_host(const flp_pool* p, size_t n_units) {
  return n_units * (size_t)flp_kv_append_columns(p->cfg.dtype, p->cfg.n_kv_heads, p->cfg.head_dim) <= 512;
}

}  // namespace

extern "C" flp_status flp_kv_append(flp_pool* p, const flp_attn_batch* b, void* hip_stream) {
  FLP_TRY(check_attn_batch(p, b, false, true, "flp_kv_append"));
  std::lock_guard<std::mutex> lk(p->mu);
  const std::vector<FlpAppendUnit> units = append_units(b);
  if (units.empty()) return FLP_OK;
  FlpStageSlot* slot = nullptr;
  const size_t bytes = units.size() * sizeof(FlpAppendUnit);
  FLP_TRY(flp_stage_acquire(p, bytes, &slot));
  memcpy(slot->host, units.data(), bytes);
  const bool direct = append_reads_host(p, units.size());
  flp_status s1 = direct ? FLP_OK : flp_stage_upload(slot, bytes, (hipStream_t)hip_stream);
  if (s1 == FLP_OK)
    s1 = flp_launch_kv_append(p->cfg.dtype, p->cfg.head_dim, make_args(p, b),
                              (const FlpAppendUnit*)(direct ? slot->host : slot->dev), (int32_t)units.size(), nullptr, nullptr, 0,
                              (hipStream_t)hip_stream);
  flp_status s2 = flp_stage_release(slot, (hipStream_t)hip_stream);
  return s1 != FLP_OK ? s1 : s2;
}

namespace {
constexpr int kTokPerUnit = 4;
enum { FLP_ATTN_APART = 0, FLP_ATTN_BEHIND, FLP_ATTN_BETWEEN };      // single tokens: a launch of their own; behind the tiles; between them

// Which kernel takes which sequence of an attention call, and in how many launches
struct AttnRoute {
  bool mfma_ok, decode_ok;     // head size and type of the matrix-core kernels; as many query heads per kv head as the decode kernel takes
  int G, bt;
  bool small_launch;
  int32_t rows;                // query rows per item of the tiled kernel
  int mix;                     // FLP_ATTN_*
  bool tiled(int64_t prefix, int64_t n) const {
    return mfma_ok && G * n >= 8 && (prefix + n + bt - 1) / bt <= kMfmaMaxBlocks && !(small_launch && n <= kTokPerUnit);
  }
};
AttnRoute attn_route(bool mfma_ok, int n_q, int n_kv, int bt, int32_t n_seqs, const int32_t* cu, const int32_t* prefix) {
  AttnRoute r{};
  r.mfma_ok = mfma_ok;
  r.G = n_q / n_kv;
  r.bt = bt;
  r.decode_ok = mfma_ok && r.G <= kDecodeMaxGroup;
  // A launch of fewer than 128 matrix-core items (a few decode sequences under grouped-query attention) goes to the
  // decode kernel (more than 16 heads per kv head: the row kernel) instead, where long contexts are split over many waves.
  //
  // Query rows per item: 256, a wave for 32 of them.  A step of a workgroup takes 1.6 us with four waves at work and 2.1 with eight,
  // so a launch whose items fit one workgroup per CU with half the rows takes those (fp16 / bf16, us, 256 rows and 128):
  //   700 + 499 positions, 32 heads         44.3   33.7     (128 items of 128 rows)
  //   2 sequences of 500 + 200, 32 heads    31.4   25.3     (128)
  //   2000 + 300 positions, 64 / 8 heads    70.0   52.0     (152)
  //   6 sequences of 300 + 120, 32 heads    23.4   23.6     (192: nothing is cut)
  //   3 of 2000 + 200, 64 / 8 heads         71.0   90.1     (312)
  //   1000 + 900 positions, 40 heads        60.4   74.6     (320)
  int64_t whole = 0, half = 0;
  const auto items_of = [&](int64_t n, int rows) { return (int64_t)n_kv * ((r.G * n + rows - 1) / rows); };
  if (mfma_ok)
    for (int32_t i = 0; i < n_seqs; ++i) {
      const int64_t n = cu[i + 1] - cu[i];
      if (r.G * n < 8) continue;
      whole += items_of(n, kMfmaRowsPerItem);
      half += items_of(n, kMfmaRowsPerItem / 2);
    }
  r.small_launch = whole < 128;
  r.rows = half <= 256 ? kMfmaRowsPerItem / 2 : kMfmaRowsPerItem;
  // Tiles are bound by the matrix cores and single tokens by memory, so where it pays a batch of both runs as one launch:
  // workgroups of the tiled kernel take eight single (token, kv head) pieces each.  Behind the tiles they take the CUs that the
  // tiles' last round leaves idle, and where that is less than a quarter of the chip there is nothing to take.  (Between the tiles of
  // one or two rounds they push some of those into another: 256 tiles of 2 x 900 tokens over 1000 positions and 100 single tokens of
  // short contexts, 32 heads, 104 us in two launches, 164 in one.)  From three rounds on they are spread over the first half of the
  // tiles, so that memory is busy beside the matrix cores.  A tile of a short context ends before a piece of a long one: then
  // only the gap between the launches is saved, and the larger workgroups cost more than that unless the single tokens are few and
  // short as well.  Two launches, behind, between (us; f16, prompts and single tokens, items):
  //   500 + 1000 positions, 100 of up to 64, 32 heads     (128)       71     55     70
  //   3 x 700 + 1000, 50 of up to 2048, 40 heads          (360)      343    308    322
  //   16 x 300 + 0, 50 of up to 2048, 32 heads           (1024)      301    301    296
  //   16 x 300 + 1000, 100 of up to 2048, 40 heads       (1280)      678    679    670
  //   2 x 500 + 0, 4 of up to 2048, 32 heads              (256)       50     56     46
  //   4 x 900 + 1000, 200 of up to 64, 32 heads           (512)      193    195    276
  //   20 + 0, 4 of up to 2048 / 64, 32 heads               (32)   39, 25 43, 23 44, 23
  // Single tokens of grouped-query batches of 128 items and more are tiles themselves: 512 sequences of up to 16 k, 64 / 8 heads,
  // 12.6 ms with tiles and 12.35 with pieces, but 100 of up to 4 k 720 and 762 us.
  int64_t items = 0, row_tokens = 0, longest_tile = 0, longest_row = 0;
  for (int32_t i = 0; i < n_seqs; ++i) {
    const int64_t n = cu[i + 1] - cu[i], len = prefix[i] + n;
    if (n <= 0) continue;
    if (r.tiled(prefix[i], n)) {
      items += items_of(n, r.rows);
      longest_tile = std::max(longest_tile, len);
    } else {
      row_tokens += n;
      longest_row = std::max(longest_row, len);
    }
  }
  const int64_t idle = (256 - items % 256) % 256;
  const bool worth = longest_tile >= 256 || (longest_row <= 256 && row_tokens * n_kv <= 4096);
  r.mix = !r.decode_ok || !items || !row_tokens || !worth ? FLP_ATTN_APART
          : items >= 768                                  ? FLP_ATTN_BETWEEN
          : idle >= 64                                    ? FLP_ATTN_BEHIND
                                                          : FLP_ATTN_APART;
  return r;
}
}  // namespace

extern "C" int32_t flp_attention_route(int32_t n_q_heads, int32_t n_kv_heads, int32_t block_tokens, int32_t n_seqs, const int32_t* cu,
                                       const int32_t* prefix) {
  return attn_route(true, n_q_heads, n_kv_heads, block_tokens, n_seqs, cu, prefix).mix;
}

extern "C" flp_status flp_paged_prefix_attention(flp_pool* p, const flp_attn_batch* b, void* hip_stream) {
  const bool with_append = b && (b->k_new || b->v_new);
  FLP_TRY(check_attn_batch(p, b, true, with_append, "flp_paged_prefix_attention"));
  std::lock_guard<std::mutex> lk(p->mu);
  hipStream_t stream = (hipStream_t)hip_stream;

  // Three kinds of work.  On a 16-bit pool with head_dim 128, sequences with at least 8 query rows per kv head (prefill,
  // or decode under grouped-query attention) go to the tiled matrix-core kernel in tiles of 256 rows (128 in small launches), and the others
  // (and all short ones of a small launch, below) token by token to the decode kernel.  fp32, head_dim 64 and more than 16
  // query heads per kv head: the row-streaming kernel in runs of up to 4 tokens.  All lists are ordered heaviest first.
  //
  // Single tokens of a grouped-query batch, tiles against decode kernel (64 / 8 heads, bf16, us per call):
  //                     6 seqs   15    16    24    32    64   128   300     contexts
  //   tiles               232   262   261   263   280   423   796  1846     1 - 16 k
  //   decode kernel        65   136   153   207   264   461   863  1969
  //   tiles               268   269   270   279   379   726  1415  3366     16 k each
  //   decode kernel       109   227   242   342   431   795  1491  3441
  // With many sequences a tile's one pass over K and V for all heads of a group is ahead, also where the batch has nothing
  // but single tokens (and with 128 prefill sequences beside 384 decoding ones: 17.5 ms for the step against 17.8); with
  // few the tiles leave the chip idle.  The line, 128 items (16 sequences here), is right for equal contexts; where they
  // differ, the longest one decides what unsplit tiles take and the decode kernel would stay ahead up to 32 sequences.
  const AttnRoute route = attn_route(p->cfg.dtype != FLP_F32 && p->cfg.head_dim == 128, b->n_q_heads, p->cfg.n_kv_heads,
                                     p->cfg.block_tokens, b->n_seqs, b->cu_new, b->prefix_len);
  const int G = route.G;
  const int n_kv = p->cfg.n_kv_heads;
  const bool decode_ok = route.decode_ok;
  std::vector<int32_t> seq_order(b->n_seqs);
  std::iota(seq_order.begin(), seq_order.end(), 0);
  auto seq_cost = [&](int32_t i) {
    int64_t n = b->cu_new[i + 1] - b->cu_new[i];
    return n * (2 * (int64_t)b->prefix_len[i] + n);
  };
  std::stable_sort(seq_order.begin(), seq_order.end(), [&](int32_t x, int32_t y) { return seq_cost(x) > seq_cost(y); });

  std::vector<FlpAttnUnit> units;
  std::vector<int64_t> cost;
  // matrix-core items: the row tiles of one (sequence, kv head) are dealt to ONE of 8 queues and
  // the queues are interleaved, so that under round-robin dispatch of workgroups over the 8
  // XCDs the tiles that re-read the same K/V run on the same XCD and share its L2.
  std::vector<FlpMfmaItem> queue[8];
  int next_q = 0;
  std::vector<int32_t> row_seqs;                      // sequences of the decode or the row kernel, heaviest first
  int64_t row_tokens = 0;
  for (int32_t i : seq_order) {
    const int32_t n = b->cu_new[i + 1] - b->cu_new[i];
    if (n <= 0) continue;
    if (route.tiled(b->prefix_len[i], n)) {
      const int32_t R = G * n;
      for (int g = 0; g < n_kv; ++g) {
        for (int32_t r0 = 0; r0 < R; r0 += route.rows)
          queue[next_q].push_back(FlpMfmaItem{i, g, r0, std::min<int32_t>(route.rows, R - r0)});
        next_q = (next_q + 1) & 7;
      }
    } else {
      row_seqs.push_back(i);
      row_tokens += n;
    }
  }
  // Split-KV.  A wave of the decode kernel takes one (token, kv head), one of the row kernel one (token, head); with
  // few tokens and long contexts (a handful of decode sequences at 16 k) that is far fewer waves than the chip holds,
  // and with unequal contexts the longest one decides.  Contexts are cut into pieces, each piece a wave; a second kernel
  // merges the pieces of a row in piece order.  Decode kernel: a row's pieces are of equal length, at most `piece` groups of
  // 16 positions each (so more than half of that), which makes about kPieces of them (twice what the chip holds) or,
  // for small launches, pieces of 8 to 16 groups.  Row kernel: below kSplitBelow waves, pieces of kMinGroups and more.
  constexpr int64_t kSplitBelow = 2048, kSplitTarget = 8192, kPieces = 4096;
  constexpr int kMinGroups = 16, kMaxSplit = 64;
  const int64_t row_waves = row_tokens * b->n_q_heads;
  const int want_split = row_waves > 0 && row_waves < kSplitBelow
                             ? (int)std::min<int64_t>(kMaxSplit, (kSplitTarget + row_waves - 1) / row_waves) : 1;
  int64_t all_groups = 0;
  if (decode_ok)
    for (int32_t i : row_seqs) {
      const int64_t n = b->cu_new[i + 1] - b->cu_new[i];
      all_groups += n * (((int64_t)b->prefix_len[i] + n + 15) / 16);
    }
  // beside tiles pieces are half as long, so that none of them is the launch's tail
  const bool mixed = route.mix != FLP_ATTN_APART;
  const int64_t piece = std::max<int64_t>(kMinGroups, all_groups * n_kv / (mixed ? 2 * kPieces : kPieces));
  std::vector<int32_t> merge_tok, merge_first{0};
  for (int32_t i : row_seqs) {
    const int32_t n = b->cu_new[i + 1] - b->cu_new[i];
    if (decode_ok || want_split > 1) {
      for (int32_t j = 0; j < n; ++j) {
        const int32_t groups = (b->prefix_len[i] + j + 1 + 15) / 16;
        const int ns = decode_ok ? (int)std::min<int64_t>(kMaxSplit, (groups + piece - 1) / piece)
                                 : std::max(1, std::min(want_split, groups / kMinGroups));
        if (ns == 1) {
          units.push_back(FlpAttnUnit{i, b->cu_new[i] + j, 1, b->prefix_len[i] + j + 1, 0, groups, -1, 0});
          cost.push_back(groups);
          continue;
        }
        const int32_t row = merge_first.back();
        merge_tok.push_back(b->cu_new[i] + j);
        merge_first.push_back(row + ns);
        for (int sidx = 0; sidx < ns; ++sidx) {
          const int32_t lo = (int32_t)((int64_t)groups * sidx / ns), hi = (int32_t)((int64_t)groups * (sidx + 1) / ns);
          units.push_back(FlpAttnUnit{i, b->cu_new[i] + j, 1, b->prefix_len[i] + j + 1, lo, hi, row + sidx, 0});
          cost.push_back(hi - lo);
        }
      }
    } else {
      for (int32_t j0 = 0; j0 < n; j0 += kTokPerUnit) {
        FlpAttnUnit u{i, b->cu_new[i] + j0, std::min(kTokPerUnit, n - j0), b->prefix_len[i] + j0 + 1, 0, 0, -1, 0};
        units.push_back(u);
        cost.push_back((int64_t)u.n_tok * (b->prefix_len[i] + j0 + u.n_tok));
      }
    }
  }
  std::vector<int32_t> order(units.size());
  std::iota(order.begin(), order.end(), 0);
  std::stable_sort(order.begin(), order.end(), [&](int32_t x, int32_t y) { return cost[x] > cost[y]; });
  size_t qmax = 0;
  for (auto& q : queue) qmax = std::max(qmax, q.size());
  // single tokens beside tiles: rows of eight workgroups, eight (unit, kv head) pairs each
  const size_t pairs = mixed ? units.size() * n_kv : 0, pair_rows = (pairs + 63) / 64;
  const size_t n_items = (qmax + pair_rows) * 8;
  if (units.empty() && n_items == 0) return FLP_OK;

  void* partials = nullptr;
  const size_t n_merge = merge_tok.size();
  if (n_merge)
    FLP_TRY(flp_attn_workspace(p, (size_t)merge_first.back() * b->n_q_heads * (p->cfg.head_dim + 2) * sizeof(float), stream,
                               &partials));
  // one staging slot: the append step's units, then what is copied to the device by the append launch (or, with the units, before
  // it): the lists of the attention launches and, for the tiled kernel, the sequences' lengths
  const std::vector<FlpAppendUnit> append = with_append ? append_units(b) : std::vector<FlpAppendUnit>{};
  const size_t S = (size_t)b->n_seqs;
  const auto up = [](size_t n) { return (n + 31) & ~(size_t)31; };
  const size_t off_units = up(append.size() * sizeof(FlpAppendUnit)), off_items = off_units + units.size() * sizeof(FlpAttnUnit);
  const size_t off_merge = off_items + n_items * sizeof(FlpMfmaItem), off_cu = off_merge + (2 * n_merge + 1) * sizeof(int32_t);
  const size_t off_pl = off_cu + (S + 1) * sizeof(int32_t), bytes = n_items ? off_pl + S * sizeof(int32_t) : off_cu;
  FlpStageSlot* slot = nullptr;
  FLP_TRY(flp_stage_acquire(p, up(bytes), &slot));
  uint8_t* const h = (uint8_t*)slot->host;
  const uint8_t* const d = (const uint8_t*)slot->dev;
  if (!append.empty()) memcpy(h, append.data(), append.size() * sizeof(FlpAppendUnit));
  FlpAttnUnit* hu = (FlpAttnUnit*)(h + off_units);
  for (size_t k = 0; k < order.size(); ++k) hu[k] = units[order[k]];
  FlpMfmaItem* hi = (FlpMfmaItem*)(h + off_items);
  size_t at = 0, done = 0;
  for (size_t s = 0; s < qmax; ++s) {
    for (; route.mix == FLP_ATTN_BETWEEN && done < pair_rows && done * qmax <= 2 * pair_rows * s; ++done)
      for (int x = 0; x < 8; ++x) hi[at++] = FlpMfmaItem{(int32_t)pairs, 0, (int32_t)(64 * done + 8 * x), -1};
    for (int x = 0; x < 8; ++x) hi[at++] = s < queue[x].size() ? queue[x][s] : FlpMfmaItem{0, 0, 0, 0};
  }
  for (; done < pair_rows; ++done)
    for (int x = 0; x < 8; ++x) hi[at++] = FlpMfmaItem{(int32_t)pairs, 0, (int32_t)(64 * done + 8 * x), -1};
  if (n_merge) memcpy(h + off_merge, merge_tok.data(), n_merge * sizeof(int32_t));
  memcpy(h + off_merge + n_merge * sizeof(int32_t), merge_first.data(), (n_merge + 1) * sizeof(int32_t));
  if (n_items) {
    memcpy(h + off_cu, b->cu_new, (S + 1) * sizeof(int32_t));
    memcpy(h + off_pl, b->prefix_len, S * sizeof(int32_t));
  }
  FlpAttnArgs a = make_args(p, b);
  a.partials = (float*)partials;
  a.cu_new = (const int32_t*)(d + off_cu);
  a.prefix_len = (const int32_t*)(d + off_pl);
  const FlpAttnUnit* du = (const FlpAttnUnit*)(d + off_units);
  const FlpMfmaItem* di = (const FlpMfmaItem*)(d + off_items);
  const int32_t* dm = (const int32_t*)(d + off_merge);
  flp_status st = FLP_OK;
  if (append_reads_host(p, append.size())) {
    st = flp_launch_kv_append(p->cfg.dtype, p->cfg.head_dim, a, (const FlpAppendUnit*)h, (int32_t)append.size(), h + off_units,
                              (uint8_t*)slot->dev + off_units, bytes - off_units, stream);
  } else {
    st = flp_stage_upload(slot, bytes, stream);
    if (st == FLP_OK)
      st = flp_launch_kv_append(p->cfg.dtype, p->cfg.head_dim, a, (const FlpAppendUnit*)d, (int32_t)append.size(), nullptr, nullptr,
                                0, stream);
  }
  if (st == FLP_OK) st = flp_launch_attn_mfma(p->cfg.dtype, a, di, (int32_t)n_items, du, stream);
  if (st == FLP_OK && !mixed)
    st = decode_ok ? flp_launch_attn_decode(p->cfg.dtype, a, du, (int32_t)units.size(), stream)
                   : flp_launch_attn_rows(p->cfg.dtype, p->cfg.head_dim, a, du, (int32_t)units.size(), stream);
  if (st == FLP_OK)
    st = flp_launch_attn_merge(p->cfg.dtype, p->cfg.head_dim, a, dm, dm + n_merge, (int32_t)n_merge, stream);
  const flp_status released = flp_stage_release(slot, stream);
  if (n_merge && released == FLP_OK) {
    p->attn_slot = slot;
    p->attn_stream = stream;
  }
  return st != FLP_OK ? st : released;
}

// ------------------------------------------------------------------------------- LoRA
extern "C" flp_status flp_lora_segment(flp_pool* p, int32_t n_tokens, const int32_t* token_adapter,
                                       int32_t n_adapters, int32_t* n_seg, int32_t* seg_adapter, int32_t* seg_start,
                                       int32_t* perm, void* hip_stream) {
  if (!p || n_tokens < 0 || n_adapters < 0 || !n_seg || !seg_adapter || !seg_start || (n_tokens > 0 && (!token_adapter || !perm))) {
    flp_set_error("flp_lora_segment: invalid argument");
    return FLP_EINVAL;
  }
  if (n_adapters > 2048) {
    flp_set_error("flp_lora_segment: %d adapters, at most 2048 supported", n_adapters);
    return FLP_ERANGE;
  }
  return flp_launch_lora_segment(n_tokens, token_adapter, n_adapters, n_seg, seg_adapter, seg_start, perm, 0, nullptr, 0,
                                 nullptr, (hipStream_t)hip_stream);
}

namespace {
flp_status lora_apply_impl(flp_pool* p, const flp_lora_batch* b, void* hip_stream, size_t budget, void* gated_out,
                           int64_t ld_gated, const FlpFixedWorkspace* fixed = nullptr, const FlpSequences* seqs = nullptr);
}

// The call and its form in a fixed buffer plan the dense products for the same room, the fixed buffer's, so that they take
// the same slices and return the same bits.
extern "C" flp_status flp_lora_apply_paged(flp_pool* p, const flp_lora_batch* b, void* hip_stream) {
  return lora_apply_impl(p, b, hip_stream, kStaticScratchBytes, nullptr, 0);
}

flp_status flp_lora_apply_fixed(flp_pool* p, const flp_lora_batch* b, void* hip_stream, const FlpFixedWorkspace& ws) {
  return lora_apply_impl(p, b, hip_stream, ws.cap, nullptr, 0, &ws);
}

flp_status flp_lora_apply_layer(flp_pool* p, const flp_lora_batch* b, const FlpSequences& seqs, void* hip_stream) {
  return lora_apply_impl(p, b, hip_stream, kLayerSliceBytes, nullptr, 0, nullptr, &seqs);
}

flp_status flp_lora_apply_gated(flp_pool* p, const flp_lora_batch* b, const FlpSequences& seqs, void* out, int64_t ld_out,
                                void* hip_stream) {
  if (!out || ((uintptr_t)out & 15)) {
    flp_set_error("flp_lora_apply_gated: out is null or misaligned");
    return FLP_EINVAL;
  }
  return lora_apply_impl(p, b, hip_stream, kLayerSliceBytes, out, ld_out, nullptr, &seqs);
}

namespace {
// dense base products that run as one launch: projections which[0 .. n) of the call
struct BaseGroup {
  int n = 0;
  int which[FLP_MAX_PROJ] = {0, 0, 0, 0};
  FlpGemmPlan plan{};
};

// groups and plans of a call's dense base products; returns the bytes their slices take, every product's rounded up to
// 256.  More than one slice is taken only where all slices stay within `room`; one slice of every product is planned
// even where that does not fit.
size_t plan_base(const flp_lora_batch* b, bool one_launch, size_t room, std::vector<BaseGroup>* groups) {
  for (int q = 0; q < b->n_proj; ++q) {
    if (!b->proj[q].w_base) continue;
    if (groups->empty() || !one_launch) groups->push_back(BaseGroup{});
    BaseGroup& g = groups->back();
    g.which[g.n++] = q;
  }
  const size_t pad = 255 * (size_t)b->n_proj;
  const size_t share = groups->empty() || room < pad ? 0 : (room - pad) / groups->size();
  for (unsigned allow = 0;; allow = FLP_GEMM_NO_SPLIT) {
    size_t total = 0;
    for (BaseGroup& g : *groups) {
      int N[FLP_MAX_PROJ];
      for (int i = 0; i < g.n; ++i) N[i] = b->proj[g.which[i]].d_out;
      g.plan = flp_gemm_plan(b->n_tokens, b->d_in, g.n, N, allow, share);
      for (int i = 0; i < g.n; ++i) total += ((size_t)g.plan.splits * b->n_tokens * N[i] * 4 + 255) & ~(size_t)255;
    }
    if (total <= room || allow) return total;          // a product larger than its share: the others may not slice either
  }
}

// most sequences that any `window` tokens of the call touch, counted from the call's first token on
int32_t most_sequences(const FlpSequences& s, int32_t n_tokens, int32_t window, int32_t* n_in_call) {
  int32_t most = 0, here = 0, at = -1, n = 0;           // sequences in window `at`
  for (int32_t i = 0; i < s.n; ++i) {
    const int64_t lo = std::max<int64_t>(0, (int64_t)s.cu[i] - s.first);
    const int64_t hi = std::min<int64_t>(n_tokens, (int64_t)s.cu[i + 1] - s.first);
    if (hi <= lo) continue;
    ++n;
    const int32_t first = (int32_t)(lo / window), last = (int32_t)((hi - 1) / window);
    here = first == at ? here + 1 : 1;
    most = std::max(most, here);
    if (last > first) here = 1;
    at = last;
  }
  *n_in_call = n;
  return most;
}

struct LoraRoute {
  bool sorted;       // tokens sorted by adapter, steps on tiles of them
  bool in_product;   // sorted, and the expand step is the dense products' epilogue
  bool long_runs;    // not sorted: a wave of the expand step goes through neighbouring tokens
};
LoraRoute lora_route(int dtype, const flp_lora_batch* b, const FlpSequences* seqs) {
  LoraRoute r{};
  // Matrix-core path with tokens sorted by adapter for 16-bit pools when every width is a multiple of the tile widths (32
  // in, 64 out) and the batch is large enough for token tiles to fill (prefill); smaller batches on the matrix cores as
  // well, but without the sort; fp32 pools and odd widths on the vector-ALU kernels.
  r.sorted = dtype != FLP_F32 && b->d_in % 32 == 0 && b->n_tokens >= 1024;
  for (int q = 0; q < b->n_proj; ++q) r.sorted = r.sorted && b->proj[q].d_out % 64 == 0;
  // Sequences of 16 tokens and more on average, and how many of them meet in a tile, or in a wave's neighbouring tokens: with the
  // mean alone 110 single tokens behind four prompts counted as 17 tokens each.
  int32_t in_tile = INT32_MAX, in_block = INT32_MAX, n = 0;
  if (seqs && seqs->cu && b->n_tokens > 64) {
    in_tile = most_sequences(*seqs, b->n_tokens, 128, &n);
    in_block = most_sequences(*seqs, b->n_tokens, kLoraLongBlock, &n);
    if (n == 0 || b->n_tokens < 16 * (int64_t)n) in_tile = in_block = INT32_MAX;
  }
  // Dense base on every projection, and products that together have enough of the large tiles: the expand step runs as
  // their epilogue (segment, shrink, then one launch for the projections, or one each where W is stored [d_in, d_out],
  // that adds the LoRA branch to its accumulators before it rounds): no fp32 copy of the product, no second pass over y.
  // The epilogue walks the adapters present among its tile's tokens, eight at a time: one or two when tokens come in sequences and as
  // many as tokens in a large pure-decode batch.  Batches of 2048 tokens and more, and from 1024 tokens on those with at most twenty
  // sequences in any 128 tokens.  (Smaller ones keep the small batches' expand step, which holds v in 32 bits: here, as in the
  // expand step of the sorted tokens, it enters as value and remainder of the 16-bit type, scaled, so that it has to stay within
  // fp16's range and has fewer bits where it is small.)  Layers, us, separate steps / epilogue:
  //                            7B, rank 16     7B, rank 64 on all seven     34B, rank 64
  //   1200                     688 /  638           1013 /  837            1860 / 1758
  //   1200 of 60 sequences     722 /  665           1205 / 1021            1938 / 1826
  //   1800 and 16 single ones 1002 /  914           1455 / 1436            2563 / 2541
  //   1800 and 32             1034 /  975           1513 / 1864            2621 / 2669
  //   1200 and 64              763 /  833           1279 / 1947            2037 / 2309
  r.in_product = r.sorted && (b->n_tokens >= 2048 || in_tile <= 20) && b->d_in % 64 == 0 &&
                 flp_gemm_offsets_fit(FLP_GEMM_256x256, b->n_tokens, b->ld_x);
  int64_t tiles = 0;                           // enough 256 x 128 tiles to occupy the chip without slices
  for (int q = 0; q < b->n_proj; ++q) {
    r.in_product = r.in_product && b->proj[q].w_base;
    tiles += (int64_t)((b->proj[q].d_out + 255) / 256) * ((b->n_tokens + 127) / 128);
  }
  r.in_product = r.in_product && tiles >= 96;
  // Most tokens are not the first of a group, and those that are do not follow each other.  Layers, us, a token per wave / eight
  // neighbouring ones:
  //   499-token prompt, 7B shapes, rank 16   413 / 382     500 tokens, 7B, rank 32 on all seven   539 / 489      34B   876 / 883
  //   500 and 8 single tokens                408 / 401                                            567 / 543      34B   897 / 948
  //   500 and 30                             445 / 447                                            604 / 609      34B  1061 / 1115
  // With four rank tiles no difference (1000 tokens of two sequences, rank 64: 674 and 676).
  r.long_runs = !r.sorted && dtype != FLP_F32 && b->n_tokens <= kLoraSmallTokens && b->max_rank <= 32 && in_block <= 2;
  return r;
}

// gated_out != nullptr: two projections (gate, up) whose results are not stored; gated_out = silu(y0) * y1
// fixed != nullptr: the intermediates go into the caller-provided buffer and nothing is allocated; a batch that
// needs more than the buffer holds is refused before anything is enqueued
// budget: bytes of intermediates that slices of dense products may bring the call to, whatever the buffer is (the sums'
// order, and with it the result's last bits, depends on the number of slices)
// seqs: the sequences the tokens come in, null: not known
flp_status lora_apply_impl(flp_pool* p, const flp_lora_batch* b, void* hip_stream, size_t budget, void* gated_out,
                           int64_t ld_gated, const FlpFixedWorkspace* fixed, const FlpSequences* seqs) {
  if (!p || !b) {
    flp_set_error("flp_lora_apply_paged: null pool or batch");
    return FLP_EINVAL;
  }
  if (b->n_tokens < 0 || b->n_proj < 1 || b->n_proj > FLP_MAX_PROJ || b->n_adapters < 0 || b->d_in <= 0 ||
      b->ld_x < b->d_in) {
    flp_set_error("flp_lora_apply_paged: bad sizes (n_tokens=%d n_proj=%d n_adapters=%d d_in=%d ld_x=%lld)",
                  b->n_tokens, b->n_proj, b->n_adapters, b->d_in, (long long)b->ld_x);
    return FLP_EINVAL;
  }
  if (b->n_tokens == 0) return FLP_OK;
  if (b->max_rank < 1 || b->max_rank > 64) {
    flp_set_error("flp_lora_apply_paged: max_rank %d outside 1..64", b->max_rank);
    return FLP_ERANGE;
  }
  if (b->n_adapters > 2048) {
    flp_set_error("flp_lora_apply_paged: %d adapters, at most 2048 supported", b->n_adapters);
    return FLP_ERANGE;
  }
  const int epl = 16 / p->elem_bytes;
  if (!b->x || !b->token_adapter || !b->rank || !b->scale || !b->block_tables || !aligned16(b->x) ||
      b->d_in % epl || b->ld_x % epl || b->d_in > p->block_elems) {
    flp_set_error("flp_lora_apply_paged: x/metadata null or misaligned, or d_in %d not a multiple of %d / larger than a block",
                  b->d_in, epl);
    return FLP_EINVAL;
  }
  for (int q = 0; q < b->n_proj; ++q) {
    const flp_lora_proj& pr = b->proj[q];
    if (pr.w_base_layout != 0 && pr.w_base_layout != 1) {
      flp_set_error("flp_lora_apply_paged: projection %d: w_base_layout %d is neither 0 nor 1", q, pr.w_base_layout);
      return FLP_EINVAL;
    }
    if (pr.d_out <= 0 || pr.ld_y < pr.d_out || pr.d_out % epl || pr.ld_y % epl || pr.d_out > p->block_elems || !pr.y ||
        !aligned16(pr.y) || !pr.a_tab_off || !pr.a_row_base || !pr.b_tab_off || !pr.b_row_base) {
      flp_set_error("flp_lora_apply_paged: projection %d has bad sizes or null/misaligned pointers", q);
      return FLP_EINVAL;
    }
    if (pr.w_base && (!aligned16(pr.w_base) || (p->elem_bytes == 2 && b->d_in % 64))) {
      flp_set_error("flp_lora_apply_paged: projection %d: w_base misaligned, or d_in %d not a multiple of 64", q,
                    b->d_in);
      return pr.w_base && aligned16(pr.w_base) ? FLP_ENOTSUP : FLP_EINVAL;
    }
  }
  std::lock_guard<std::mutex> lk(p->mu);
  hipStream_t stream = (hipStream_t)hip_stream;
  const size_t T = (size_t)b->n_tokens;

  const LoraRoute route = lora_route(p->cfg.dtype, b, seqs);
  const bool mfma_ok = route.sorted, fused = route.in_product;
  FlpLoraMfma c{};
  size_t v_elems = T * b->n_proj * b->max_rank;
  if (mfma_ok) {
    c.mt = b->n_tokens >= 2048 ? 2 : 1;
    const int tm = 16 * c.mt;
    // The number of segments is only known on the device.  The bounds (every adapter present, each adding a
    // partly filled tile) size the buffers; the launches cover the tiles of up to 64 present adapters in one
    // pass and loop for the rest, so that a pool of thousands of adapters does not launch thousands of
    // workgroups that find nothing to do.
    const int32_t seg_bound = (int32_t)std::min<size_t>((size_t)b->n_adapters, T);
    c.tiles_bound = (int32_t)((T + tm - 1) / tm) + seg_bound;
    c.tiles_grid = (std::min(c.tiles_bound, (int32_t)((T + tm - 1) / tm) + 64) + 7) / 8 * 8;
    // split K until enough workgroups are in flight, in pieces of 128 coefficients: about 2048 for the kernel
    // that reads its operands from global memory (it lives on loads in flight), about 1024 for the LDS-staged
    // ones (they keep three chunks in flight themselves; fewer partial sums for the expand kernel to add)
    const int wg_target = (c.mt == 2 && b->d_in % 64 == 0) ? 1024 : 2048;
    int ks = 1;
    while (ks < 8 && c.tiles_grid * ks < wg_target && b->d_in / (ks * 2) >= 256) ks *= 2;
    c.k_splits = ks;
    c.k_per_split = ((b->d_in + ks - 1) / ks + 127) / 128 * 128;
    c.v_rows = c.tiles_bound * tm;
    const int nt = (b->max_rank + 15) / 16 <= 2 ? (b->max_rank + 15) / 16 : 4;
    // Tokens per workgroup of the expand step: its slab of B is laid out once for all of them, so long groups are cheap, but a
    // few hundred workgroups leave the chip idle.  Measured with 64, 128 and 256 tokens each (us for the call; workgroups at 256):
    //   1500 tokens, 40 heads, q,k,v of rank 32   (360)    76    93    84
    //   3000 tokens, 64 / 8 heads, rank 64        (480)   160   174   202
    //   5000 tokens, 40 heads, gate and up        (2160)  245   241   269
    //   20123 tokens, 32 heads, q,k,v of rank 16  (3792)  281   257   256
    //   49712 tokens, 64 / 8 heads, rank 64       (7800)    -  1322  1272
    int64_t wgs = 0;
    for (int q = 0; q < b->n_proj; ++q) wgs += (int64_t)((T + 255) / 256) * ((b->proj[q].d_out + 255) / 256);
    c.group_tokens = wgs < 1024 ? 64 : wgs < 4096 ? 128 : 256;
    c.groups_bound = (int32_t)((T + c.group_tokens - 1) / c.group_tokens) + seg_bound;
    c.groups_grid = (std::min(c.groups_bound, (int32_t)((T + c.group_tokens - 1) / c.group_tokens) + 64) + 7) / 8 * 8;
    const int rp = 16 * nt;
    v_elems = (size_t)ks * c.v_rows * b->n_proj * rp;
  }
  if (gated_out) {
    const bool ok = fused && b->n_proj == 2 && b->proj[0].d_out == b->proj[1].d_out && b->proj[0].d_out % 32 == 0 &&
                    b->proj[0].w_base_layout == 1 && b->proj[1].w_base_layout == 1 && ld_gated >= b->proj[0].d_out &&
                    ld_gated % epl == 0;
    if (!ok) return FLP_ENOTSUP;                // nothing launched: the caller takes the separate products
  }
  size_t wt_bytes = 0;                         // transposed copy of the widest dense base matrix
  bool one_launch = true;                      // matrices stored [d_out, d_in] go in one launch, others one by one
  if (p->elem_bytes == 2)
    for (int q = 0; q < b->n_proj; ++q)
      if (b->proj[q].w_base && b->proj[q].w_base_layout == 0) {
        wt_bytes = std::max(wt_bytes, (size_t)b->d_in * b->proj[q].d_out * 2);
        one_launch = false;
      }
  wt_bytes = (wt_bytes + 255) & ~(size_t)255;
  size_t v_bytes = (v_elems * 4 + 255) & ~(size_t)255;
  const size_t seg_bytes = ((size_t)(4 * b->n_adapters + 5) * 4 + 255) & ~(size_t)255;
  const size_t perm_bytes = (T * 4 + 255) & ~(size_t)255;
  // token -> position in segment order, adapter -> first row of its tokens in the shrink output
  const size_t inv_bytes = fused ? perm_bytes + (((size_t)b->n_adapters * 4 + 255) & ~(size_t)255) : 0;
  // Batches of up to 1024 tokens: slices of d_in until some thousand waves are in flight.  Two slices, four (us): 300 tokens, o of
  // ranks 8-64, 64 heads 74.0, 63.3; 300 tokens, q,k,v of rank 16, 32 heads 49.1, 50.8; 499 tokens of one adapter of rank 16, o, 40
  // heads 30.4, 28.4, q,k,v, 32 heads 38.1, 40.3.  The intermediates are larger than the vector kernels' (slices of v, ranks in
  // sixteens, a record per token): a batch that only fits the call's buffer without them takes those kernels, so that what a
  // fixed buffer accepts does not depend on it.
  FlpLoraSmall small{};
  size_t group_bytes = 0;
  if (!mfma_ok && p->elem_bytes == 2 && b->n_tokens <= kLoraSmallTokens && b->d_in % 64 == 0) {
    small.n_tiles = b->max_rank <= 16 ? 1 : b->max_rank <= 32 ? 2 : 4;
    small.k_splits = b->n_tokens <= 16 ? 16 : b->n_tokens <= 64 ? 8
                     : b->n_tokens <= 256 || b->n_tokens * b->n_proj <= 768 ? 4 : 2;
    while (small.k_splits > 1 && b->d_in / 64 / small.k_splits < 4) small.k_splits /= 2;
    small.long_runs = route.long_runs;
    const size_t v_small = ((size_t)small.k_splits * T * b->n_proj * 16 * small.n_tiles * 4 + 255) & ~(size_t)255;
    const size_t g_small = (T * sizeof(FlpLoraGroup) + 255) & ~(size_t)255;
    size_t total = v_small + g_small + seg_bytes + perm_bytes + wt_bytes;
    for (int q = 0; q < b->n_proj; ++q)
      if (b->proj[q].w_base) total += (T * b->proj[q].d_out * 4 + 255) & ~(size_t)255;
    if (total <= budget) {
      v_bytes = v_small;
      group_bytes = g_small;
    }
  }
  // dense products that are not fused with the expand step leave their unrounded result in the workspace, in slices
  // of the contraction where the batch is small
  std::vector<BaseGroup> groups;
  size_t base_total = 0;
  if (p->elem_bytes == 2 && !fused) {
    const size_t rest = v_bytes + group_bytes + seg_bytes + perm_bytes + wt_bytes;
    base_total = plan_base(b, one_launch, budget > rest ? budget - rest : 0, &groups);
  }
  void* ws = nullptr;
  const size_t ws_bytes = v_bytes + seg_bytes + perm_bytes + wt_bytes + base_total + inv_bytes + group_bytes;
  if (fixed) {
    if (ws_bytes > fixed->cap) {
      flp_set_error("%s: the batch needs %zu bytes of intermediates, the fixed buffer holds %zu (fewer tokens, a lower "
                    "max_rank or no dense base make it fit)", fixed->who, ws_bytes, fixed->cap);
      return FLP_ENOSPC;
    }
    FLP_TRY(fixed->resolve(p, &ws));
  } else {
    FLP_TRY(flp_workspace(p, ws_bytes, &ws));
  }
  FlpLoraArgs a{};
  a.pool = p->dev_base;
  a.block_elems = p->block_elems;
  a.T = b->n_tokens;
  a.d_in = b->d_in;
  a.n_adapters = b->n_adapters;
  a.max_rank = b->max_rank;
  a.n_proj = b->n_proj;
  a.ld_x = b->ld_x;
  a.x = b->x;
  a.token_adapter = b->token_adapter;
  a.rank = b->rank;
  a.scale = b->scale;
  a.tables = b->block_tables;
  for (int q = 0; q < b->n_proj; ++q) a.proj[q] = b->proj[q];
  uint8_t* w = (uint8_t*)ws;
  a.v = (float*)w;
  a.n_seg = (int32_t*)(w + v_bytes);
  a.seg_adapter = a.n_seg + 1;
  a.seg_start = a.seg_adapter + b->n_adapters;
  a.tile_start = a.seg_start + b->n_adapters + 1;
  a.group_start = a.tile_start + b->n_adapters + 1;
  a.perm = (int32_t*)(w + v_bytes + seg_bytes);
  if (fused) {
    int32_t* inv_perm = (int32_t*)(w + v_bytes + seg_bytes + perm_bytes + wt_bytes);
    uint8_t* wt = w + v_bytes + seg_bytes + perm_bytes;
    int32_t* vrow_base = (int32_t*)((uint8_t*)inv_perm + perm_bytes);
    FLP_TRY(flp_launch_lora_segment(a.T, a.token_adapter, a.n_adapters, a.n_seg, a.seg_adapter, a.seg_start, a.perm,
                                    16 * c.mt, a.tile_start, c.group_tokens, a.group_start, stream, inv_perm, vrow_base));
    c.shrink_only = 1;
    FLP_TRY(flp_launch_lora_mfma(p->cfg.dtype, a, c, stream));
    const int nt = (b->max_rank + 15) / 16 <= 2 ? (b->max_rank + 15) / 16 : 4;
    auto branch = [&](int q) {
      FlpGemmLora lp{};
      lp.token_adapter = a.token_adapter;
      lp.rank = a.rank;
      lp.scale = a.scale;
      lp.tables = a.tables;
      lp.b_tab_off = b->proj[q].b_tab_off;
      lp.b_row_base = b->proj[q].b_row_base;
      lp.pool = a.pool;
      lp.block_elems = a.block_elems;
      lp.v = a.v;
      lp.v_rows = c.v_rows;
      lp.k_splits = c.k_splits;
      lp.n_proj = b->n_proj;
      lp.p = q;
      lp.rp = 16 * nt;
      lp.n_adapters = b->n_adapters;
      lp.max_rank = b->max_rank < 16 * nt ? b->max_rank : 16 * nt;
      lp.inv_perm = inv_perm;
      lp.vrow_base = vrow_base;
      return lp;
    };
    FlpGemmLora lp[FLP_MAX_PROJ];
    FlpGemmOut out[FLP_MAX_PROJ] = {};
    int N[FLP_MAX_PROJ];
    for (int q = 0; q < b->n_proj; ++q) {
      lp[q] = branch(q);
      N[q] = out[q].N = b->proj[q].d_out;
      out[q].w = b->proj[q].w_base;
      out[q].y = b->proj[q].y;
      out[q].ld_y = b->proj[q].ld_y;
    }
    const unsigned allow = FLP_GEMM_NO_SPLIT | FLP_GEMM_LARGE_ONLY;
    if (gated_out) {
      out[0].w2 = out[1].w;
      N[0] = out[0].N = 2 * b->proj[0].d_out;
      out[0].y = gated_out;
      out[0].ld_y = ld_gated;
      const FlpGemmPlan plan = flp_gemm_plan(b->n_tokens, b->d_in, 1, N, allow, 0);
      return flp_launch_gemm(p->cfg.dtype, b->x, b->ld_x, b->n_tokens, b->d_in, plan, 1, out, true, lp, stream);
    }
    const int step = one_launch ? b->n_proj : 1;
    for (int q = 0; q < b->n_proj; q += step) {
      if (b->proj[q].w_base_layout == 0) {
        FLP_TRY(flp_launch_transpose16(out[q].w, wt, b->d_in, N[q], stream));
        out[q].w = wt;
      }
      const FlpGemmPlan plan = flp_gemm_plan(b->n_tokens, b->d_in, step, N + q, allow, 0);
      FLP_TRY(flp_launch_gemm(p->cfg.dtype, b->x, b->ld_x, b->n_tokens, b->d_in, plan, step, out + q, false, lp + q, stream));
    }
    return FLP_OK;
  }
  // base term first where the caller asked for it (x . W_base), then the adapters' deltas on top.
  // 16-bit pools also keep the product unrounded in the workspace so that base + delta is rounded once.  Where y is written
  // already, by an unsliced product or by the kernel that adds slices, tokens without an adapter keep that rounded value; with
  // base_slices > 1 nothing has written y yet, and the small batches' expand step writes every token's, those without a
  // branch included.
  if (p->elem_bytes == 4) {
    for (int q = 0; q < b->n_proj; ++q)
      if (b->proj[q].w_base)
        FLP_TRY(flp_launch_gemm_f32((const float*)b->x, b->ld_x, (const float*)b->proj[q].w_base, b->proj[q].w_base_layout,
                                    (float*)b->proj[q].y, b->proj[q].ld_y, b->n_tokens, b->proj[q].d_out, b->d_in, stream));
  } else {
    uint8_t* wt = w + v_bytes + seg_bytes + perm_bytes;
    uint8_t* basep = wt + wt_bytes;
    for (const BaseGroup& g : groups) {
      FlpGemmOut out[FLP_MAX_PROJ] = {};
      for (int i = 0; i < g.n; ++i) {
        const flp_lora_proj& pr = b->proj[g.which[i]];
        out[i].w = pr.w_base;
        out[i].y = pr.y;
        out[i].ld_y = pr.ld_y;
        out[i].part = (float*)basep;
        out[i].N = pr.d_out;
        a.base32[g.which[i]] = (float*)basep;
        basep += ((size_t)g.plan.splits * T * pr.d_out * 4 + 255) & ~(size_t)255;
        if (pr.w_base_layout == 0) {
          FLP_TRY(flp_launch_transpose16(pr.w_base, wt, b->d_in, pr.d_out, stream));
          out[i].w = wt;
        }
      }
      FLP_TRY(flp_launch_gemm(p->cfg.dtype, b->x, b->ld_x, b->n_tokens, b->d_in, g.plan, g.n, out, false, nullptr, stream));
      // the small batches' expand step adds the slices itself
      if (g.plan.splits > 1 && !group_bytes)
        FLP_TRY(flp_launch_gemm_reduce(p->cfg.dtype, b->n_tokens, g.n, out, g.plan.splits, false, FLP_REDUCE_KEEP, stream));
      for (int i = 0; i < g.n; ++i) a.base_slices[g.which[i]] = group_bytes ? g.plan.splits : 1;
    }
  }
  if (group_bytes) {
    small.groups = (FlpLoraGroup*)(w + v_bytes + seg_bytes + perm_bytes + wt_bytes + base_total);
    return flp_launch_lora_small(p->cfg.dtype, a, small, stream);
  }
  if (!mfma_ok) return flp_launch_lora_simple(p->cfg.dtype, a, stream);
  FLP_TRY(flp_launch_lora_segment(a.T, a.token_adapter, a.n_adapters, a.n_seg, a.seg_adapter, a.seg_start, a.perm,
                                  16 * c.mt, a.tile_start, c.group_tokens, a.group_start, stream));
  return flp_launch_lora_mfma(p->cfg.dtype, a, c, stream);
}
}  // namespace

extern "C" int32_t flp_lora_layer_route(int32_t dtype, int32_t n_tokens, int32_t d_in, int32_t n_proj, const int32_t* d_out,
                                        int32_t max_rank, int32_t n_seqs, const int32_t* cu, int32_t first) {
  flp_lora_batch b{};
  b.n_tokens = n_tokens;
  b.d_in = d_in;
  b.ld_x = d_in;
  b.max_rank = max_rank;
  b.n_proj = n_proj;
  for (int q = 0; q < n_proj; ++q) {
    b.proj[q].d_out = d_out[q];
    b.proj[q].w_base = &b;                     // there is one
  }
  const FlpSequences seqs{cu, n_seqs, first};
  const LoraRoute r = lora_route(dtype, &b, &seqs);
  return r.in_product ? FLP_LORA_IN_PRODUCT : r.sorted ? FLP_LORA_SORTED : r.long_runs ? FLP_LORA_TOKENS_LONG : FLP_LORA_TOKENS;
}
