"""GPU parity: the HIP path through the C ABI against the CPU oracle, element by element."""
import numpy as np
import pytest
import torch

import oracle
from helpers import TOL, GpuStep, build_pools, close, dense_plan, resident_pool, to_dev, to_np
from paper_2505_03756_amd import flpool
from paper_2505_03756_amd import workload as wl

pytestmark = pytest.mark.gpu


def small_cfg(dtype, **kw):
    base = dict(name="small_" + dtype, dtype=dtype, hidden=512, n_q_heads=4, n_kv_heads=4, head_dim=128,
                n_dev_blocks=400, n_host_blocks=512, n_adapters=6, ranks=(8, 16, 32), projections=("q", "k", "v", "o"),
                n_seqs=7, prefix_range=(0, 300), new_range=(1, 70), swap_in_frac=0.4, seed=77)
    base.update(kw)
    return wl.LayerConfig(**base)


CASES = {
    "tiny": lambda: wl.config("tiny"),
    "f16_prefill": lambda: small_cfg("f16"),
    "bf16_decode": lambda: small_cfg("bf16", n_seqs=19, prefix_range=(1, 700), new_range=(1, 1), decode_frac=1.0,
                                     n_dev_blocks=1200, seed=78),
    "bf16_gqa_mixed": lambda: small_cfg("bf16", n_q_heads=8, n_kv_heads=2, hidden=1024, decode_frac=0.5,
                                        prefix_range=(0, 500), seed=79),
    "f16_d64": lambda: small_cfg("f16", head_dim=64, n_q_heads=8, n_kv_heads=8, seed=80),
    "bf16_d64_gqa": lambda: small_cfg("bf16", head_dim=64, n_q_heads=8, n_kv_heads=4, decode_frac=0.4, seed=93),
    "f32_d128": lambda: small_cfg("f32", n_seqs=4, prefix_range=(0, 120), new_range=(1, 40), seed=81),
    # blocks of 32 token positions (the block size of the paper's vLLM baseline, section 2.2) as a layout variant:
    # prefill on the matrix-core kernel, decode / mixed and fp32 on the row kernel, head_dim 64
    "f16_prefill_bt32": lambda: small_cfg("f16", block_tokens=32, seed=91),
    "bf16_gqa_mixed_bt32": lambda: small_cfg("bf16", block_tokens=32, n_q_heads=8, n_kv_heads=2, hidden=1024,
                                             decode_frac=0.5, prefix_range=(0, 500), seed=92),
    "bf16_decode_bt32": lambda: small_cfg("bf16", block_tokens=32, n_seqs=19, prefix_range=(1, 700), new_range=(1, 1),
                                          decode_frac=1.0, n_dev_blocks=1200, seed=93),
    "f32_d64_bt32": lambda: small_cfg("f32", block_tokens=32, head_dim=64, n_q_heads=8, n_kv_heads=8, n_seqs=4,
                                      prefix_range=(0, 120), new_range=(1, 40), seed=94),
}


@pytest.fixture(scope="module", params=list(CASES))
def case(request):
    cfg = CASES[request.param]()
    step = wl.make_step(cfg)
    print("\n[case %s] T=%d S=%d dtype=%s" % (request.param, step.n_tokens, cfg.n_seqs, cfg.dtype), flush=True)
    return step


def test_swap_in_out_bit_exact(case):
    step, cfg = case, case.cfg
    dev0, host0 = build_pools(step, poison_rest=True)
    g = GpuStep(step, dev0, host0)
    # oracle
    dev_ref, host_ref = dev0.copy(), host0.copy()
    oracle.swap(host_ref, dev_ref, step.swap_out_dev, step.swap_out_host)
    oracle.swap(dev_ref, host_ref, step.swap_in_host, step.swap_in_dev)
    # library: swap-out first, then swap-in (the order the paper gives when the device tier is full)
    g.pool.swap_out(step.swap_out_dev, step.swap_out_host)
    g.pool.swap_in(step.swap_in_host, step.swap_in_dev)
    assert np.array_equal(g.dev_image().view(np.uint8), dev_ref.view(np.uint8))
    assert np.array_equal(g.host_image().view(np.uint8), host_ref.view(np.uint8))
    # after the swap-in every needed block is resident with its content
    assert np.array_equal(g.dev_image()[step.content_ids].view(np.uint8), step.content.view(np.uint8))


def test_swap_round_trip_every_block():
    cfg = wl.config("tiny")
    rng = np.random.default_rng(5)
    dev0 = rng.standard_normal((cfg.n_dev_blocks, cfg.block_elems)).astype(np.float32)
    host0 = np.zeros((cfg.n_dev_blocks, cfg.block_elems), np.float32)
    step = wl.make_step(cfg, with_acts=False)
    g = GpuStep(step, dev0, host0)
    ids = np.arange(cfg.n_dev_blocks, dtype=np.int32)
    perm, back = rng.permutation(ids).astype(np.int32), rng.permutation(ids).astype(np.int32)
    g.pool.swap_out(ids, perm)
    assert np.array_equal(g.host_image()[perm], dev0)
    g.dev.zero_()
    g.pool.swap_in(perm, back)
    assert np.array_equal(g.dev_image()[back], dev0)


def test_kv_append_bit_exact(case):
    step, cfg = case, case.cfg
    dev0 = resident_pool(step)
    g = GpuStep(step, dev0, np.zeros((1, cfg.block_elems), dev0.dtype))
    ref = dev0.copy()
    oracle.kv_append(ref, cfg.dtype, cfg.block_tokens, cfg.n_kv_heads, cfg.head_dim, step.cu_new, step.prefix_len,
                     step.kv_tables, step.acts["k_new"], step.acts["v_new"])
    g.pool.kv_append(g.acts["k_new"], g.acts["v_new"], step.cu_new, step.prefix_len, g.kv_tables)
    assert np.array_equal(g.dev_image().view(np.uint8), ref.view(np.uint8))


@pytest.mark.parametrize("dtype,bt,kv,d", [("f16", 16, 2, 128), ("bf16", 32, 17, 128), ("f32", 16, 4, 64), ("f16", 32, 3, 64),
                                           ("f32", 32, 9, 128)])
def test_append_of_units_of_every_length(dtype, bt, kv, d):
    """1 .. 17 new tokens at every offset of a group of 16 positions: units of every length, short ones whose slots are
    written one by one and longer ones whose runs are merged, in rows of less and more than one workgroup's width.  Bit for
    bit, the slots around them included; once as the append call and once in front of the attention step."""
    rng = np.random.default_rng(3)
    st = np.float32 if dtype == "f32" else np.uint16
    seqs = [(p, n) for p in range(0, 18) for n in (1, 2, 3, 4, 5, 15, 16, 17)]
    nb = [(p + n + bt - 1) // bt for p, n in seqs]
    tables = np.full((len(seqs), max(nb)), -1, np.int32)
    ids = rng.permutation(sum(nb)).astype(np.int32)
    at = 0
    for i, k in enumerate(nb):
        tables[i, :k] = ids[at:at + k]
        at += k
    cu = np.concatenate([[0], np.cumsum([n for _, n in seqs])]).astype(np.int32)
    prefix = np.array([p for p, _ in seqs], np.int32)
    rand = lambda shape: rng.standard_normal(shape).astype(np.float32) if dtype == "f32" else \
        rng.integers(0, 0x3c00, shape).astype(np.uint16)                           # finite in either 16-bit type
    pool0, k, v, q = rand((at, 2 * bt * kv * d)), rand((int(cu[-1]), kv * d)), rand((int(cu[-1]), kv * d)), rand((int(cu[-1]), kv * d))
    want = pool0.copy()
    oracle.kv_append(want, dtype, bt, kv, d, cu, prefix, tables, k, v)
    up = lambda a: torch.from_numpy(a if dtype == "f32" else a.view(np.int16)).cuda()
    for attend in (False, True):
        dev = up(pool0.copy())
        pool = flpool.Pool(dtype, kv, d, at, 0, block_tokens=bt, dev=dev)
        if attend:
            pool.paged_prefix_attention(up(q), torch.empty_like(up(q)), cu, prefix, torch.from_numpy(tables).cuda(),
                                        kv, k_new=up(k), v_new=up(v))
        else:
            pool.kv_append(up(k), up(v), cu, prefix, torch.from_numpy(tables).cuda())
        torch.cuda.synchronize()
        assert np.array_equal(dev.cpu().numpy().view(st).view(np.uint8), want.view(np.uint8)), attend
        pool.close()


@pytest.mark.parametrize("dtype,kv,d,units", [("bf16", 1, 128, 512), ("bf16", 1, 128, 513), ("f16", 17, 128, 256), ("f16", 17, 128, 257),
                                              ("f32", 5, 64, 513)])
def test_append_of_as_many_units_as_are_read_from_the_host_and_of_more(dtype, kv, d, units):
    """512 workgroups read their units from pinned memory, more have them copied first (17 kv heads of 128: two workgroups per unit).
    Single tokens and one longer sequence; the append call bit for bit, and in front of the attention step with its result."""
    rng = np.random.default_rng(units)
    st = np.float32 if dtype == "f32" else np.uint16
    seqs = [(int(p), 1) for p in rng.integers(0, 40, units - 3)] + [(7, 40)]               # 9 + 16 + 15 slots
    nb = [(p + n + 15) // 16 for p, n in seqs]
    assert sum((p + n - 1) // 16 - p // 16 + 1 for p, n in seqs) == units
    tables = np.full((len(seqs), max(nb)), -1, np.int32)
    ids, at = rng.permutation(sum(nb)).astype(np.int32), 0
    for i, k in enumerate(nb):
        tables[i, :k] = ids[at:at + k]
        at += k
    cu = np.concatenate([[0], np.cumsum([n for _, n in seqs])]).astype(np.int32)
    prefix = np.array([p for p, _ in seqs], np.int32)
    T = int(cu[-1])
    rand = lambda shape: wl.quantize(rng.standard_normal(shape).astype(np.float32), dtype)
    pool0, k, v, q = rand((at, 2 * 16 * kv * d)), rand((T, kv * d)), rand((T, kv * d)), rand((T, kv * d))
    want = pool0.copy()
    oracle.kv_append(want, dtype, 16, kv, d, cu, prefix, tables, k, v)
    out = oracle.paged_attention(want, dtype, 16, kv, d, kv, cu, prefix, tables, q)
    up = lambda a: torch.from_numpy(a if dtype == "f32" else a.view(np.int16)).cuda()
    for attend in (False, True):
        dev = up(pool0.copy())
        pool = flpool.Pool(dtype, kv, d, at, 0, block_tokens=16, dev=dev)
        got = torch.empty_like(up(q))
        for _ in range(2):                               # another staging slot, the same result
            if attend:
                pool.paged_prefix_attention(up(q), got, cu, prefix, torch.from_numpy(tables).cuda(), kv, k_new=up(k), v_new=up(v))
            else:
                pool.kv_append(up(k), up(v), cu, prefix, torch.from_numpy(tables).cuda())
        torch.cuda.synchronize()
        assert np.array_equal(dev.cpu().numpy().view(st).view(np.uint8), want.view(np.uint8)), attend
        if attend:
            rtol, atol = TOL[dtype]
            ok, worst, nbad = close(wl.dequantize(got.cpu().numpy().view(st), dtype).reshape(out.shape), out, rtol, atol)
            assert ok, "max err %g (%d bad)" % (worst, nbad)
        pool.close()


def test_attention_matches_oracle(case):
    step, cfg = case, case.cfg
    dev0 = resident_pool(step)       # fresh blocks hold NaN patterns until the append fills their slots
    g = GpuStep(step, dev0, np.zeros((1, cfg.block_elems), dev0.dtype))
    got = wl.dequantize(g.attention(append=True), cfg.dtype).reshape(step.n_tokens, cfg.n_q_heads, cfg.head_dim)
    ref_pool = dev0.copy()
    oracle.kv_append(ref_pool, cfg.dtype, cfg.block_tokens, cfg.n_kv_heads, cfg.head_dim, step.cu_new,
                     step.prefix_len, step.kv_tables, step.acts["k_new"], step.acts["v_new"])
    want = oracle.paged_attention(ref_pool, cfg.dtype, cfg.block_tokens, cfg.n_kv_heads, cfg.head_dim, cfg.n_q_heads,
                                  step.cu_new, step.prefix_len, step.kv_tables, step.acts["q"])
    rtol, atol = TOL[cfg.dtype]
    ok, worst, nbad = close(got, want, rtol, atol)
    assert ok, "max err %g, %d elements out of tolerance" % (worst, nbad)
    # second entry form: K/V already appended, k_new = v_new = NULL
    got2 = wl.dequantize(g.attention(append=False), cfg.dtype).reshape(got.shape)
    assert np.array_equal(got, got2)


def test_lora_matches_oracle(case):
    step, cfg = case, case.cfg
    dev0 = resident_pool(step)
    g = GpuStep(step, dev0, np.zeros((1, cfg.block_elems), dev0.dtype))
    rtol, atol = TOL[cfg.dtype]
    groups = [[p for p in cfg.projections if p in ("q", "k", "v")], [p for p in cfg.projections if p == "o"]]
    for names in groups:
        if not names:
            continue
        x_key = "x" if names[0] != "o" or cfg.proj_dims("o")[0] == cfg.hidden else "x_%d" % cfg.proj_dims("o")[0]
        got = g.lora(names, x_key=x_key)
        for n in names:
            pr = step.proj[n]
            want = oracle.lora_apply(dev0, cfg.dtype, step.acts[x_key], step.token_adapter, step.rank, step.scale,
                                     pr.a_tab_off, pr.a_row_base, pr.b_tab_off, pr.b_row_base, step.lora_tables,
                                     pr.d_out, y_in=step.acts["base_" + n])
            ok, worst, nbad = close(wl.dequantize(got[n], cfg.dtype), want, rtol, atol)
            assert ok, "%s: max err %g, %d elements out of tolerance" % (n, worst, nbad)
            delta = np.abs(want - wl.dequantize(step.acts["base_" + n], cfg.dtype)).max()
            assert delta > 10 * atol or cfg.dtype == "f32"      # the test would notice a missing delta


LORA_CASES = {
    # T >= 2048 selects the 32-token tiles; rank 16 -> one rank tile; Zipf gives one long segment and a tail
    "f16_long_segments": lambda: small_cfg("f16", hidden=1024, n_q_heads=8, n_kv_heads=8, n_seqs=24,
                                           prefix_range=(0, 0), new_range=(40, 180), n_adapters=12, ranks=(16,),
                                           adapter_dist="zipf", n_dev_blocks=600, swap_in_frac=0.0, seed=82),
    # ranks 8..64 mixed -> four rank tiles with partially filled ones; many short segments, 16-token tiles
    "bf16_mixed_rank": lambda: small_cfg("bf16", hidden=1024, n_q_heads=8, n_kv_heads=8, n_seqs=200,
                                         prefix_range=(0, 0), new_range=(2, 11), n_adapters=60,
                                         ranks=(8, 16, 32, 64), n_dev_blocks=2500, swap_in_frac=0.0, seed=83),
    # the same shapes as a small decode batch (kernels for up to 1024 tokens)
    "bf16_mixed_rank_decode": lambda: small_cfg("bf16", hidden=1024, n_q_heads=8, n_kv_heads=8, n_seqs=200,
                                                prefix_range=(0, 0), new_range=(1, 1), decode_frac=1.0,
                                                n_adapters=60, ranks=(8, 16, 32, 64), n_dev_blocks=2500,
                                                swap_in_frac=0.0, seed=83),
    # rank 64 with 32-token tiles and a k/v width different from q/o (grouped-query shapes)
    # the paper's LoRA distributions at 1000-2000 LoRAs (section 6.9): adapters handed out in turn (every
    # sequence its own adapter, hundreds of short segments in one tiled launch), ...
    "f16_distinct_2000": lambda: small_cfg("f16", hidden=1024, n_q_heads=8, n_kv_heads=8, n_seqs=300,
                                           prefix_range=(0, 0), new_range=(2, 40), n_adapters=2000, ranks=(16,),
                                           adapter_dist="distinct", n_dev_blocks=4000, swap_in_frac=0.0, seed=85),
    # ... uniform over 2000 (almost all distinct), mixed ranks ...
    "bf16_uniform_2000": lambda: small_cfg("bf16", hidden=1024, n_q_heads=8, n_kv_heads=8, n_seqs=260,
                                           prefix_range=(0, 0), new_range=(1, 24), n_adapters=2000,
                                           ranks=(8, 16, 32, 64), adapter_dist="uniform", n_dev_blocks=6000,
                                           swap_in_frac=0.0, seed=86),
    # ... and a Gaussian over the ids (a few dozen adapters carry the batch), as a decode batch
    "bf16_skewed_1000_decode": lambda: small_cfg("bf16", hidden=1024, n_q_heads=8, n_kv_heads=8, n_seqs=700,
                                                 prefix_range=(0, 0), new_range=(1, 1), decode_frac=1.0,
                                                 n_adapters=1000, ranks=(16, 32), adapter_dist="skewed", skew_std=12.0,
                                                 n_dev_blocks=6000, swap_in_frac=0.0, seed=87),
    # over 1024 tokens with output widths that are not multiples of the large GEMM tile (q, o: 320 of 256; k, v: 64)
    "bf16_dense_tail": lambda: small_cfg("bf16", hidden=320, n_q_heads=5, n_kv_heads=1, head_dim=64, n_seqs=20,
                                         prefix_range=(0, 0), new_range=(40, 80), n_adapters=4, ranks=(16,),
                                         n_dev_blocks=1200, swap_in_frac=0.0, seed=88),
    # enough 256 x 256 tiles (11 token rows x 9 feature columns; 9.5 columns in the bf16 case) for the large-batch GEMM
    # when a dense base is given
    "f16_dense_large": lambda: small_cfg("f16", hidden=512, n_q_heads=18, n_kv_heads=18, n_seqs=24, prefix_range=(0, 0),
                                         new_range=(110, 160), n_adapters=6, ranks=(8, 16), n_dev_blocks=1500,
                                         swap_in_frac=0.0, seed=89),
    "bf16_dense_large_tail": lambda: small_cfg("bf16", hidden=512, n_q_heads=19, n_kv_heads=19, n_seqs=24,
                                               prefix_range=(0, 0), new_range=(110, 160), n_adapters=6, ranks=(16, 32),
                                               n_dev_blocks=1500, swap_in_frac=0.0, seed=90),
    "f16_rank64_gqa": lambda: small_cfg("f16", hidden=1024, n_q_heads=8, n_kv_heads=2, n_seqs=38,
                                        prefix_range=(0, 0), new_range=(30, 120), n_adapters=5, ranks=(64,),
                                        n_dev_blocks=1500, swap_in_frac=0.0, seed=84),
}


@pytest.mark.parametrize("name", list(LORA_CASES))
def test_lora_matrix_core_shapes(name):
    cfg = LORA_CASES[name]()
    step = wl.make_step(cfg)
    print("\n[lora case %s] T=%d adapters=%d" % (name, step.n_tokens, int((step.rank > 0).sum())), flush=True)
    if name in ("f16_long_segments", "f16_rank64_gqa", "f16_dense_large", "bf16_dense_large_tail"):
        assert step.n_tokens >= 2048, "this case is meant for the 32-token tiles"
    dev0 = resident_pool(step)
    g = GpuStep(step, dev0, np.zeros((1, cfg.block_elems), dev0.dtype))
    rtol, atol = TOL[cfg.dtype]
    got = g.lora(["q", "k", "v"])
    got.update(g.lora(["o"]))
    for n in ("q", "k", "v", "o"):
        pr = step.proj[n]
        want = oracle.lora_apply(dev0, cfg.dtype, step.acts["x"], step.token_adapter, step.rank, step.scale,
                                 pr.a_tab_off, pr.a_row_base, pr.b_tab_off, pr.b_row_base, step.lora_tables,
                                 pr.d_out, y_in=step.acts["base_" + n])
        ok, worst, nbad = close(wl.dequantize(got[n], cfg.dtype), want, rtol, atol)
        assert ok, "%s: max err %g, %d elements out of tolerance" % (n, worst, nbad)
        # the delta itself (not just base + delta) must be right: compare it at a tolerance scaled to its size
        base = wl.dequantize(step.acts["base_" + n], cfg.dtype)
        ulp = 2.0 ** (-10 if cfg.dtype == "f16" else -7)
        err = np.abs((wl.dequantize(got[n], cfg.dtype) - base) - (want - base))
        assert err.max() <= ulp * (np.abs(want).max() + 1.0), (n, err.max())


@pytest.mark.parametrize("dtype,ranks", [("f16", (16,)), ("bf16", (8, 32, 64))])
def test_lora_long_batch_with_input_width_not_a_multiple_of_64(dtype, ranks):
    """32-token tiles (2048 tokens and more) with an input width of 288 = 9 x 32: the LDS-staged shrink kernels need
    whole 64-coefficient chunks, so this batch takes the shrink kernel that reads its operands from global memory."""
    cfg = small_cfg(dtype, hidden=288, n_q_heads=4, n_kv_heads=2, n_seqs=24, prefix_range=(0, 0), new_range=(90, 140),
                    n_adapters=7, ranks=ranks, n_dev_blocks=1200, swap_in_frac=0.0, seed=94)
    step = wl.make_step(cfg)
    assert step.n_tokens >= 2048 and step.proj["q"].d_in == 288
    dev0 = resident_pool(step)
    g = GpuStep(step, dev0, np.zeros((1, cfg.block_elems), dev0.dtype))
    rtol, atol = TOL[cfg.dtype]
    got = g.lora(["q", "k", "v"])
    for n in ("q", "k", "v"):
        pr = step.proj[n]
        want = oracle.lora_apply(dev0, cfg.dtype, step.acts["x"], step.token_adapter, step.rank, step.scale,
                                 pr.a_tab_off, pr.a_row_base, pr.b_tab_off, pr.b_row_base, step.lora_tables,
                                 pr.d_out, y_in=step.acts["base_" + n])
        ok, worst, nbad = close(wl.dequantize(got[n], cfg.dtype), want, rtol, atol)
        assert ok, "%s: max err %g, %d elements out of tolerance" % (n, worst, nbad)
        base = wl.dequantize(step.acts["base_" + n], cfg.dtype)
        assert np.abs(want - base).max() > 10 * atol


@pytest.mark.parametrize("case", ["f16_long_segments", "bf16_dense_large_tail", "f16_rank64_gqa"])
@pytest.mark.parametrize("names", [("q", "k"), ("q", "k", "v", "o"), ("v",)])
def test_lora_call_with_one_two_or_four_projections(names, case):
    """The staged shrink kernels are compiled per number of projections in the call (they share x): calls with 1, 2
    and 4 projections on a batch long enough for the 32-token tiles (q, k, v together is covered above), at ranks
    up to 16, up to 32 and at 64 (one, two and four rank tiles; at 64 a workgroup takes two token tiles).  All
    projections read the same x here, "o" included where its input is as wide: the call does not care what x
    means."""
    cfg = LORA_CASES[case]()
    step = wl.make_step(cfg)
    assert step.n_tokens >= 2048 and cfg.hidden % 64 == 0
    assert int(step.rank.max()) == {"f16_long_segments": 16, "bf16_dense_large_tail": 32, "f16_rank64_gqa": 64}[case]
    names = tuple(n for n in names if step.proj[n].d_in == cfg.hidden)
    dev0 = resident_pool(step)
    g = GpuStep(step, dev0, np.zeros((1, cfg.block_elems), dev0.dtype))
    rtol, atol = TOL[cfg.dtype]
    got = g.lora(list(names))
    for n in names:
        pr = step.proj[n]
        assert pr.d_in == cfg.hidden
        want = oracle.lora_apply(dev0, cfg.dtype, step.acts["x"], step.token_adapter, step.rank, step.scale,
                                 pr.a_tab_off, pr.a_row_base, pr.b_tab_off, pr.b_row_base, step.lora_tables,
                                 pr.d_out, y_in=step.acts["base_" + n])
        ok, worst, nbad = close(wl.dequantize(got[n], cfg.dtype), want, rtol, atol)
        assert ok, "%s: max err %g, %d elements out of tolerance" % (n, worst, nbad)
        base = wl.dequantize(step.acts["base_" + n], cfg.dtype)
        ulp = 2.0 ** (-10 if cfg.dtype == "f16" else -7)
        err = np.abs((wl.dequantize(got[n], cfg.dtype) - base) - (want - base))
        assert err.max() <= ulp * (np.abs(want).max() + 1.0), (n, err.max())
        assert np.abs(want - base).max() > 10 * atol


@pytest.mark.parametrize("dtype,ranks,heads,scale", [("f16", (16,), 3, 1), ("bf16", (8, 32), 5, 1), ("bf16", (64,), 6, 1),
                                                     ("f16", (8, 64), 7, 1), ("f16", (16,), 67, 4)])
def test_lora_expand_slab_and_group_edges(dtype, ranks, heads, scale):
    """Long batches: the expand step takes slabs of 256 columns in halves of 128 and groups of 64 tokens (128 with 17 slabs in
    each of three projections) sixteen at a time.  Widths of 192, 320, 384, 448 and 4288 columns (last slabs of 64, 128 and 192),
    and adapters that own one token, one less, as many and one more than a sub-tile, four sub-tiles, and one and two
    groups, each scattered over the batch; tokens without an adapter keep their bits."""
    cfg = small_cfg(dtype, hidden=128, n_q_heads=heads, n_kv_heads=heads, head_dim=64, n_seqs=40, prefix_range=(0, 0),
                    new_range=(28 * scale, 36 * scale), n_adapters=24, ranks=ranks, adapter_dist="distinct", n_dev_blocks=1200,
                    swap_in_frac=0.0, seed=500 + heads)
    step = wl.make_step(cfg)
    T = step.n_tokens
    present = np.unique(step.token_adapter)
    runs = [1, 15, 16, 17, 63, 64, 65, 127, 128, 129, 255, 257]
    ta = np.full(T, present[-1], np.int32)
    ta[:7] = -1
    at = 7
    for ad, n in zip(present, runs):
        ta[at:at + n] = ad
        at += n
    assert T >= 1024 and at < T - 1 and len(present) > len(runs)
    step.token_adapter = ta[np.random.default_rng(heads).permutation(T)]
    dev0 = resident_pool(step)
    g = GpuStep(step, dev0, np.zeros((1, cfg.block_elems), dev0.dtype))
    rtol, atol = TOL[cfg.dtype]
    got = g.lora(["q", "k", "v"])
    for n in ("q", "k", "v"):
        pr = step.proj[n]
        want = oracle.lora_apply(dev0, cfg.dtype, step.acts["x"], step.token_adapter, step.rank, step.scale,
                                 pr.a_tab_off, pr.a_row_base, pr.b_tab_off, pr.b_row_base, step.lora_tables,
                                 pr.d_out, y_in=step.acts["base_" + n])
        ok, worst, nbad = close(wl.dequantize(got[n], cfg.dtype), want, rtol, atol)
        assert ok, "%s: max err %g, %d elements out of tolerance" % (n, worst, nbad)
        base = wl.dequantize(step.acts["base_" + n], cfg.dtype)
        ulp = 2.0 ** (-10 if cfg.dtype == "f16" else -7)
        err = np.abs((wl.dequantize(got[n], cfg.dtype) - base) - (want - base))
        assert err.max() <= ulp * (np.abs(want).max() + 1.0), (n, err.max())
        none = step.token_adapter < 0
        assert np.array_equal(got[n][none], step.acts["base_" + n][none])


@pytest.mark.parametrize("dtype,ranks,heads", [("f16", (8, 16), 17), ("bf16", (16,), 6), ("f16", (8, 32), 17)])
def test_lora_expand_of_many_adapters_with_few_tokens(dtype, ranks, heads):
    """1024 tokens and more of 300 adapters with 1 to 20 tokens each: more groups than the launch takes in one turn, most of up to
    sixteen tokens, whose workgroup takes four slabs of 256 columns (ranks up to 16; widths of 1088 and 384 columns: five slabs
    and two), some of more."""
    cfg = small_cfg(dtype, hidden=128, n_q_heads=heads, n_kv_heads=heads, head_dim=64, n_seqs=300, prefix_range=(0, 0), new_range=(1, 8),
                    n_adapters=300, ranks=ranks, adapter_dist="distinct", n_dev_blocks=2400, swap_in_frac=0.0, seed=520 + heads)
    step = wl.make_step(cfg)
    rng = np.random.default_rng(heads)
    for ad in rng.choice(step.seq_adapter, 20, replace=False):          # up to 20 tokens, scattered
        step.token_adapter[rng.choice(step.n_tokens, 14, replace=False)] = ad
    step.token_adapter[::31] = -1
    present, counts = np.unique(step.token_adapter[step.token_adapter >= 0], return_counts=True)
    assert step.n_tokens >= 1024 and len(present) > 200 and counts.max() > 16 and (counts <= 16).sum() > 200
    dev0 = resident_pool(step)
    g = GpuStep(step, dev0, np.zeros((1, cfg.block_elems), dev0.dtype))
    rtol, atol = TOL[cfg.dtype]
    got = g.lora(["q", "k", "v"])
    for n in ("q", "k", "v"):
        pr = step.proj[n]
        want = oracle.lora_apply(dev0, cfg.dtype, step.acts["x"], step.token_adapter, step.rank, step.scale,
                                 pr.a_tab_off, pr.a_row_base, pr.b_tab_off, pr.b_row_base, step.lora_tables,
                                 pr.d_out, y_in=step.acts["base_" + n])
        base = wl.dequantize(step.acts["base_" + n], cfg.dtype)
        value = wl.dequantize(got[n], cfg.dtype)
        ok, worst, nbad = close(value, want, rtol, atol)
        assert ok, "%s: max err %g, %d elements out of tolerance" % (n, worst, nbad)
        ulp = 2.0 ** (-10 if cfg.dtype == "f16" else -7)
        assert np.abs((value - base) - (want - base)).max() <= ulp * (np.abs(want).max() + 1.0)
        none = step.token_adapter < 0
        assert np.array_equal(got[n][none], step.acts["base_" + n][none])


@pytest.mark.parametrize("dtype,T", [("bf16", 1), ("bf16", 63), ("f32", 257), ("bf16", 1023), ("f16", 1024),
                                     ("f32", 1025)])
def test_lora_small_batches_share_adapter_pages(dtype, T):
    """Batches of up to 1024 tokens take the tokens of one adapter together, sixteen at a time in 16 bits and four at a time in
    the vector kernels (fp32): batches around that limit and around the 64-token words of the kernels' bit masks, with
    adapters that own one token, a few, or a third of the batch, tokens without an adapter, and widths that do not
    fill the column slabs."""
    cfg = small_cfg(dtype, hidden=320, n_q_heads=5, n_kv_heads=1, head_dim=64, n_seqs=T, prefix_range=(0, 0),
                    new_range=(1, 1), decode_frac=1.0, n_adapters=40, ranks=(8, 16, 32, 64), n_dev_blocks=2600,
                    swap_in_frac=0.0, seed=300 + T)
    step = wl.make_step(cfg)
    rng = np.random.default_rng(T)
    ta = step.token_adapter.copy()
    if T > 8:
        ta[rng.choice(T, size=T // 3, replace=False)] = 3               # one heavy adapter: many fours
        ta[rng.choice(T, size=T // 10, replace=False)] = -1             # tokens without an adapter
        ta[T - 1] = 3
    step.token_adapter = ta
    dev0 = resident_pool(step)
    g = GpuStep(step, dev0, np.zeros((1, cfg.block_elems), dev0.dtype))
    rtol, atol = TOL[cfg.dtype]
    got = g.lora(["q", "k", "v"])
    got.update(g.lora(["o"]))
    for n in ("q", "k", "v", "o"):
        pr = step.proj[n]
        want = oracle.lora_apply(dev0, cfg.dtype, step.acts["x"], ta, step.rank, step.scale, pr.a_tab_off,
                                 pr.a_row_base, pr.b_tab_off, pr.b_row_base, step.lora_tables, pr.d_out,
                                 y_in=step.acts["base_" + n])
        ok, worst, nbad = close(wl.dequantize(got[n], cfg.dtype), want, rtol, atol)
        assert ok, "%s: max err %g, %d elements out of tolerance" % (n, worst, nbad)
        base = wl.dequantize(step.acts["base_" + n], cfg.dtype)
        none = ta < 0
        if none.any():                                                   # rows without an adapter are untouched
            assert np.array_equal(got[n][none], step.acts["base_" + n][none])
        assert np.abs(want - base)[~none].max() > 0


@pytest.mark.parametrize("name", ["tiny", "f16_prefill", "bf16_gqa_mixed", "f16_long_segments", "bf16_dense_tail",
                                  "f16_dense_large", "bf16_dense_large_tail"])
def test_lora_with_dense_base(name):
    """w_base given: y = x.W_base + delta, the library computes the base term itself (Eq. 1's W)."""
    cfg = (CASES.get(name) or LORA_CASES[name])()
    step = wl.make_step(cfg)
    rng = np.random.default_rng(55)
    if "large" in name:
        # tokens without an adapter inside the batch: one whole sequence, and single tokens inside other sequences
        # (the LoRA branch is added inside the GEMM there, per adapter present among a wave's 128 tokens)
        ta = step.token_adapter.copy()
        ta[step.cu_new[3]:step.cu_new[4]] = -1
        ta[rng.choice(step.n_tokens, size=50, replace=False)] = -1
        ta[step.cu_new[7] + 5:step.cu_new[7] + 9] = step.token_adapter[step.cu_new[9]]   # another sequence's adapter mid-sequence
        step.token_adapter = ta
    dev0 = resident_pool(step)
    g = GpuStep(step, dev0, np.zeros((1, cfg.block_elems), dev0.dtype))
    rtol, atol = TOL[cfg.dtype]
    names = [p for p in cfg.projections if p in ("q", "k", "v")]
    W = {n: wl.quantize((rng.standard_normal((cfg.hidden, step.proj[n].d_out)) / np.sqrt(cfg.hidden)).astype(np.float32),
                        cfg.dtype) for n in names}
    got = g.lora(names, w_base={n: to_dev(W[n]) for n in names})
    # a random sample, both ends of every sequence (where the adapter changes inside a tile) and the end of the batch
    T = step.n_tokens
    sel = np.unique(np.concatenate([rng.choice(T, size=min(T, 64), replace=False), step.cu_new[:-1],
                                    step.cu_new[1:] - 1, np.arange(max(0, T - 40), T)])).astype(np.int32)
    if "large" in name:
        sel = np.unique(np.concatenate([sel, np.flatnonzero(step.token_adapter < 0)[:60],
                                        np.arange(step.cu_new[7], step.cu_new[7] + 12)])).astype(np.int32)
    sel = sel[(sel >= 0) & (sel < T)]
    for n in names:
        pr = step.proj[n]
        want = oracle.lora_apply(dev0, cfg.dtype, step.acts["x"], step.token_adapter, step.rank, step.scale,
                                 pr.a_tab_off, pr.a_row_base, pr.b_tab_off, pr.b_row_base, step.lora_tables,
                                 pr.d_out, w_base=W[n], sel=sel)
        ok, worst, nbad = close(wl.dequantize(got[n][sel], cfg.dtype), want, rtol, atol)
        assert ok, "%s: max err %g, %d elements out of tolerance" % (n, worst, nbad)
        assert np.abs(want).max() > 1.0          # the base term is really there


def test_segmentation_bit_exact():
    import torch
    rng = np.random.default_rng(9)
    pool = flpool.Pool("f16", 1, 64, 2, 0)
    for T, n_ad in [(1, 1), (63, 5), (64, 5), (1000, 40), (5000, 300), (20000, 2048), (257, 100)]:
        ta = rng.integers(-1, n_ad, size=T).astype(np.int32)
        if T > 100:
            ta[rng.integers(0, T, size=T // 2)] = rng.integers(0, min(3, n_ad))      # a few heavy adapters
        seg_adapter, seg_start, perm = oracle.segment(ta, n_ad)
        d_ta = to_dev(ta)
        d_nseg = torch.zeros(1, dtype=torch.int32, device="cuda")
        d_sa = torch.full((n_ad,), -7, dtype=torch.int32, device="cuda")
        d_ss = torch.full((n_ad + 1,), -7, dtype=torch.int32, device="cuda")
        d_perm = torch.full((T,), -7, dtype=torch.int32, device="cuda")
        pool.lora_segment(d_ta, T, n_ad, d_nseg, d_sa, d_ss, d_perm)
        torch.cuda.synchronize()
        n = int(d_nseg.item())
        assert n == len(seg_adapter)
        assert np.array_equal(d_sa.cpu().numpy()[:n], seg_adapter)
        assert np.array_equal(d_ss.cpu().numpy()[:n + 1], seg_start)
        assert np.array_equal(d_perm.cpu().numpy()[:seg_start[n]], perm)


@pytest.mark.parametrize("T,n_ad", [(1023, 7), (1024, 1), (1025, 40), (2049, 3), (16384, 2048), (16385, 17), (33000, 500)])
def test_segmentation_by_several_workgroups(T, n_ad):
    """Batches of one workgroup's range and around it, the most workgroups, and ranges of several steps; runs of equal ids as
    sequences make them, over the edges of the ranges, mixed ids, and ids that name no adapter."""
    rng = np.random.default_rng(T)
    ta = np.repeat(rng.integers(-1, n_ad, size=T), rng.integers(1, 400, size=T))[:T].astype(np.int32)
    ta[T // 3:T // 2] = rng.integers(-1, n_ad + 1, size=T // 2 - T // 3)
    seg_adapter, seg_start, perm = oracle.segment(np.where(ta < n_ad, ta, -1).astype(np.int32), n_ad)
    pool = flpool.Pool("f16", 1, 64, 2, 0)
    d_nseg, d_sa, d_ss, d_perm = (torch.full((n,), -7, dtype=torch.int32, device="cuda") for n in (1, n_ad, n_ad + 1, T))
    pool.lora_segment(to_dev(ta), T, n_ad, d_nseg, d_sa, d_ss, d_perm)
    n = int(d_nseg.item())
    assert n == len(seg_adapter)
    assert np.array_equal(d_sa.cpu().numpy()[:n], seg_adapter) and bool((d_sa[n:] == -7).all())
    assert np.array_equal(d_ss.cpu().numpy()[:n + 1], seg_start)
    assert np.array_equal(d_perm.cpu().numpy()[:seg_start[n]], perm[:seg_start[n]]) and bool((d_perm[seg_start[n]:] == -7).all())
    pool.close()


def test_degenerate_batches():
    import torch
    cfg = small_cfg("f16", n_seqs=5, prefix_range=(64, 64), new_range=(16, 16), seed=90)
    step = wl.make_step(cfg)
    # sequences with zero new tokens, zero prefix, a single token, a prefix ending on a block boundary
    step.prefix_len[:] = [0, 16, 33, 0, 48]
    step.new_len[:] = [1, 0, 5, 17, 16]
    step.cu_new[1:] = np.cumsum(step.new_len)
    T = int(step.cu_new[-1])
    for k in ("q", "k_new", "v_new"):
        step.acts[k] = step.acts[k][:T].copy()
    dev0 = resident_pool(step)
    dev0[step.content_ids] = wl.quantize(np.random.default_rng(1).standard_normal(step.content.shape), "f16")
    g = GpuStep(step, dev0, np.zeros((1, cfg.block_elems), dev0.dtype))
    got = wl.dequantize(g.attention(append=True), "f16").reshape(T, cfg.n_q_heads, cfg.head_dim)
    ref_pool = dev0.copy()
    oracle.kv_append(ref_pool, "f16", 16, cfg.n_kv_heads, cfg.head_dim, step.cu_new, step.prefix_len, step.kv_tables,
                     step.acts["k_new"], step.acts["v_new"])
    want = oracle.paged_attention(ref_pool, "f16", 16, cfg.n_kv_heads, cfg.head_dim, cfg.n_q_heads, step.cu_new,
                                  step.prefix_len, step.kv_tables, step.acts["q"])
    ok, worst, nbad = close(got, want, *TOL["f16"])
    assert ok, (worst, nbad)
    # P = 0, N = 1: the output is exactly v0 (softmax over a single key)
    v0 = wl.dequantize(step.acts["v_new"][0], "f16").reshape(cfg.n_kv_heads, cfg.head_dim)
    assert np.array_equal(got[0], v0)
    # empty batch and all-empty sequences enqueue nothing and succeed
    g.pool.paged_prefix_attention(g.acts["q"], g.acts["q"], [0], [], g.kv_tables, cfg.n_q_heads)
    g.pool.paged_prefix_attention(g.acts["q"], g.acts["q"], [0, 0, 0], [3, 4], g.kv_tables, cfg.n_q_heads)
    g.pool.swap_in([], [])
    torch.cuda.synchronize()


def test_lora_no_adapter_tokens_and_zero_b():
    cfg = small_cfg("bf16", seed=91)
    step = wl.make_step(cfg)
    step.token_adapter[::3] = -1
    dev0 = resident_pool(step)
    g = GpuStep(step, dev0, np.zeros((1, cfg.block_elems), dev0.dtype))
    got = g.lora(["q"])["q"]
    none = np.flatnonzero(step.token_adapter < 0)
    assert np.array_equal(got[none], step.acts["base_q"][none])           # untouched rows, bit for bit
    pr = step.proj["q"]
    want = oracle.lora_apply(dev0, "bf16", step.acts["x"], step.token_adapter, step.rank, step.scale, pr.a_tab_off,
                             pr.a_row_base, pr.b_tab_off, pr.b_row_base, step.lora_tables, pr.d_out,
                             y_in=step.acts["base_q"])
    ok, worst, nbad = close(wl.dequantize(got, "bf16"), want, *TOL["bf16"])
    assert ok, (worst, nbad)
    # B = 0 for every adapter: y is the base term exactly
    zero = dev0.copy()
    for a in np.flatnonzero(step.rank):
        for rho in range(step.rank[a]):
            oracle.lora_write_row(zero, "bf16", step.lora_tables[pr.b_tab_off[a]:], pr.b_row_base[a] + rho,
                                  np.zeros(pr.d_out, np.uint16))
    g2 = GpuStep(step, zero, np.zeros((1, cfg.block_elems), dev0.dtype))
    assert np.array_equal(g2.lora(["q"])["q"], step.acts["base_q"])


@pytest.mark.parametrize("with_base", [False, True])
@pytest.mark.parametrize("dtype,ranks", [("f16", (16,)), ("bf16", (32,)), ("f16", (64,)), ("bf16", (8, 16, 32, 64))])
def test_lora_adapters_drawn_per_token(dtype, ranks, with_base):
    """Every token draws its adapter on its own (12 adapters and "none"), so a 32-token tile of the sorted batch, a
    256-token tile group and the 128 tokens of a GEMM wave all mix adapters, segments end inside tiles, and rows
    without an adapter sit between the others: on the tiled path (2816 tokens and more), without a dense base
    (shrink and expand kernels) and with one (the LoRA branch inside the large-batch GEMM), at one, two and four
    rank tiles and with mixed ranks."""
    cfg = small_cfg(dtype, hidden=512, n_q_heads=18, n_kv_heads=18, n_seqs=24, prefix_range=(0, 0),
                    new_range=(118, 160), n_adapters=12, ranks=ranks, adapter_dist="distinct", n_dev_blocks=2400,
                    swap_in_frac=0.0, seed=120 + len(ranks) + ranks[0])
    step = wl.make_step(cfg)                    # "distinct" over 24 sequences: all 12 adapters get pages
    T = step.n_tokens
    assert T >= 2816 and int((step.rank > 0).sum()) == 12
    rng = np.random.default_rng(ranks[0])
    step.token_adapter = rng.integers(-1, 12, size=T).astype(np.int32)
    dev0 = resident_pool(step)
    g = GpuStep(step, dev0, np.zeros((1, cfg.block_elems), dev0.dtype))
    rtol, atol = TOL[cfg.dtype]
    names = ["q", "k", "v"]
    W = None
    if with_base:
        W = {n: wl.quantize((rng.standard_normal((cfg.hidden, step.proj[n].d_out)) / np.sqrt(cfg.hidden))
                            .astype(np.float32), cfg.dtype) for n in names}
    got = g.lora(names, w_base={n: to_dev(W[n]) for n in names} if W else None)
    sel = np.arange(T, dtype=np.int32) if not with_base else np.unique(np.concatenate(
        [rng.choice(T, size=300, replace=False), np.arange(0, 140), np.arange(T - 140, T)])).astype(np.int32)
    none = step.token_adapter < 0
    assert none.sum() > 100
    ulp = 2.0 ** (-10 if cfg.dtype == "f16" else -7)
    for n in names:
        pr = step.proj[n]
        want = oracle.lora_apply(dev0, cfg.dtype, step.acts["x"], step.token_adapter, step.rank, step.scale,
                                 pr.a_tab_off, pr.a_row_base, pr.b_tab_off, pr.b_row_base, step.lora_tables,
                                 pr.d_out, y_in=None if W else step.acts["base_" + n], w_base=W[n] if W else None,
                                 sel=sel)
        ok, worst, nbad = close(wl.dequantize(got[n][sel], cfg.dtype), want, rtol, atol)
        assert ok, "%s: max err %g, %d elements out of tolerance" % (n, worst, nbad)
        if not W:
            base = wl.dequantize(step.acts["base_" + n], cfg.dtype)
            assert np.array_equal(got[n][none], step.acts["base_" + n][none])     # rows without an adapter untouched
            err = np.abs((wl.dequantize(got[n], cfg.dtype) - base) - (want - base))
            assert err.max() <= ulp * (np.abs(want).max() + 1.0), (n, err.max())
            assert np.abs(want - base)[~none].max() > 10 * atol
        else:
            # the branch is there: rows with an adapter differ from the dense product alone by more than the bound
            dense = oracle.lora_apply(dev0, cfg.dtype, step.acts["x"], np.full(T, -1, np.int32), step.rank, step.scale,
                                      pr.a_tab_off, pr.a_row_base, pr.b_tab_off, pr.b_row_base, step.lora_tables,
                                      pr.d_out, w_base=W[n], sel=sel)
            with_ad = ~none[sel]
            assert np.abs(want - dense)[with_ad].max() > 10 * atol
            # compare the branch itself at one spacing of the element type at the output's magnitude plus the
            # rounding of the sum
            err = np.abs((wl.dequantize(got[n][sel], cfg.dtype) - dense) - (want - dense))
            assert err.max() <= 1.5 * ulp * (np.abs(want).max() + 1.0), (n, err.max())


@pytest.mark.parametrize("dtype,bt,gqa", [("f16", 16, False), ("bf16", 16, True), ("f16", 32, False)])
def test_attention_over_shared_prefix_blocks(dtype, bt, gqa):
    """Sequences of one adapter share the physical blocks of a common prefix (paper section 4.1; KV of different
    LoRAs is never shared, section 2.1): block ids repeat across tables.  Append writes only the sequences' own
    blocks; attention reads the shared ones from every table that names them.  Prefill rows (matrix-core kernel)
    and, in the grouped-query case, decode rows mixed in."""
    kw = dict(n_q_heads=8, n_kv_heads=2, hidden=1024, decode_frac=0.4) if gqa else {}
    cfg = small_cfg(dtype, block_tokens=bt, n_seqs=24, n_adapters=3, prefix_range=(40, 420), new_range=(1, 90),
                    share_frac=0.85, n_dev_blocks=1500, swap_in_frac=0.0, seed=131 + bt + gqa, **kw)
    step = wl.make_step(cfg)
    ids, counts = np.unique(step.kv_tables[step.kv_tables >= 0], return_counts=True)
    assert (counts > 1).sum() >= 20 and counts.max() >= 3, "the case shares too little"
    dev0 = resident_pool(step)
    g = GpuStep(step, dev0, np.zeros((1, cfg.block_elems), dev0.dtype))
    n_kv, d, n_h = cfg.n_kv_heads, cfg.head_dim, cfg.n_q_heads
    out = g.attention(append=True)
    ref = dev0.copy()
    oracle.kv_append(ref, cfg.dtype, bt, n_kv, d, step.cu_new, step.prefix_len, step.kv_tables, step.acts["k_new"],
                     step.acts["v_new"])
    assert np.array_equal(g.dev_image().view(np.uint8), ref.view(np.uint8)), "append touched a shared block"
    shared = ids[counts > 1]
    assert np.array_equal(ref[shared], dev0[shared])                      # shared blocks are prefix blocks: unchanged
    want = oracle.paged_attention(ref, cfg.dtype, bt, n_kv, d, n_h, step.cu_new, step.prefix_len, step.kv_tables,
                                  step.acts["q"])
    ok, worst, nbad = close(wl.dequantize(out, cfg.dtype).reshape(want.shape), want, *TOL[cfg.dtype])
    assert ok, "max err %g (%d bad)" % (worst, nbad)


@pytest.mark.parametrize("dtype,heads,kv,d,seqs,prefix,new", [
    ("bf16", 32, 32, 128, 3, (3000, 9000), (1, 1)),       # a handful of decode sequences with long contexts
    ("f16", 8, 8, 64, 2, (2000, 5000), (1, 1)),
    ("f32", 4, 4, 128, 2, (1500, 2500), (1, 1)),
    ("bf16", 16, 2, 128, 4, (4000, 12000), (1, 1)),       # grouped-query decode: too few matrix-core items, rows + split
    ("f16", 8, 8, 128, 5, (100, 6000), (1, 3)),           # short and long contexts mixed, up to three new tokens
])
def test_split_kv_for_few_long_sequences(dtype, heads, kv, d, seqs, prefix, new):
    """Few rows over long contexts: the context of a row is cut into pieces, a wave each, and the pieces are merged in
    a fixed order (the split-KV form of the same softmax).  Against the oracle, and twice for identical bits."""
    cfg = small_cfg(dtype, hidden=heads * d, n_q_heads=heads, n_kv_heads=kv, head_dim=d, n_seqs=seqs,
                    prefix_range=prefix, new_range=new, decode_frac=1.0 if new == (1, 1) else 0.0, n_adapters=2,
                    ranks=(8,), projections=("q",), n_dev_blocks=seqs * (prefix[1] // 16 + 3) + 64, swap_in_frac=0.0,
                    seed=500 + heads + seqs)
    step = wl.make_step(cfg)
    assert step.n_tokens * heads < 2048                        # under the kernel's fill: the split path is taken
    dev0 = resident_pool(step)
    g = GpuStep(step, dev0, np.zeros((1, cfg.block_elems), dev0.dtype))
    out1 = g.attention(append=True)
    out2 = g.attention(append=False)                           # the fresh K/V are in place: same inputs, same bits
    assert np.array_equal(out1, out2)
    ref = dev0.copy()
    oracle.kv_append(ref, dtype, 16, kv, d, step.cu_new, step.prefix_len, step.kv_tables, step.acts["k_new"],
                     step.acts["v_new"])
    want = oracle.paged_attention(ref, dtype, 16, kv, d, heads, step.cu_new, step.prefix_len, step.kv_tables,
                                  step.acts["q"])
    ok, worst, nbad = close(wl.dequantize(out1, dtype).reshape(want.shape), want, *TOL[dtype])
    assert ok, "max err %g (%d bad)" % (worst, nbad)


@pytest.mark.parametrize("dtype,bt,heads,kv,ctx", [
    ("f16", 16, 8, 8, (1, 2, 15, 16, 17, 31, 32, 33)),          # one row per kv head; one, two and three tiles of positions
    ("bf16", 16, 32, 2, (1, 33, 255, 256, 257, 511, 513)),      # 16 rows per kv head, around one piece and two
    ("f16", 32, 15, 5, (16, 17, 32, 47, 48, 65, 300, 1100)),    # 3 rows per kv head, blocks of 32, kv heads not a multiple of 4
    ("bf16", 32, 16, 2, (31, 64, 769, 1025, 2047)),
    ("bf16", 16, 8, 2, (7, 300, 513)),                          # 4 and 5 rows per kv head
    ("f16", 32, 20, 4, (33, 600)),
    ("f16", 16, 34, 2, (5, 40, 700)),                           # 17 rows per kv head: past what one wave holds
])
def test_single_token_attention_at_the_edges_of_groups_tiles_and_pieces(dtype, bt, heads, kv, ctx):
    """One new token per sequence, contexts around the edges of groups (16), tiles (32) and pieces (256 positions).
    Slots past a context hold NaN, one visible V is infinite (its channel of that sequence alone becomes infinite)."""
    d = 128
    rng = np.random.default_rng(7 + heads + len(ctx))
    n_blk = [(c + bt - 1) // bt for c in ctx]
    n = sum(n_blk)
    ids = rng.permutation(n).astype(np.int32)
    tables = np.full((len(ctx), max(n_blk)), -1, np.int32)
    at = 0
    for i, k in enumerate(n_blk):
        tables[i, :k] = ids[at:at + k]
        at += k
    cu, prefix = np.arange(len(ctx) + 1, dtype=np.int32), np.array(ctx, np.int32) - 1
    tt = torch.float16 if dtype == "f16" else torch.bfloat16
    K, V = (torch.from_numpy(rng.standard_normal((n, kv, bt, d)).astype(np.float32)).to(tt) for _ in range(2))
    V = V.transpose(2, 3).contiguous()                          # [block, kv head, channel, slot]
    for i, c in enumerate(ctx):
        if c % bt:
            K[tables[i, n_blk[i] - 1], :, c % bt:] = float("nan")
            V[tables[i, n_blk[i] - 1], :, :, c % bt:] = float("nan")
    V[tables[-1, 0], 0, 3, 2] = float("inf")
    q = torch.from_numpy(rng.standard_normal((len(ctx), heads, d)).astype(np.float32)).to(tt)
    dev = torch.cat([K.reshape(n, -1), V.reshape(n, -1)], 1).contiguous().cuda()
    pool = flpool.Pool(dtype, kv, d, n, 0, block_tokens=bt, dev=dev)
    out = torch.empty_like(q, device="cuda")
    pool.paged_prefix_attention(q.cuda(), out, cu, prefix, torch.from_numpy(tables).cuda(), heads)
    got = out.cpu().double()
    G = heads // kv
    for i, c in enumerate(ctx):
        tab = torch.from_numpy(tables[i, :n_blk[i]].astype(np.int64))
        k = K[tab].double().permute(1, 0, 2, 3).reshape(kv, -1, d)[:, :c].repeat_interleave(G, 0)
        v = V[tab].double().permute(1, 0, 3, 2).reshape(kv, -1, d)[:, :c].repeat_interleave(G, 0)
        w = torch.softmax(torch.einsum("hd,hcd->hc", q[i].double(), k) / d ** 0.5, 1)
        want = torch.einsum("hc,hcd->hd", w, v)
        inf = torch.isinf(want)
        assert torch.equal(got[i][inf], want[inf]) and int(inf.sum()) == (G if i == len(ctx) - 1 else 0)
        err = (got[i] - want)[~inf].abs()
        # the result's own rounding (2^-11 or 2^-8 of it) plus the errors of 32-bit weights and sums over up to 2^11 positions
        bound = (2.0 ** -11 if dtype == "f16" else 2.0 ** -8) * want.abs() + 2.0 ** -15 * torch.einsum("hc,hcd->hd", w, v.abs())
        assert bool((err <= bound[~inf] + 1e-7).all()), (c, float(err.max()))


@pytest.mark.parametrize("dtype,bt,heads,kv,seqs", [
    # (prefix, new): one key tile and its neighbours, one row tile of a wave (16 rows) and of a workgroup (256) and theirs
    ("f16", 16, 2, 2, ((0, 8), (0, 15), (0, 17), (0, 63), (0, 64), (0, 65), (1, 31), (47, 33), (63, 256), (64, 257))),
    ("bf16", 16, 16, 2, ((0, 5), (59, 5), (60, 5), (120, 9), (511, 32), (500, 33))),           # 8 rows per token
    ("bf16", 32, 3, 3, ((0, 33), (31, 95), (32, 96), (129, 130), (190, 300))),
    ("f16", 32, 10, 2, ((0, 7), (700, 26), (13, 52))),                                         # 5 rows per token
    # items of 128 rows (144 of them) and, with more than 256 of those, of 256 (320)
    ("bf16", 16, 16, 16, ((0, 127), (0, 128), (0, 129), (63, 256), (64, 257))),
    ("f16", 16, 32, 32, ((63, 256), (64, 257), (0, 255), (130, 300))),
    # single tokens beside tiles in one launch: contexts of one piece and of several, pairs that do not fill a workgroup, and more
    # workgroups of them than of tiles
    ("bf16", 16, 5, 5, ((0, 1), (255, 1), (256, 1), (1500, 1), (33, 7), (63, 256), (2100, 2))),
    ("f16", 32, 4, 2, ((700, 1), (0, 3), (90, 40))),
    ("f16", 16, 3, 3, tuple((40 * i, 1) for i in range(60)) + ((9, 8),)),
])
def test_tiled_attention_at_the_edges_of_tiles(dtype, bt, heads, kv, seqs):
    """New tokens over prefixes around the edges of key tiles (64 positions), the row tiles of a wave and of a workgroup.
    Slots past a sequence's end hold NaN."""
    d, G = 128, heads // kv
    rng = np.random.default_rng(17 + heads + bt)
    n_blk = [(p + n + bt - 1) // bt for p, n in seqs]
    ids = rng.permutation(sum(n_blk)).astype(np.int32)
    tables = np.full((len(seqs), max(n_blk)), -1, np.int32)
    at = 0
    for i, k in enumerate(n_blk):
        tables[i, :k] = ids[at:at + k]
        at += k
    cu = np.concatenate([[0], np.cumsum([n for _, n in seqs])]).astype(np.int32)
    prefix = np.array([p for p, _ in seqs], np.int32)
    tt = torch.float16 if dtype == "f16" else torch.bfloat16
    K, V = (torch.from_numpy(rng.standard_normal((at, kv, bt, d)).astype(np.float32)).to(tt) for _ in range(2))
    V = V.transpose(2, 3).contiguous()                          # [block, kv head, channel, slot]
    for i, (p, n) in enumerate(seqs):
        if (p + n) % bt:
            K[tables[i, n_blk[i] - 1], :, (p + n) % bt:] = float("nan")
            V[tables[i, n_blk[i] - 1], :, :, (p + n) % bt:] = float("nan")
    q = torch.from_numpy(rng.standard_normal((int(cu[-1]), heads, d)).astype(np.float32)).to(tt)
    dev = torch.cat([K.reshape(at, -1), V.reshape(at, -1)], 1).contiguous().cuda()
    pool = flpool.Pool(dtype, kv, d, at, 0, block_tokens=bt, dev=dev)
    out = torch.empty_like(q, device="cuda")
    pool.paged_prefix_attention(q.cuda(), out, cu, prefix, torch.from_numpy(tables).cuda(), heads)
    got = out.cpu().double()
    u = 2.0 ** -11 if dtype == "f16" else 2.0 ** -8
    for i, (p, n) in enumerate(seqs):
        tab = torch.from_numpy(tables[i, :n_blk[i]].astype(np.int64))
        k = K[tab].double().permute(1, 0, 2, 3).reshape(kv, -1, d)[:, :p + n].repeat_interleave(G, 0)
        v = V[tab].double().permute(1, 0, 3, 2).reshape(kv, -1, d)[:, :p + n].repeat_interleave(G, 0)
        s = torch.matmul(q[cu[i]:cu[i + 1]].double().transpose(0, 1), k.transpose(1, 2)) / d ** 0.5      # [head, row, key]
        s = s.masked_fill(torch.arange(p + n)[None, None] > p + torch.arange(n)[None, :, None], float("-inf"))
        w = torch.softmax(s, 2)
        want, size = torch.matmul(w, v).transpose(0, 1), torch.matmul(w, v.abs()).transpose(0, 1)
        # the result's rounding, that of the 16-bit weights and of their sum, and fp16 weights below the normal range (their
        # sum is at least 1, so each is off by at most 2^-25 of it), plus 32-bit sums
        bound = u * want.abs() + (2 * u + 2.0 ** -15) * size + 2.0 ** -25 * v.abs().sum(1)[None]
        err = (got[cu[i]:cu[i + 1]] - want).abs()
        assert bool((err <= bound).all()), (p, n, float((err / bound).max()))


@pytest.mark.parametrize("route,dtype,bt,heads,kv,seqs", [
    ("behind", "bf16", 16, 5, 5, ((0, 1), (255, 1), (256, 1), (1500, 1), (33, 7), (63, 256), (2100, 2))),
    ("behind", "f16", 32, 4, 2, ((700, 1), (0, 3), (290, 40))),
    ("behind", "f16", 16, 3, 3, tuple((40 * i, 1) for i in range(60)) + ((300, 8),)),
    ("behind", "bf16", 16, 8, 8, ((30, 20), (255, 1), (0, 1))),                                # all of them short
    ("between", "f16", 16, 16, 16, tuple((3 * i, 9) for i in range(47)) + ((600, 1), (250, 9), (0, 1), (1300, 1), (77, 3))),
    ("apart", "bf16", 16, 16, 16, tuple((3 * i, 9) for i in range(15)) + ((600, 1), (250, 9), (0, 1), (77, 3))),       # 256 items
    ("apart", "f16", 16, 4, 4, ((30, 20), (256, 1))),
])
def test_single_tokens_beside_tiles(route, dtype, bt, heads, kv, seqs):
    """Single tokens in the tiles' launch, behind and between them, and in their own: contexts of one piece and of several, pairs that
    do not fill a workgroup, and more workgroups of them than of tiles."""
    from helpers import attention_route
    assert attention_route(heads, kv, bt, seqs) == route
    test_tiled_attention_at_the_edges_of_tiles(dtype, bt, heads, kv, seqs)


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_merge_of_up_to_64_pieces(dtype):
    """8, 9, 16, 17, 32, 33 and 64 pieces of 256 positions: the edges of what the merge requests together."""
    test_single_token_attention_at_the_edges_of_groups_tiles_and_pieces(dtype, 16, 2, 2, (2048, 2049, 4096, 4097, 8192, 8193, 16384))


def _single_tokens(dtype, ctx, q, K, V):
    """Attention of one new token per sequence of `ctx` positions: q [seqs, heads, d], K and V [seqs, heads, ctx, d] in
    the pool's type.  Returns the result and, in fp64, the weights' sum with V and with |V|."""
    n, heads, d = q.shape
    bt = 16
    nb = (ctx + bt - 1) // bt
    pad = torch.zeros((n, heads, nb * bt - ctx, d), dtype=K.dtype)
    kb, vb = (torch.cat([t, pad], 2).reshape(n, heads, nb, bt, d).permute(0, 2, 1, 3, 4) for t in (K, V))
    dev = torch.cat([kb.reshape(n * nb, -1), vb.transpose(3, 4).reshape(n * nb, -1)], 1).contiguous().cuda()
    pool = flpool.Pool(dtype, heads, d, n * nb, 0, block_tokens=bt, dev=dev)
    out = torch.empty_like(q, device="cuda")
    tables = torch.arange(n * nb, dtype=torch.int32).reshape(n, nb).cuda()
    pool.paged_prefix_attention(q.cuda(), out, np.arange(n + 1, dtype=np.int32), np.full(n, ctx - 1, np.int32), tables, heads)
    got = out.cpu().double()
    pool.close()
    w = torch.softmax((K.double() * q.double()[:, :, None]).sum(3) / d ** 0.5, 2)[..., None]
    return got, (w * V.double()).sum(2), (w * V.double().abs()).sum(2)


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("drop", [0.3, 12.0, 24.0])
def test_single_token_weights_keep_32_bits(dtype, drop):
    """Four positions of weights 1 : 2^-drop : almost the same : 0 where the second and third have opposite V: the sum
    shows their difference, and with it every bit of the weights, above the rounding of the result."""
    tt = torch.float16 if dtype == "f16" else torch.bfloat16
    n, heads, d = 16, 32, 128
    g = torch.Generator().manual_seed(int(drop) + 3)
    q = (0.5 + torch.rand((n, heads, d), generator=g)).to(tt)
    K = torch.zeros((n, heads, 4, d), dtype=tt)
    ch = [5, 40, 77, 126]                                   # one channel in every 32: exact products, three additions
    K[:, :, 1, ch] = (-drop * np.log(2) * d ** 0.5 / 4 / q[:, :, ch].float()).to(tt)
    K[:, :, 2] = K[:, :, 1]
    K[:, :, 2, 5] = (K[:, :, 1, 5].view(torch.int16) + 1).view(tt)
    K[:, :, 3, ch] = (-200 * np.log(2) * d ** 0.5 / 4 / q[:, :, ch].float()).to(tt)
    V = torch.zeros((n, heads, 4, d), dtype=tt)
    big = (40000.0 if drop > 1 else 1.0) * (1 + torch.rand((n, heads, d), generator=g) / 2)
    V[:, :, 1], V[:, :, 2] = big.to(tt), -big.to(tt)
    got, want, size = _single_tokens(dtype, 4, q, K, V)
    # a weight: its exponent (a few roundings of a number of about drop) and its own two roundings; the sum: two additions
    rel = (4 + 8 * drop) * 2.0 ** -24
    bound = (2.0 ** -11 if dtype == "f16" else 2.0 ** -8) * want.abs() + rel * size + (2.0 ** -25 if dtype == "f16" else 0)
    worst = float(((got - want).abs() / bound).max())
    assert worst <= 1, worst


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("ctx", [20, 700])
def test_single_tokens_see_an_infinite_v_at_any_weight(dtype, ctx):
    """An infinite V makes its channel infinite as long as its weight is not zero in 32 bits, however small it is; the
    other channels and heads keep finite results."""
    tt = torch.float16 if dtype == "f16" else torch.bfloat16
    heads, d = 8, 128
    drops = [0.0, 20.0, 30.0, 40.0, 60.0, 100.0]            # the weight of position 7 in powers of two below the largest
    g = torch.Generator().manual_seed(5)
    q = torch.ones((len(drops), heads, d), dtype=tt)
    K = torch.zeros((len(drops), heads, ctx, d), dtype=tt)
    V = torch.randn((len(drops), heads, ctx, d), generator=g).to(tt)
    for i, drop in enumerate(drops):
        K[i, :, 7] = -drop * np.log(2) * d ** 0.5 / d
        V[i, 3, 7, 11], V[i, 5, 7, 100] = float("inf"), -float("inf")
    got, want, size = _single_tokens(dtype, ctx, q, K, V)
    assert torch.equal(torch.isinf(want), torch.isinf(got)) and int(torch.isinf(got).sum()) == 2 * len(drops)
    assert torch.equal(got[torch.isinf(got)], want[torch.isinf(want)])
    fin = ~torch.isinf(want)
    assert float(((got - want).abs() / (size + 1e-3))[fin].max()) < (2.0 ** -10 if dtype == "f16" else 2.0 ** -7)


def test_single_tokens_of_large_bfloat16_values_stay_finite():
    """V of up to 2^120: the weighted sum of 64 of them is below the largest 32-bit number, so the result is finite."""
    g = torch.Generator().manual_seed(6)
    q = torch.randn((3, 8, 128), generator=g).to(torch.bfloat16)
    K = torch.randn((3, 8, 64, 128), generator=g).to(torch.bfloat16)
    V = (torch.randn((3, 8, 64, 128), generator=g) * 2.0 ** 118).to(torch.bfloat16)
    got, want, size = _single_tokens("bf16", 64, q, K, V)
    assert bool(torch.isfinite(got).all()) and bool(((got - want).abs() <= 2.0 ** -7 * size).all())


@pytest.mark.parametrize("dtype,heads,kv", [("bf16", 32, 32), ("f16", 32, 8)])
def test_split_attention_of_two_streams_over_one_pool(dtype, heads, kv):
    """Two batches of single tokens over one pool, each on a stream of its own with nothing between them: the pieces of their
    contexts (both split) do not meet."""
    d, bt, n, ctx = 128, 16, 80, 1500
    tt = torch.float16 if dtype == "f16" else torch.bfloat16
    nb = (ctx + bt - 1) // bt
    g = torch.Generator(device="cuda").manual_seed(9)
    dev = torch.empty((2 * n * nb, 2 * bt * kv * d), dtype=tt, device="cuda").normal_(generator=g)
    pool = flpool.Pool(dtype, kv, d, 2 * n * nb, 0, block_tokens=bt, dev=dev)
    tables = torch.arange(2 * n * nb, dtype=torch.int32, device="cuda").reshape(2, n, nb)
    q = torch.randn((2, n, heads, d), generator=g, device="cuda").to(tt)
    cu, prefix = np.arange(n + 1, dtype=np.int32), np.full(n, ctx - 1, np.int32)
    run = lambda i, out, stream: pool.paged_prefix_attention(q[i], out, cu, prefix, tables[i], heads, stream=stream)
    want, got = torch.empty_like(q), torch.empty((6,) + q.shape, dtype=tt, device="cuda")
    for i in range(2):
        run(i, want[i], torch.cuda.current_stream())
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    for k in range(6):
        for i in range(2):
            run(i, got[k, i], streams[i])
    torch.cuda.synchronize()
    assert bool((got == want).all())
    pool.close()


def _lora_call(dtype, T, d_in, widths, adapters, ranks, seed, poison=None):
    """x, dense bases and LoRA pages of adapters with `ranks`, tokens drawn from `adapters` (-1: none); `poison`: an adapter
    whose B holds infinities and NaN.  Returns the tokens' adapters, the results, their reference in fp64 and the bound of
    an entry: its rounding, 32-bit sums of the dense product, v as value and remainder (2^-16 of it in bf16)."""
    tt = torch.float16 if dtype == "f16" else torch.bfloat16
    g = torch.Generator(device="cuda").manual_seed(seed)
    rnd = lambda shape, std: (torch.randn(shape, generator=g, device="cuda") * std).to(tt)
    n_ad, E = len(ranks), 2 * 16 * 8 * 128
    pages, tab, place = [], [], []
    for w in widths:
        pl = {k: np.zeros(n_ad, np.int32) for k in ("a_tab_off", "a_row_base", "b_tab_off", "b_row_base")}
        mats = []
        for a, r in enumerate(ranks):
            A, B = rnd((r, d_in), d_in ** -0.5), rnd((r, w), 0.3)
            if a == poison:
                B[0, ::3], B[r - 1, 1::3] = float("inf"), float("nan")
            for key, m in (("a", A), ("b", B)):
                rpb = E // m.shape[1]
                pl[key + "_tab_off"][a] = len(tab)
                for lo in range(0, r, rpb):
                    blk = torch.full((E,), float("nan"), dtype=tt, device="cuda")
                    part = m[lo:lo + rpb].reshape(-1)
                    blk[:part.numel()] = part
                    tab.append(len(pages))
                    pages.append(blk)
            mats.append((A, B))
        place.append((pl, mats))
    pool = flpool.Pool(dtype, 8, 128, len(pages), 0, block_tokens=16, dev=torch.stack(pages).contiguous())
    x, w = rnd((T, d_in), 1.0), [rnd((n, d_in), d_in ** -0.5) for n in widths]
    ta = torch.from_numpy(np.random.default_rng(seed).choice(np.asarray(adapters, np.int32), T)).cuda()
    rank = torch.tensor(ranks, dtype=torch.int32, device="cuda")
    scale = torch.linspace(0.5, 1.5, n_ad, device="cuda")
    y = [torch.full((T, n), float("nan"), dtype=tt, device="cuda") for n in widths]
    up = lambda pl: {k: torch.from_numpy(v).cuda() for k, v in pl.items()}
    projs = [dict(y=yi, d_out=n, w_base=wi, w_base_layout=1, **up(pl)) for yi, n, wi, (pl, _) in zip(y, widths, w, place)]
    pool.lora_apply_paged(x, ta, rank, scale, torch.tensor(tab, dtype=torch.int32, device="cuda"), projs, n_tokens=T, d_in=d_in,
                          n_adapters=n_ad, max_rank=max(ranks))
    want, bound = [], []
    for wi, (_, mats) in zip(w, place):
        r, m = x.double() @ wi.double().T, 2.0 ** -19 * x.double().abs() @ wi.double().abs().T
        for a, (A, B) in enumerate(mats):
            sel = ta == a
            v = float(scale[a]) * x[sel].double() @ A.double().T
            r[sel] += v @ B.double()
            m[sel] += 2.0 ** -15 * v.abs() @ B.double().abs()
        want.append(r)
        bound.append((2.0 ** -11 if dtype == "f16" else 2.0 ** -8) * r.abs() + m + 1e-7)
    torch.cuda.synchronize()
    pool.close()
    return ta, y, want, bound


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("T,widths", [(2100, (1024, 1024, 1024)),       # three outputs, 68 tiles of 256 x 128 each
                                      (2049, (2048,)), (4100, (4096,)),  # one output: few tiles and many
                                      (1500, (512,))])                   # outside the fused path
def test_an_adapter_s_infinities_stay_with_its_tokens(dtype, T, widths):
    """Adapters mixed token by token, one of them with infinities and NaN in its B: every other token's result is what
    it is without that adapter."""
    ta, y, want, bound = _lora_call(dtype, T, 512, widths, [-1, 0, 1, 2, 3], [16, 8, 64, 40], T, poison=1)
    ok = ta != 1
    for yi, wi, bi in zip(y, want, bound):
        assert bool(torch.isfinite(yi[ok]).all())
        assert not bool(torch.isfinite(yi[~ok]).all(1).any())
        assert bool(((yi[ok].double() - wi[ok]).abs() <= bi[ok]).all())


@pytest.mark.parametrize("T,d_in,widths,plan", [
    (1, 1024, (264, 72, 72), ("64x32", 1)), (1, 2048, (72,), ("64x32", 8)), (7, 2048, (264, 72, 72), ("64x32", 8)),
    (129, 1024, (2056, 4104, 4104), ("128x64", 1)), (33, 4096, (2056, 4104, 4104), ("128x64", 3)), (33, 11008, (2056,), ("128x64", 12)),
    (129, 1024, (4104, 4104, 4104), ("128x128", 1)), (300, 8192, (264, 72, 72), ("128x128", 16)),
    (257, 1024, (4104, 4104, 4104), ("256x128", 1)), (33, 8192, (2056, 264, 264), ("256x128", 16)), (33, 8192, (4104,), ("256x128", 12)),
    (641, 1024, (2056, 4104, 4104), ("256x256", 1)), (129, 8192, (2056, 4104, 4104), ("256x256", 4)), (1000, 8192, (4104,), ("256x256", 3)),
])
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_dense_products_with_adapters_on_every_tile_whole_and_in_slices(dtype, T, d_in, widths, plan):
    """Each tile with the whole contraction and with slices, with one output and three, remainders in tokens and features;
    a third of the tokens has no adapter and keeps the rounded product, the others add their branch to the unrounded one."""
    assert dense_plan(T, d_in, widths, room=60 << 20) == plan
    ta, y, want, bound = _lora_call(dtype, T, d_in, widths, [-1, 0, 2], [8, 16, 64], T)
    for yi, wi, bi in zip(y, want, bound):
        assert bool(((yi.double() - wi).abs() <= bi).all())


@pytest.mark.parametrize("T,d_in,widths,room,plan", [
    (1100, 11008, (4096,), 60 << 20, ("256x256", 3)),      # slices added by a kernel that keeps the unrounded sum, sorted tokens
    (1100, 4096, (1032, 72), 60 << 20, ("256x128", 4)),    # the same in front of the vector kernels, every token alone
    (1000, 512, (16392, 8200), 0, ("256x256", 1)),         # 98 MB of sums: vector kernels, tokens of an adapter in fours
])
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_dense_products_with_adapters_outside_the_small_batch_kernels(dtype, T, d_in, widths, room, plan):
    """16-bit batches with dense bases whose branches neither the kernels for small batches nor the fused product take."""
    assert dense_plan(T, d_in, widths, room=room) == plan
    ta, y, want, bound = _lora_call(dtype, T, d_in, widths, [-1, 0, 1, 2, 3], [8, 16, 64, 33], T)
    for yi, wi, bi in zip(y, want, bound):
        assert bool(((yi.double() - wi).abs() <= bi).all())


@pytest.mark.parametrize("T,d_in,widths,ld_x,plan", [
    (641, 1024, (2056, 4104, 4104), (1 << 23) + 64, ("256x256", 1)),        # 256 rows span a little more than 4 GiB
    (300, 8192, (264, 72, 72), (1 << 24) + 64, ("128x128", 16)),            # 128 rows do
    (2100, 512, (1024, 1024, 1024), (1 << 23) + 64, ("256x128", 1)),        # as many tokens as the fused path takes
])
def test_dense_products_of_rows_far_apart(T, d_in, widths, ld_x, plan):
    """Token rows of x so far apart that a tile's rows do not all lie within 32-bit byte offsets of its first one."""
    assert dense_plan(T, d_in, widths, large_only=T >= 2048, room=60 << 20) == plan
    g = torch.Generator(device="cuda").manual_seed(T)
    store = torch.empty(((T - 1) * ld_x + d_in,), dtype=torch.float16, device="cuda")
    x = store.as_strided((T, d_in), (ld_x, 1))
    x.copy_(torch.randn((T, d_in), generator=g, device="cuda"))
    w = [(torch.randn((n, d_in), generator=g, device="cuda") / d_in ** 0.5).half() for n in widths]
    pool = flpool.Pool("f16", 8, 128, 2, 0, block_tokens=16)
    z = torch.zeros(1, dtype=torch.int32, device="cuda")
    y = [torch.full((T, n), float("nan"), dtype=torch.float16, device="cuda") for n in widths]
    projs = [dict(y=yi, d_out=n, w_base=wi, w_base_layout=1, a_tab_off=z, a_row_base=z, b_tab_off=z, b_row_base=z)
             for yi, n, wi in zip(y, widths, w)]
    none = torch.full((T,), -1, dtype=torch.int32, device="cuda")
    pool.lora_apply_paged(store, none, z, torch.ones(1, device="cuda"), z, projs, n_tokens=T, d_in=d_in, n_adapters=1,
                          max_rank=8, ld_x=ld_x)
    for yi, wi in zip(y, w):
        want = x.double() @ wi.double().T
        bound = 2.0 ** -11 * want.abs() + 2.0 ** -19 * (x.double().abs() @ wi.double().abs().T) + 1e-7
        assert bool(((yi.double() - want).abs() <= bound).all())
    pool.close()


@pytest.mark.parametrize("dtype,T,d_in,widths,counts,ranks", [
    ("bf16", 96, 64, (8, 136), (1, 4, 5, 16, 17, 33), (16, 1, 15, 8, 16, 7)),           # one chunk of d_in, ragged columns
    ("f16", 96, 704, (128, 264, 8), (1, 4, 5, 16, 17, 33), (17, 32, 1, 31, 16, 32)),    # two tiles of ranks, 16 or fewer among them
    ("bf16", 1024, 4096, (136,), (1, 3, 64, 500, 19, 437), (33, 64, 48, 1, 16, 49)),    # four tiles, the largest batch
    ("f16", 3, 8192, (1032,), (3,), (64,)),                                             # sixteen slices of d_in
    ("bf16", 96, 288, (8, 136), (1, 4, 5, 16, 17, 33), (16, 1, 15, 8, 64, 7)),          # d_in no multiple of 64: the vector kernels,
    ("f16", 1000, 288, (128, 264, 1032), (1, 3, 64, 500, 19, 400), (33, 64, 48, 2, 16, 32)),    # tokens of an adapter in fours
    ("f16", 1100, 704, (72, 264), (1, 3, 64, 500, 19, 437), (33, 64, 48, 2, 16, 32)),   # too long for that: every token alone
    ("f16", 512, 1024, (264, 8, 1160), (8, 9, 7, 200, 24, 25), (64, 33, 48, 64, 17, 49)),   # 64 ranks by two waves, groups of 8 and 9
    ("bf16", 513, 1024, (8, 1160, 264), (8, 9, 7, 200, 24, 25), (64, 33, 48, 64, 32, 49)),  # and by one
])
def test_lora_of_small_batches_in_groups_of_every_size(dtype, T, d_in, widths, counts, ranks):
    """Adapters with 1 to 500 tokens, mixed over the batch (a group takes up to sixteen of one adapter, up to four go to
    another form of the product), ranks at the edges of a rank tile, columns at those of a chunk; the rest of the tokens has no
    adapter.  v keeps 32 bits: a large base-free delta is compared to within its rounding and 32-bit sums."""
    tt = torch.float16 if dtype == "f16" else torch.bfloat16
    g = torch.Generator(device="cuda").manual_seed(T + d_in)
    rnd = lambda shape, std: (torch.randn(shape, generator=g, device="cuda") * std).to(tt)
    n_ad, E = len(ranks), 2 * 16 * 8 * 128
    ta = np.full(T, -1, np.int32)
    ta[np.random.default_rng(T).permutation(T)[:sum(counts)]] = np.repeat(np.arange(n_ad), counts)
    pages, tab = [], []

    def put(m):
        off, rpb = len(tab), E // m.shape[1]
        for lo in range(0, len(m), rpb):
            blk = torch.full((E,), float("nan"), dtype=tt, device="cuda")
            part = m[lo:lo + rpb].reshape(-1)
            blk[:part.numel()] = part
            tab.append(len(pages))
            pages.append(blk)
        return off

    i32 = lambda v: torch.tensor(v, dtype=torch.int32, device="cuda")
    mats = [[(rnd((r, d_in), d_in ** -0.5), rnd((r, w), 1.0)) for r in ranks] for w in widths]
    projs = [dict(d_out=w, a_tab_off=i32([put(a) for a, _ in m]), b_tab_off=i32([put(b) for _, b in m]), a_row_base=i32([0] * n_ad),
                  b_row_base=i32([0] * n_ad)) for w, m in zip(widths, mats)]
    x, scale = rnd((T, d_in), 1.0), torch.linspace(0.5, 1.5, n_ad, device="cuda")
    y0 = [rnd((T, w), 2.0 ** -6) for w in widths]
    pool = flpool.Pool(dtype, 8, 128, len(pages), 0, block_tokens=16, dev=torch.stack(pages).contiguous())
    y = [t.clone() for t in y0]
    pool.lora_apply_paged(x, torch.from_numpy(ta).cuda(), i32(ranks), scale, i32(tab), [dict(p, y=t) for p, t in zip(projs, y)],
                          n_tokens=T, d_in=d_in, n_adapters=n_ad, max_rank=max(ranks))
    for yi, y0i, m in zip(y, y0, mats):
        want, size = y0i.double(), y0i.double().abs()
        for a, (A, B) in enumerate(m):
            sel = torch.from_numpy(ta == a).cuda()
            v = float(scale[a]) * x[sel].double() @ A.double().T
            vs = float(scale[a]) * x[sel].double().abs() @ A.double().abs().T
            want[sel] += v @ B.double()
            size[sel] += vs @ B.double().abs()
        none = torch.from_numpy(ta < 0).cuda()
        assert torch.equal(yi[none], y0i[none])
        # the rounding of the result, and chains of at most 64 additions in 32 bits of terms that add up to `size`
        bound = (2.0 ** -11 if dtype == "f16" else 2.0 ** -8) * want.abs() + 64 * 2.0 ** -24 * size + 1e-7
        assert bool(((yi.double() - want).abs() <= bound).all())
    pool.close()


@pytest.mark.parametrize("tokens_each", [3, 16])
@pytest.mark.parametrize("T,d_in,rank", [(96, 4096, 64), (240, 8192, 64), (240, 5120, 40), (960, 4096, 64)])
def test_lora_of_small_batches_sums_in_short_chains(T, d_in, rank, tokens_each):
    """The branch's own error, below the 16-bit rounding of y: a first call over y = 0 leaves y1 = round(s delta), a second one over
    -y1 leaves s delta - y1, which 16 bits hold to 2^-23 of delta.  64 products of equal size added one after the other in 32
    bits are off by 1.9e-7 of the sum (each addition rounds a partial sum of k of them, sqrt(k) in size, by 2^-24 / sqrt(3):
    sqrt(1/2 64) 3.4e-8); in tiles of 16 that are then added it is 1.1e-7.  With the shrink step's sums and the rounding of the
    second result (0.3e-7 to 0.9e-7 each) the whole is 1.5e-7, and was 2.1e-7 with one chain."""
    n_ad, d_out, E = T // tokens_each, 2048, 2 * 16 * 8 * 128
    g = torch.Generator(device="cuda").manual_seed(T + d_in + rank)
    rnd = lambda shape, std: (torch.randn(shape, generator=g, device="cuda") * std).half()
    A, B, x = rnd((rank, d_in), d_in ** -0.5), rnd((rank, d_out), rank ** -0.5), rnd((T, d_in), 1.0)
    rows_a, rows_b = E // d_in, E // d_out               # page rows per block; every adapter has the same pages
    pages = [torch.zeros(E, dtype=torch.float16, device="cuda") for _ in range(-(-rank // rows_a) - (-rank // rows_b))]
    for m, rpb, first in ((A, rows_a, 0), (B, rows_b, -(-rank // rows_a))):
        for k, lo in enumerate(range(0, rank, rpb)):
            part = m[lo:lo + rpb].reshape(-1)
            pages[first + k][:part.numel()] = part
    pool = flpool.Pool("f16", 8, 128, len(pages), 0, block_tokens=16, dev=torch.stack(pages).contiguous())
    i32 = lambda v: torch.as_tensor(v, dtype=torch.int32, device="cuda")
    z, y = i32(np.zeros(n_ad)), torch.zeros((T, d_out), dtype=torch.float16, device="cuda")
    proj = dict(y=y, d_out=d_out, a_tab_off=z, a_row_base=z, b_tab_off=z + -(-rank // rows_a), b_row_base=z)
    ta = i32(np.random.default_rng(T).permutation(np.repeat(np.arange(n_ad), tokens_each)))
    call = lambda: pool.lora_apply_paged(x, ta, z + rank, torch.ones(n_ad, device="cuda"), i32(np.arange(len(pages))), [proj],
                                         n_tokens=T, d_in=d_in, n_adapters=n_ad, max_rank=rank)
    call()
    y.neg_()
    first = y.double()
    call()
    delta = (x.double() @ A.double().T) @ B.double()
    err = float((y.double() - (first + delta)).norm() / delta.norm())
    assert err < 1.8e-7, err
    pool.close()


@pytest.mark.parametrize("T,widths,plan", [(2050, (1088, 320), ("256x128", 1)), (2177, (4032,), ("256x256", 1)),
                                           (4100, (1088, 1088, 320), ("256x256", 1))])
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_branches_inside_the_product_with_many_adapters_and_remainders(dtype, T, widths, plan):
    """Thirteen adapters mixed token by token: a tile's adapters take two rounds of the epilogue's tables, in the last, partly
    filled tile as well (of 2, 129 and 4 tokens); widths that are no multiple of the tile."""
    assert dense_plan(T, 512, widths, large_only=True) == plan
    ranks = [8, 16, 64, 40, 1, 33, 24, 8, 16, 64, 32, 48, 8]
    ta, y, want, bound = _lora_call(dtype, T, 512, widths, list(range(-1, 13)), ranks, T)
    for yi, wi, bi in zip(y, want, bound):
        assert bool(((yi.double() - wi).abs() <= bi).all())


@pytest.mark.parametrize("T", [1, 31, 33, 127, 129, 255, 257, 513, 1025, 2049])
@pytest.mark.parametrize("dtype,d_in,widths", [
    ("f16", 64, (64, 32, 40)),                 # one step of the contraction, widths that no tile divides
    ("bf16", 1088, (264, 136, 72)),            # three outputs in one launch, remainders in the last tiles
    ("f16", 4096, (4096, 1032)),               # enough contraction for slices at small batches, whole tiles at large ones
])
def test_dense_products_at_the_edges_of_their_tiles(dtype, d_in, widths, T):
    """Tokens without an adapter keep the dense product, over batch sizes around every tile's (the first two sets of widths
    stay with the smallest tile at all of them, the third has slices at small batches and large tiles at large ones)."""
    tt = torch.float16 if dtype == "f16" else torch.bfloat16
    g = torch.Generator().manual_seed(T + d_in)
    x = torch.randn((T, d_in), generator=g).to(tt)
    w = [(torch.randn((n, d_in), generator=g) / d_in ** 0.5).to(tt) for n in widths]
    pool = flpool.Pool(dtype, 4, 128, 4, 0, dev=torch.zeros((4, 2 * 16 * 4 * 128), dtype=tt, device="cuda"))
    zero = torch.zeros(1, dtype=torch.int32, device="cuda")
    dx, dw = x.cuda(), [m.cuda() for m in w]
    y = [torch.full((T, n), float("nan"), dtype=tt, device="cuda") for n in widths]
    projs = [dict(y=yi, d_out=n, w_base=wi, w_base_layout=1, a_tab_off=zero, a_row_base=zero, b_tab_off=zero, b_row_base=zero)
             for yi, n, wi in zip(y, widths, dw)]
    none = torch.full((T,), -1, dtype=torch.int32, device="cuda")
    rank, scale = torch.full((1,), 8, dtype=torch.int32, device="cuda"), torch.ones(1, device="cuda")
    pool.lora_apply_paged(dx, none, rank, scale, zero, projs, n_tokens=T, d_in=d_in, n_adapters=1, max_rank=8)
    half_ulp = 2.0 ** -11 if dtype == "f16" else 2.0 ** -8
    for yi, wi in zip(y, dw):
        want = dx.double() @ wi.double().T
        # the result's rounding, and d_in additions in 32 bits
        bound = half_ulp * want.abs() + d_in * 2.0 ** -24 * (dx.double().abs() @ wi.double().abs().T) + 1e-7
        assert bool(((yi.double() - want).abs() <= bound).all())
