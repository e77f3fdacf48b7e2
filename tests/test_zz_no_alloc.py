"""flp_lora_apply_paged_static (the entry point that allocates nothing: its intermediates live in a fixed device
array) against flp_lora_apply_paged, through the C ABI: the two run the same kernels on the same inputs, so their
outputs must agree bit for bit (and both within tolerance of the oracle).  Two calls in a row on the shared array,
the second with a smaller input, then a third on another pool; a batch that does not fit is refused."""
import numpy as np
import pytest

import oracle
from helpers import TOL, GpuStep, close, resident_pool, to_dev
from paper_2505_03756_amd import flpool
from paper_2505_03756_amd import workload as wl

pytestmark = pytest.mark.gpu


def _cfg(dtype, **kw):
    base = dict(name="noalloc_" + dtype, dtype=dtype, hidden=512, n_q_heads=4, n_kv_heads=4, head_dim=128,
                n_dev_blocks=1500, n_host_blocks=4, n_adapters=6, ranks=(8, 16, 32), projections=("q", "k", "v", "o"),
                n_seqs=7, prefix_range=(0, 0), new_range=(1, 70), swap_in_frac=0.0, seed=501)
    base.update(kw)
    return wl.LayerConfig(**base)


def _both(step, names, w_base=None):
    cfg = step.cfg
    dev0 = resident_pool(step)
    g = GpuStep(step, dev0, np.zeros((4, cfg.block_elems), dev0.dtype))
    wb = {n: to_dev(w_base[n]) for n in names} if w_base else None
    want = g.lora(names, w_base=wb)
    got = g.lora(names, w_base=wb, static=True)
    rtol, atol = TOL[cfg.dtype]
    for n in names:
        assert np.array_equal(got[n], want[n]), "%s: static and allocating entry points differ" % n
        pr = step.proj[n]
        ref = oracle.lora_apply(dev0, cfg.dtype, step.acts["x"], step.token_adapter, step.rank, step.scale,
                                pr.a_tab_off, pr.a_row_base, pr.b_tab_off, pr.b_row_base, step.lora_tables, pr.d_out,
                                y_in=None if w_base else step.acts["base_" + n], w_base=w_base[n] if w_base else None)
        ok, worst, nbad = close(wl.dequantize(got[n], cfg.dtype), ref, rtol, atol)
        assert ok, "%s: max err %g (%d bad)" % (n, worst, nbad)
        if not w_base:
            base = wl.dequantize(step.acts["base_" + n], cfg.dtype)
            assert np.abs(ref - base).max() > 10 * atol, "the case carries no delta"
    g.pool.close()


def test_static_entry_point_matches_on_two_calls_in_a_row():
    assert flpool.static_scratch_bytes() == 64 << 20
    # 1) a prefill batch on the 32-token tiles with a dense base that is small enough to fit (large-batch GEMM with
    #    the LoRA branch inside: transposed base matrix, inverse permutation and segment lists in the array)
    big = wl.make_step(_cfg("f16", n_q_heads=18, n_kv_heads=18, n_seqs=24, new_range=(110, 160), ranks=(8, 16),
                            seed=502))
    assert big.n_tokens >= 2048
    rng = np.random.default_rng(5)
    W = {n: wl.quantize((rng.standard_normal((512, big.proj[n].d_out)) / np.sqrt(512)).astype(np.float32), "f16")
         for n in ("q", "k", "v")}
    _both(big, ["q", "k", "v"], w_base=W)
    # 2) right after it a smaller one without a base: the array still holds the first call's bits
    mid = wl.make_step(_cfg("f16", n_seqs=30, new_range=(40, 90), ranks=(16, 32), seed=503))
    assert 1024 <= mid.n_tokens < big.n_tokens
    _both(mid, ["q", "k", "v"])
    _both(mid, ["o"])
    # 3) and a decode batch (the kernels for up to 1024 tokens, mixed ranks, bf16) on yet another pool
    small = wl.make_step(_cfg("bf16", n_seqs=97, new_range=(1, 1), decode_frac=1.0, n_adapters=20,
                              ranks=(8, 16, 32, 64), seed=504))
    assert small.n_tokens == 97
    _both(small, ["q", "k", "v"])


def test_static_entry_point_refuses_what_does_not_fit():
    """A dense base at 20 000 tokens needs the unrounded product beside y (hundreds of MB): refused with FLP_ENOSPC
    before anything runs; y is untouched."""
    import torch
    cfg = _cfg("f16", hidden=1024, n_q_heads=8, n_kv_heads=8)
    pool = flpool.Pool(cfg.dtype, cfg.n_kv_heads, cfg.head_dim, 64, 4)
    T = 1000                                         # small-batch GEMM: keeps 4 * T * d_out bytes per projection
    x = torch.zeros((T, 16384), dtype=torch.int16, device="cuda")
    y = torch.full((T, 16384), 7, dtype=torch.int16, device="cuda")
    w = torch.zeros((16384, 16384), dtype=torch.int16, device="cuda")
    z = torch.zeros(4, dtype=torch.int32, device="cuda")
    proj = dict(y=y, d_out=16384, w_base=w, a_tab_off=z, a_row_base=z, b_tab_off=z, b_row_base=z)
    with pytest.raises(flpool.FlpError) as e:
        pool.lora_apply_paged(x, torch.full((T,), -1, dtype=torch.int32, device="cuda"), z,
                              torch.zeros(4, device="cuda"), z, [proj], n_tokens=T, d_in=16384, n_adapters=4,
                              max_rank=8, static=True)
    assert e.value.code == flpool.FLP_ENOSPC and "fixed buffer" in str(e.value)
    torch.cuda.synchronize()
    assert bool((y == 7).all())
    pool.close()


SLICED = [   # tokens, d_in, widths, max_rank, and how many slices a layer's larger room would give
    (1747, 13824, (5120,), 8, 3),          # one slice in 64 MiB
    (257, 22016, (8192,), 8, 8),           # fewer than eight
    (347, 16384, (12072, 12024), 16, 3),   # two slices would fill the array to the last byte, before every product is rounded up
    (33, 4096, (4096, 4096, 4096), 16, 4),
    (499, 4096, (4096, 4096, 4096), 16, 1),
]


@pytest.mark.parametrize("T,d_in,widths,max_rank,layer_slices", SLICED)
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_static_entry_point_sums_dense_products_in_the_same_order(dtype, T, d_in, widths, max_rank, layer_slices):
    """Dense bases outside the fused path: both entry points cut the contraction into the same slices, so the results
    agree bit for bit also where the fixed array holds fewer slices than the pool's workspace would."""
    import torch
    from helpers import dense_plan
    assert dense_plan(T, d_in, widths)[1] == layer_slices
    tt = torch.float16 if dtype == "f16" else torch.bfloat16
    pool = flpool.Pool(dtype, 8, 128, 2, 0, block_tokens=16)
    g = torch.Generator(device="cuda").manual_seed(T)
    x = torch.randn((T, d_in), generator=g, device="cuda").to(tt)
    w = [(torch.randn((n, d_in), generator=g, device="cuda") / d_in ** 0.5).to(tt) for n in widths]
    z = torch.zeros(1, dtype=torch.int32, device="cuda")
    none = torch.full((T,), -1, dtype=torch.int32, device="cuda")
    got = []
    for static in (False, True):
        y = [torch.full((T, n), float("nan"), dtype=tt, device="cuda") for n in widths]
        projs = [dict(y=yi, d_out=n, w_base=wi, w_base_layout=1, a_tab_off=z, a_row_base=z, b_tab_off=z, b_row_base=z)
                 for yi, n, wi in zip(y, widths, w)]
        pool.lora_apply_paged(x, none, z, torch.ones(1, device="cuda"), z, projs, n_tokens=T, d_in=d_in, n_adapters=1,
                              max_rank=max_rank, static=static)
        got.append(y)
    torch.cuda.synchronize()
    for a, b, wi in zip(got[0], got[1], w):
        assert torch.equal(a, b), "static and allocating entry points differ"
        want = x.float() @ wi.float().T
        # one rounding of a result of standard deviation 1, and two fp32 sums in different orders
        assert float((b.float() - want).abs().max()) < (2.0 ** -8 if dtype == "f16" else 2.0 ** -5)
    pool.close()


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_slices_at_the_edge_of_the_fixed_array(dtype):
    """Beside its other intermediates the fixed array has room for two slices of 347 x 24096 sums to the last byte, and each product's are
    rounded up to 256: the call has to take one slice.  With eight columns less it takes two (the last bits show it), with eight
    less and a segment list of 2048 adapters beside them one again."""
    import torch
    T, d_in, n1, n2 = 347, 16384, 12072, 12024
    up = lambda n: (n + 255) & ~255
    # slices of v (4, of 16 ranks), a record of 112 bytes per token, the segment list of one adapter, the permutation
    rest = up(4 * T * 2 * 16 * 4) + up(112 * T) + up(9 * 4) + up(4 * T)
    assert 2 * T * (n1 + n2) * 4 == flpool.static_scratch_bytes() - rest
    assert up(2 * T * n1 * 4) + up(2 * T * n2 * 4) > flpool.static_scratch_bytes() - rest
    tt = torch.float16 if dtype == "f16" else torch.bfloat16
    pool = flpool.Pool(dtype, 8, 128, 2, 0, block_tokens=16)
    g = torch.Generator(device="cuda").manual_seed(T)
    x = torch.randn((T, d_in), generator=g, device="cuda").to(tt)
    w = [(torch.randn((n, d_in), generator=g, device="cuda") / d_in ** 0.5).to(tt) for n in (n1, n2)]
    none = torch.full((T,), -1, dtype=torch.int32, device="cuda")

    def call(widths, n_adapters):
        z = torch.zeros(n_adapters, dtype=torch.int32, device="cuda")
        got = []
        for static in (False, True):
            y = [torch.full((T, n), float("nan"), dtype=tt, device="cuda") for n in widths]
            projs = [dict(y=yi, d_out=n, w_base=wi, w_base_layout=1, a_tab_off=z, a_row_base=z, b_tab_off=z, b_row_base=z)
                     for yi, n, wi in zip(y, widths, w)]
            pool.lora_apply_paged(x, none, z, torch.ones(n_adapters, device="cuda"), z, projs, n_tokens=T, d_in=d_in,
                                  n_adapters=n_adapters, max_rank=16, static=static)
            got.append(torch.cat([y[0], y[1][:, :n2 - 8]], 1))
        assert torch.equal(got[0], got[1]), "static and allocating entry points differ"
        return got[1]

    edge, two, one = call((n1, n2), 1), call((n1, n2 - 8), 1), call((n1, n2 - 8), 2048)
    assert torch.equal(edge, one)
    assert not torch.equal(edge, two)
    pool.close()
