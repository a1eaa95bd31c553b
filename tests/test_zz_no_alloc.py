"""The entry point that allocates nothing (bs_attention_noalloc) against bs_attention: same kernels,
same descriptor, so the outputs must be equal bit for bit; two calls in a row on one context, the
second with a smaller batch (the scratch array keeps the first call's contents), then a batch beyond
the stated limits, which must be refused before anything is enqueued."""
import numpy as np
import pytest

from paper_2411_16102_amd import workloads as W

pytestmark = pytest.mark.gpu


def test_noalloc_attention_matches_the_allocating_entry_point(lib):
    import torch
    shape = W.LayerShape(512, 8, 2, 128, 256)
    layer = lib.Layer(shape, device=0)
    layer.set_chunk_pages(4)
    for seed, (n_pre, n_dec, ctx) in enumerate([(4, 48, 900), (2, 9, 200)]):
        batch = W.batch_random(40 + seed, n_prefill=n_pre, n_decode=n_dec, max_q=120, max_ctx=ctx, n_roots=3)
        tens = W.make_tensors(shape, batch, seed)
        rng = np.random.default_rng(seed)
        q = W.round_to_bf16(rng.standard_normal((batch.n_rows, shape.n_q_heads * shape.head_dim), dtype=np.float32))
        tq = torch.from_numpy(q).cuda().to(torch.bfloat16)
        pool = layer.pack_pool(tens.k_pool, tens.v_pool)
        ref = layer.attention(batch, tq, pool, batch.n_pages)
        out = torch.zeros_like(tq)
        torch.cuda.synchronize()
        free_before = torch.cuda.mem_get_info()[0]   # the driver's figure: sees the library's own allocations too
        layer.attention_noalloc(batch, tq, pool, batch.n_pages, out)
        torch.cuda.synchronize()
        assert torch.cuda.mem_get_info()[0] == free_before
        assert torch.equal(out, ref), "call %d differs from bs_attention" % seed
        assert bool(torch.isfinite(out.float()).all())


@pytest.mark.parametrize("members,prefix_pages,tail,loose", [(400, 100, 1000, 300), (50, 256, 20, 3), (400, 8, 100, 300)])
def test_noalloc_attention_matches_on_default_chunks(lib, members, prefix_pages, tail, loose):
    # wide nodes in a step that is large enough for the longest chunks, one whose short chunks the scratch array
    # would not hold, and one of many short contexts
    import torch
    shape = W.LayerShape(512, 32, 8, 128, 256) if members < 300 else W.LayerShape(512, 8, 2, 64, 256)
    layer = lib.Layer(shape, device=0)
    seqs = [(1, 16 * prefix_pages + tail + i, 0) for i in range(members)] + [(1, tail + 5 * i, -1) for i in range(loose)]
    batch = W.assemble_batch(16, seqs, 0, [(-1, prefix_pages)], np.random.default_rng(members))
    gen = torch.Generator(device="cuda").manual_seed(members)
    q = torch.randn((batch.n_rows, shape.n_q_heads * shape.head_dim), generator=gen, device="cuda").to(torch.bfloat16)
    pool = torch.randn(batch.n_pages * (layer.page_bytes() // 2), generator=gen, device="cuda").to(torch.bfloat16)
    ref = layer.attention(batch, q, pool, batch.n_pages)
    out = layer.attention_noalloc(batch, q, pool, batch.n_pages, torch.zeros_like(q))
    assert torch.equal(out, ref) and bool(torch.isfinite(out.float()).all())


def test_noalloc_attention_refuses_what_does_not_fit(lib):
    import torch
    # 8B heads: one partial state is 32 x 130 floats = 16.6 KB, so 15 MiB hold 945 of them; 1200 decode
    # sequences need 1200
    shape = W.LayerShape(512, 32, 8, 128, 256)
    layer = lib.Layer(shape, device=0)
    batch = W.batch_decode_only(1200, 40, seed=1)
    tens = W.make_tensors(shape, batch, 1)
    pool = layer.pack_pool(tens.k_pool, tens.v_pool)
    q = torch.zeros((batch.n_rows, shape.n_q_heads * shape.head_dim), dtype=torch.bfloat16, device="cuda")
    out = torch.full_like(q, 3.0)
    with pytest.raises(lib.BlendStepError) as ei:
        layer.attention_noalloc(batch, q, pool, batch.n_pages, out)
    assert ei.value.code == -1 and "exceed the limit" in str(ei.value)
    torch.cuda.synchronize()
    assert bool((out == 3.0).all())
    # the allocating entry point takes the same batch
    assert bool(torch.isfinite(layer.attention(batch, q, pool, batch.n_pages).float()).all())


def test_captured_calls_replay_behind_other_calls(lib):
    # a captured call of either kind reads its own descriptor with every replay, whatever was called since: calls that
    # turn to both halves of the staging buffer again, and one whose descriptor takes a larger buffer
    import torch
    shape = W.LayerShape(256, 8, 2, 64, 256)
    layer = lib.Layer(shape, device=0)
    rng = np.random.default_rng(5)
    mine = W.batch_random(61, n_prefill=3, n_decode=30, max_q=90, max_ctx=500, n_roots=2)
    others = [W.assemble_batch(16, [(1, 16 * pages + 5 + i % 40, 0) for i in range(n)], 0, [(-1, pages)], rng)
              for n, pages in ((900, 333), (900, 333), (900, 333), (900, 333), (700, 1000), (20, 9))]
    assert max(4 * len(b.page_ids) for b in others) > 2 << 20 and 4 * len(others[0].page_ids) > 1 << 20
    pages = max(b.n_pages for b in others + [mine])
    gen = torch.Generator(device="cuda").manual_seed(2)
    pool = torch.randn(pages * (layer.page_bytes() // 2), generator=gen, device="cuda").to(torch.bfloat16)
    qs = [torch.randn((b.n_rows, 512), generator=gen, device="cuda").to(torch.bfloat16) for b in others + [mine]]
    dev = layer.upload(W.make_tensors(shape, mine, 3), mine)
    # every workspace has its size, every kernel has run
    want_o = layer.attention(mine, qs[-1], pool, pages)
    want_y = layer.blend_step(dev, mine)
    for b, q in zip(others, qs):
        layer.attention(b, q, pool, pages)
    fresh = lib.Layer(shape, device=0)   # its staging buffer has not grown yet, and its workspace is not captured
    o, y = torch.zeros_like(want_o), torch.zeros_like(want_y)
    torch.cuda.synchronize()
    one, two = torch.cuda.CUDAGraph(), torch.cuda.CUDAGraph()
    with torch.cuda.graph(one):
        fresh.attention_noalloc(mine, qs[-1], pool, pages, o)
    with torch.cuda.graph(two):
        layer.blend_step(dev, mine, y=y)
    for i in range(len(others) + 1):
        o.zero_()
        y.zero_()
        one.replay()
        two.replay()
        torch.cuda.synchronize()
        assert torch.equal(o, want_o), "attention, replay %d" % i
        assert torch.equal(y, want_y), "step, replay %d" % i
        if i < len(others):
            for l in (layer, fresh):
                l.attention(others[i], qs[i], pool, pages)
