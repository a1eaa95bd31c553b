"""Parity of the HIP path with the CPU oracle, through the C ABI, at sizes the
oracle finishes in seconds (several tiles and ragged tails included).

Tolerances: the one rule of tests/parity_rule.py (max relative error 2e-2 over a tensor; mean
absolute error against the exact oracle rounded to bfloat16 at most 1e-3, or 1.25 times the error
that bfloat16 storage alone causes at that shape where that is larger).  Integer work (page and
slot of every appended row, which pool elements change) is compared exactly.
"""
import numpy as np
import pytest

from oracle import layer as O
from paper_2411_16102_amd import workloads as W
from parity_rule import MAE, MAXREL, check, errs

pytestmark = pytest.mark.gpu


def to_np(t):
    return t.float().cpu().numpy().astype(np.float64)


def run_step(lib, shape, batch, tens, flags=0, tiles=0):
    import torch
    layer = lib.Layer(shape, device=0)
    layer.set_gemm_tiles(tiles)
    dev = layer.upload(tens, batch)
    y = layer.blend_step(dev, batch, flags=flags)
    torch.cuda.synchronize()
    k, v = layer.unpack_pool(dev.kv_pool, dev.n_pages)
    return to_np(y), to_np(k), to_np(v), layer


def check_step(lib, shape, batch, tens, flags=0, tiles=0):
    ref = O.layer_step(shape, tens, batch)
    diag = O.layer_step(shape, tens, batch, storage="bf16")
    y, k, v, layer = run_step(lib, shape, batch, tens, flags, tiles)
    check(y, ref["y"], diag["y"], "rows=%d" % batch.n_rows)
    # KV append: exactly the destination slots change, and they hold k, v of the rows
    k0 = W.bf16_bits_to_f32(tens.k_pool).astype(np.float64)
    v0 = W.bf16_bits_to_f32(tens.v_pool).astype(np.float64)
    written = np.zeros(k0.shape[:2], dtype=bool)
    written[ref["dest"][:, 0], ref["dest"][:, 1]] = True
    assert np.array_equal(k[~written], k0[~written]), "a slot outside the append destinations changed (K)"
    assert np.array_equal(v[~written], v0[~written]), "a slot outside the append destinations changed (V)"
    kn = k[ref["dest"][:, 0], ref["dest"][:, 1]]
    vn = v[ref["dest"][:, 0], ref["dest"][:, 1]]
    check(kn, ref["k_new"], diag["k_new"], "appended keys")
    check(vn, ref["v_new"], diag["v_new"], "appended values")
    pg, sl = layer.resolve_rows(batch)
    assert np.array_equal(pg, ref["dest"][:, 0]) and np.array_equal(sl, ref["dest"][:, 1])
    return y, ref


# ---------------------------------------------------------------------------
# stand-alone operators
# ---------------------------------------------------------------------------
@pytest.mark.parametrize("m,n,k", [(136, 512, 256), (300, 264, 688), (1, 8, 8), (1030, 1544, 520), (2048, 1024, 512),
                                   # at most 256 / 128 rows and a row of tiles that fills the chip: the deep weight ring
                                   (200, 16512, 520), (256, 16384, 192), (100, 33000, 328), (128, 32768, 1024),
                                   # the few-row kernel: one and two blocks of rows and of columns, several items per
                                   # workgroup, a partial last k-tile, eight and more k-tiles per wavefront
                                   (7, 520, 1032), (16, 4104, 4096), (17, 264, 8), (33, 2056, 2048), (64, 520, 4096), (256, 512, 256),
                                   # 64x128 and 128x128 tiles on the deep ring, begun at shifted k-tiles and at the first
                                   (50, 9000, 2048), (64, 9000, 1000), (100, 9000, 2048), (65, 9000, 1000)])
def test_gemm_nt(lib, m, n, k):
    import torch
    rng = np.random.default_rng(m + n + k)
    a = W.round_to_bf16(rng.standard_normal((m, k), dtype=np.float32))
    b = W.round_to_bf16(rng.standard_normal((n, k), dtype=np.float32) * 0.05)
    layer = lib.Layer(W.TINY, device=0)
    ta = torch.from_numpy(a).cuda().to(torch.bfloat16)
    tb = torch.from_numpy(b).cuda().to(torch.bfloat16)
    c = to_np(layer.gemm_nt(ta, tb))
    ref = a.astype(np.float64) @ b.astype(np.float64).T
    maxrel, mae = errs(c, ref)
    # a bf16 result is within half an ulp (2^-9 relative) of the exact value plus fp32 accumulation error
    assert np.max(np.abs(c - ref) / (np.abs(ref) + 1e-3 * np.max(np.abs(ref)))) < 6e-3
    assert maxrel < 4e-3


@pytest.mark.parametrize("tiles,m", [(1, 300), (2, 330), (3, 130)])
@pytest.mark.parametrize("k", [8, 64, 72, 128, 192, 200, 256, 320, 456])
def test_gemm_nt_around_the_look_ahead(lib, tiles, m, k):
    # one to eight k-tiles, whole and ragged: fewer than the panel rings hold, as many, and more (two or three panels
    # requested ahead, by the tile shape; chunks beyond K among the first, the refilled and the last)
    import torch
    rng = np.random.default_rng(m + k)
    a = W.round_to_bf16(rng.standard_normal((m, k), dtype=np.float32))
    b = W.round_to_bf16(rng.standard_normal((264, k), dtype=np.float32) * 0.05)
    layer = lib.Layer(W.TINY, device=0)
    layer.set_gemm_tiles(tiles)
    c = to_np(layer.gemm_nt(torch.from_numpy(a).cuda().to(torch.bfloat16), torch.from_numpy(b).cuda().to(torch.bfloat16)))
    ref = a.astype(np.float64) @ b.astype(np.float64).T
    assert np.max(np.abs(c - ref) / (np.abs(ref) + 1e-3 * np.max(np.abs(ref)))) < 6e-3
    assert errs(c, ref)[0] < 4e-3


@pytest.mark.parametrize("m,n,k", [(2600, 4104, 520),    # 187 tiles for 256 workgroups: every tile cut along K
                                   (4096, 4096, 192),    # 256 tiles: one whole round, nothing shared
                                   (4100, 5000, 328),    # 340 tiles: all shared, more than a tile's worth each
                                   (5000, 7000, 200),    # 560 tiles: a round of whole tiles, then 304 shared ones
                                   (300, 704, 8200),     # 6 tiles, 129 k-tiles each: dozens of parts per tile
                                   (256, 256, 64), (1, 8, 8)])
def test_gemm_nt_on_shared_tiles(lib, m, n, k):
    # tile shape 6: persistent workgroups, the tiles of the last rounds cut along K; whoever arrives
    # last at a tile adds its parts up in a fixed order, so two runs agree bit for bit
    import torch
    rng = np.random.default_rng(m + n + k)
    a = W.round_to_bf16(rng.standard_normal((m, k), dtype=np.float32))
    b = W.round_to_bf16(rng.standard_normal((n, k), dtype=np.float32) * 0.05)
    layer = lib.Layer(W.TINY, device=0)
    layer.set_gemm_tiles(6)
    ta = torch.from_numpy(a).cuda().to(torch.bfloat16)
    tb = torch.from_numpy(b).cuda().to(torch.bfloat16)
    c1 = layer.gemm_nt(ta, tb)
    c2 = layer.gemm_nt(ta, tb)       # also: the arrival counters were left at zero
    torch.cuda.synchronize()
    assert torch.equal(c1, c2)
    c = to_np(c1)
    ref = a.astype(np.float64) @ b.astype(np.float64).T
    maxrel, mae = errs(c, ref)
    assert np.max(np.abs(c - ref) / (np.abs(ref) + 1e-3 * np.max(np.abs(ref)))) < 6e-3
    assert maxrel < 4e-3


@pytest.mark.parametrize("shape", [W.LayerShape(1024, 8, 2, 128, 2056), W.LayerShape(512, 8, 2, 64, 33024)])
def test_layer_step_on_shared_tiles(lib, shape):
    # every GEMM of the step, with its fused epilogue, on shared tiles (ragged in every dimension)
    import torch
    batch = W.assemble_batch(16, [(700, 700, -1), (391, 500, -1)] + [(1, 200 + 7 * i, -1) for i in range(50)], 2,
                             [], np.random.default_rng(5))
    tens = W.make_tensors(shape, batch, 5, gains="random")
    ref = O.layer_step(shape, tens, batch)
    diag = O.layer_step(shape, tens, batch, storage="bf16")
    layer = lib.Layer(shape, device=0)
    layer.set_gemm_tiles(6)
    dev = layer.upload(tens, batch)
    y = layer.blend_step(dev, batch)
    torch.cuda.synchronize()
    check(to_np(y), ref["y"], diag["y"], "shared tiles")
    k, v = layer.unpack_pool(dev.kv_pool, dev.n_pages)
    k, v = to_np(k), to_np(v)
    check(k[ref["dest"][:, 0], ref["dest"][:, 1]], ref["k_new"], diag["k_new"], "appended keys")
    check(v[ref["dest"][:, 0], ref["dest"][:, 1]], ref["v_new"], diag["v_new"], "appended values")


@pytest.mark.parametrize("rows", [77, 256, 257, 640, 1000])
def test_layer_step_on_tiles_cut_along_k(lib, rows):
    # few enough rows that whole tiles would leave CUs idle: the down projection (193 k-tiles, the last one
    # partial) is cut into ranges of 128x128, 256x128, 160x256 and 256x256 tiles
    shape = W.LayerShape(4096, 8, 2, 128, 12296)
    assert lib.Layer(shape, device=-1).gemm_division("down", rows) == {77: (3, 8), 256: (5, 8), 257: (2, 8), 640: (2, 4), 1000: (1, 4)}[rows]
    seqs = [(rows - 13, rows - 3, -1)] + [(1, 20 + 9 * i, -1) for i in range(13)]
    batch = W.assemble_batch(16, seqs, 1, [], np.random.default_rng(rows))
    check_step(lib, shape, batch, W.make_tensors(shape, batch, rows, gains="random"))


@pytest.mark.parametrize("shape,rows,want", [
    # 128x256 tiles on the deep weight ring: every product of at most 128 rows, and QKV of 64-wide heads
    (W.LayerShape(6656, 32, 16, 128, 4104), 97, [(4, 8), (4, 8), (4, 8)]), (W.LayerShape(6656, 32, 16, 128, 4104), 128, [(4, 8), (4, 8), (4, 8)]),
    (W.LayerShape(4096, 64, 64, 64, 512), 100, [(4, 5), (3, 8), (3, 1)]),
    # 160x256 and 256x256 tiles cut along K under the QKV and the output projection
    (W.LayerShape(4096, 64, 8, 64, 1032), 271, [(2, 6), (2, 8), (3, 1)]), (W.LayerShape(5120, 40, 8, 128, 520), 389, [(2, 3), (2, 4), (3, 1)]),
    (W.LayerShape(5120, 40, 8, 128, 520), 499, [(1, 4), (1, 5), (3, 1)]), (W.LayerShape(4096, 32, 32, 128, 520), 389, [(1, 2), (2, 5), (3, 1)])])
def test_layer_step_on_wide_tiles_cut_along_k(lib, shape, rows, want):
    layer = lib.Layer(shape, device=-1)
    assert [layer.gemm_division(p, rows) for p in ("qkv", "o", "down")] == want
    seqs = [(rows - 21, rows - 5, -1)] + [(1, 20 + 9 * i, -1) for i in range(21)]
    batch = W.assemble_batch(16, seqs, 1, [], np.random.default_rng(rows))
    check_step(lib, shape, batch, W.make_tensors(shape, batch, rows, gains="random"))


def attention_reference(shape, batch, q, k_pool, v_pool, storage="exact"):
    out = np.zeros((batch.n_rows, shape.n_q_heads * shape.head_dim))
    for s in range(batch.n_seq):
        r0, r1 = int(batch.row_start[s]), int(batch.row_start[s + 1])
        L = int(batch.kv_len[s])
        K, V = O.gather_kv(batch, s, L, k_pool, v_pool)
        o = O.attention(q[r0:r1].reshape(r1 - r0, shape.n_q_heads, shape.head_dim), K, V, L - (r1 - r0), storage)
        out[r0:r1] = o.reshape(r1 - r0, -1)
    return out


def check_attention(shape, batch, q, tens, out, what="attention"):
    ref = attention_reference(shape, batch, q.astype(np.float64), tens.k_pool, tens.v_pool)
    diag = attention_reference(shape, batch, q.astype(np.float64), tens.k_pool, tens.v_pool, "bf16")
    diag = W.round_to_bf16(diag.astype(np.float32)).astype(np.float64)   # the output is stored in bfloat16 too
    check(out, ref, diag, what)


@pytest.mark.parametrize("shape", [W.LayerShape(256, 4, 2, 64, 688), W.LayerShape(512, 8, 2, 128, 256),
                                   W.LayerShape(512, 8, 1, 128, 256), W.LayerShape(256, 4, 4, 64, 256)])
@pytest.mark.parametrize("seed", [0, 1, 2])
def test_attention_alone(lib, shape, seed):
    import torch
    batch = W.batch_random(seed, n_prefill=4, n_decode=40, max_q=100, max_ctx=700, n_roots=3)
    tens = W.make_tensors(shape, batch, seed)
    rng = np.random.default_rng(seed)
    q = W.round_to_bf16(rng.standard_normal((batch.n_rows, shape.n_q_heads * shape.head_dim), dtype=np.float32))
    layer = lib.Layer(shape, device=0)
    layer.set_chunk_pages(4)  # several chunks per node and per tail
    pool = layer.pack_pool(tens.k_pool, tens.v_pool)
    tq = torch.from_numpy(q).cuda().to(torch.bfloat16)
    out = to_np(layer.attention(batch, tq, pool, batch.n_pages))
    check_attention(shape, batch, q, tens, out)


@pytest.mark.parametrize("shape", [W.LayerShape(256, 4, 2, 64, 256), W.LayerShape(512, 8, 2, 128, 256),
                                   W.LayerShape(1024, 8, 1, 128, 256)])
@pytest.mark.parametrize("members", [[2, 9], [5, 17, 33], [8, 16, 70]])
def test_attention_node_member_counts(lib, shape, members):
    # prefix nodes whose members fill one to several blocks of 16 query rows, some of
    # them partly: a root of 35 tokens per member count, one child node under the first
    import torch
    nodes, seqs = [], [(7, 40, -1)]
    rng = np.random.default_rng(sum(members))
    for k, n in enumerate(members):
        root = len(nodes)
        nodes.append((-1, 2 + k))
        leaf = root
        if k == 0:
            nodes.append((root, 3))
            leaf = root + 1
        for j in range(n):
            shared = 16 * ((2 + k) + (3 if leaf != root else 0))
            nd = leaf if j < (n + 1) // 2 or leaf == root else root
            sh = shared if nd == leaf else 16 * (2 + k)
            seqs.append((1, sh + 1 + int(rng.integers(0, 90)), nd))
    # members of the child node come first within the root's run: already so by construction
    batch = W.assemble_batch(16, seqs, 1, nodes, rng)
    tens = W.make_tensors(shape, batch, 5)
    q = W.round_to_bf16(rng.standard_normal((batch.n_rows, shape.n_q_heads * shape.head_dim), dtype=np.float32))
    layer = lib.Layer(shape, device=0)
    pool = layer.pack_pool(tens.k_pool, tens.v_pool)
    out = to_np(layer.attention(batch, torch.from_numpy(q).cuda().to(torch.bfloat16), pool, batch.n_pages))
    check_attention(shape, batch, q, tens, out)


@pytest.mark.parametrize("root_pages,n_members", [(20, 40), (14, 41)])
def test_attention_wide_items_alternate_with_narrow_ones(lib, root_pages, n_members):
    # one long shared root cut into chunks of two pages, short private tails: the workgroups of
    # 64-row items are more than a third of the launch (they go first; many of them in turn with
    # narrow ones: test_wide_items_in_turn_with_narrow_ones)
    import torch
    shape = W.LayerShape(512, 8, 2, 128, 256)
    rng = np.random.default_rng(root_pages * 100 + n_members)
    nodes = [(-1, root_pages)]
    seqs = [(7, 40, -1)] + [(1, 16 * root_pages + 1 + int(rng.integers(0, 30)), 0) for _ in range(n_members)]
    batch = W.assemble_batch(16, seqs, 1, nodes, rng)
    tens = W.make_tensors(shape, batch, 11)
    q = W.round_to_bf16(rng.standard_normal((batch.n_rows, shape.n_q_heads * shape.head_dim), dtype=np.float32))
    layer = lib.Layer(shape, device=0)
    layer.set_chunk_pages(2)
    pool = layer.pack_pool(tens.k_pool, tens.v_pool)
    out = to_np(layer.attention(batch, torch.from_numpy(q).cuda().to(torch.bfloat16), pool, batch.n_pages))
    check_attention(shape, batch, q, tens, out)


@pytest.mark.parametrize("shape", [W.LayerShape(256, 4, 2, 64, 256), W.LayerShape(512, 8, 2, 128, 256)])
@pytest.mark.parametrize("lens,root_pages", [([1], 0), ([127, 128, 129], 0), ([4001, 16], 0), ([33] * 70, 0),
                                             ([40] * 9, 9), ([17, 300] * 5, 33)])
def test_attention_of_few_sequences(lib, shape, lens, root_pages):
    # the library's own division into chunks where the step cannot fill the chip (8 pages at the least:
    # contexts that end before, at and behind a chunk), decode rows alone, with and without a prefix
    # node; the two entry points divide and compute alike
    import torch
    rng = np.random.default_rng(len(lens) * 100 + root_pages)
    nodes = [(-1, root_pages)] if root_pages else []
    batch = W.assemble_batch(16, [(1, 16 * root_pages + n, 0 if nodes else -1) for n in lens], 0, nodes, rng)
    tens = W.make_tensors(shape, batch, 7)
    q = W.round_to_bf16(rng.standard_normal((batch.n_rows, shape.n_q_heads * shape.head_dim), dtype=np.float32))
    layer = lib.Layer(shape, device=0)
    pool = layer.pack_pool(tens.k_pool, tens.v_pool)
    tq = torch.from_numpy(q).cuda().to(torch.bfloat16)
    out = layer.attention(batch, tq, pool, batch.n_pages)
    check_attention(shape, batch, q, tens, to_np(out))
    assert torch.equal(out, layer.attention_noalloc(batch, tq, pool, batch.n_pages, torch.zeros_like(tq)))


@pytest.mark.parametrize("shape", [W.LayerShape(256, 4, 1, 64, 256), W.LayerShape(256, 4, 2, 128, 256), W.LayerShape(128, 2, 2, 64, 256)])
@pytest.mark.parametrize("rows,cached", [(1, 0), (16, 16), (32, 1), (33, 31), (64, 0), (65, 190), (129, 0), (257, 255), (300, 517)])
def test_prefill_attention_edges(lib, shape, rows, cached):
    # four, two and one query heads per workgroup (one, two and four blocks of 64 query rows); walks of one
    # to 26 blocks of 32 tokens (odd and even, shorter and longer than the ring of eight), last ones
    # partial; wavefronts without rows.  Slots behind the context hold NaN.
    import torch
    batch = W.assemble_batch(16, [(rows, rows + cached, -1), (5, 5 + cached // 2, -1)], 2, [], np.random.default_rng(rows))
    tens = W.make_tensors(shape, batch, 3)
    kp, vp = tens.k_pool.copy(), tens.v_pool.copy()
    for s in range(batch.n_seq):
        L = int(batch.kv_len[s])
        if L % 16:
            pg = int(batch.page_ids[int(batch.page_start[s]) + (L - 1) // 16])
            kp[pg, L % 16:] = 0x7FC0
            vp[pg, L % 16:] = 0x7FC0
    q = W.round_to_bf16(np.random.default_rng(cached).standard_normal((batch.n_rows, shape.n_q_heads * shape.head_dim), dtype=np.float32))
    layer = lib.Layer(shape, device=0)
    pool = layer.pack_pool(kp, vp)
    out = to_np(layer.attention(batch, torch.from_numpy(q).cuda().to(torch.bfloat16), pool, batch.n_pages))
    check_attention(shape, batch, q, tens, out)


@pytest.mark.parametrize("heads,dh", [((16, 16), 64), ((8, 8), 128), ((24, 8), 64), ((16, 8), 128)])
@pytest.mark.parametrize("segments,rows,cached", [(90, 1, 0), (60, 16, 16), (60, 32, 1), (48, 33, 31), (40, 64, 0), (36, 65, 190), (96, 70, 47)])
def test_prefill_attention_without_the_ring(lib, heads, dh, segments, rows, cached):
    # many short chunks of one, two and three query heads per KV head; walks of one to 11 blocks of 32 tokens, last ones
    # partial, one or both blocks of 32 query rows.  Slots behind the contexts hold NaN.
    import torch
    shape = W.LayerShape(256, heads[0], heads[1], dh, 256)
    batch = W.assemble_batch(16, [(rows, rows + cached + i % 3, -1) for i in range(segments)] + [(1, 33, -1)], segments, [],
                             np.random.default_rng(rows))
    layer = lib.Layer(shape, device=0)
    assert layer.attention_division(batch).prefill_rows == 64
    tens = W.make_tensors(shape, batch, 3)
    kp, vp = tens.k_pool.copy(), tens.v_pool.copy()
    for s in range(batch.n_seq):
        L = int(batch.kv_len[s])
        if L % 16:
            pg = int(batch.page_ids[int(batch.page_start[s]) + (L - 1) // 16])
            kp[pg, L % 16:] = 0x7FC0
            vp[pg, L % 16:] = 0x7FC0
    q = W.round_to_bf16(np.random.default_rng(cached).standard_normal((batch.n_rows, shape.n_q_heads * shape.head_dim), dtype=np.float32))
    pool = layer.pack_pool(kp, vp)
    out = to_np(layer.attention(batch, torch.from_numpy(q).cuda().to(torch.bfloat16), pool, batch.n_pages))
    check_attention(shape, batch, q, tens, out)


def test_attention_ignores_stale_slots(lib):
    # slots past kv_len in the last page hold NaN bit patterns: they must never reach the output
    import torch
    shape = W.LayerShape(256, 4, 2, 64, 688)
    batch = W.assemble_batch(16, [(5, 21, -1), (1, 35, -1), (1, 17, -1)], 1, [], None)
    tens = W.make_tensors(shape, batch, 3)
    kp, vp = tens.k_pool.copy(), tens.v_pool.copy()
    for s in range(batch.n_seq):
        L = int(batch.kv_len[s])
        pg = int(batch.page_ids[int(batch.page_start[s]) + (L - 1) // 16])
        kp[pg, L % 16:] = 0x7FC0 if L % 16 else kp[pg, L % 16:]
        vp[pg, L % 16:] = 0x7FC0 if L % 16 else vp[pg, L % 16:]
    rng = np.random.default_rng(0)
    q = W.round_to_bf16(rng.standard_normal((batch.n_rows, 256), dtype=np.float32))
    layer = lib.Layer(shape, device=0)
    pool = layer.pack_pool(kp, vp)
    out = to_np(layer.attention(batch, torch.from_numpy(q).cuda().to(torch.bfloat16), pool, batch.n_pages))
    assert np.isfinite(out).all()
    ref = attention_reference(shape, batch, q.astype(np.float64), tens.k_pool, tens.v_pool)
    assert errs(out, ref)[0] <= MAXREL


# ---------------------------------------------------------------------------
# the whole step
# ---------------------------------------------------------------------------
def test_tiny_config(lib):
    batch = W.batch_tiny(0)
    tens = W.make_tensors(W.TINY, batch, 0)
    check_step(lib, W.TINY, batch, tens)


@pytest.mark.parametrize("seed", [0, 1, 2, 3])
@pytest.mark.parametrize("flags", [0, 1])
def test_random_batches_tiny_shape(lib, seed, flags):
    batch = W.batch_random(seed, n_prefill=3, n_decode=20, max_q=90, max_ctx=400, n_roots=2)
    tens = W.make_tensors(W.TINY, batch, seed, gains="random")
    check_step(lib, W.TINY, batch, tens, flags)


@pytest.mark.parametrize("seed", [0, 1])
def test_random_batches_head_dim_128(lib, seed):
    shape = W.LayerShape(512, 8, 2, 128, 1288)
    batch = W.batch_random(10 + seed, n_prefill=4, n_decode=30, max_q=150, max_ctx=600, n_roots=3)
    tens = W.make_tensors(shape, batch, seed, gains="random")
    check_step(lib, shape, batch, tens)


@pytest.mark.parametrize("heads", [(3, 3), (4, 2), (6, 2), (10, 2)])
@pytest.mark.parametrize("dh", [64, 128])
def test_step_with_few_heads_per_group(lib, heads, dh):
    # one, two, three and five query heads per KV head: long and short chunks beside decode rows with and without a prefix
    shape = W.LayerShape(256, heads[0], heads[1], dh, 264)
    seqs = [(300, 517, -1), (40, 90, -1), (257, 257, -1)] + [(1, 200 + 13 * i, 0) for i in range(40)] + [(1, 7 + 31 * i, -1) for i in range(20)]
    batch = W.assemble_batch(16, seqs, 3, [(-1, 11)], np.random.default_rng(heads[0]))
    check_step(lib, shape, batch, W.make_tensors(shape, batch, dh, gains="random"))


@pytest.mark.parametrize("tiles", [0, 1, 2])
def test_many_rows_use_large_tiles(lib, tiles):
    # several rows of tiles, ragged in every dimension: as chosen (128x128, cut along K or whole), and every
    # product on whole 256x256 and 160x256 tiles (QKV, whose wavefronts must cover whole heads, not on the latter)
    shape = W.LayerShape(1024, 8, 2, 128, 2056)
    layer = lib.Layer(shape, device=-1)
    layer.set_gemm_tiles(tiles)
    got = [layer.gemm_division(p, 1141) for p in ("qkv", "o", "down")]
    assert got == ([(3, 1), (3, 2), (3, 3)], [(1, 1)] * 3, [(3, 2), (2, 1), (2, 1)])[tiles]
    batch = W.assemble_batch(16, [(700, 700, -1), (391, 500, -1)] + [(1, 200 + 7 * i, -1) for i in range(50)], 2,
                             [], np.random.default_rng(5))
    tens = W.make_tensors(shape, batch, 5)
    check_step(lib, shape, batch, tens, tiles=tiles)


@pytest.mark.parametrize("n_decode,q_rows", [(60, 40), (120, 80), (97, 0)])
def test_few_rows_take_the_deep_weight_ring(lib, n_decode, q_rows):
    # at most 256 rows: the QKV, output and down projections run as k-ranges of a single row of 256x128 tiles on the
    # pipeline with its own look-ahead for the weight panel; of 128 rows and less, this narrow, on 128x128 tiles
    # (wide ones on 128x256 tiles: test_layer_step_on_wide_tiles_cut_along_k)
    shape = W.LayerShape(1024, 8, 2, 128, 2048)
    layer = lib.Layer(shape, device=-1)
    assert [layer.gemm_division(p, n_decode + q_rows)[0] for p in ("qkv", "o", "down")] == [5 if n_decode + q_rows > 128 else 3] * 3
    seqs = ([(q_rows, q_rows + 30, -1)] if q_rows else []) + [(1, 50 + 11 * i, -1) for i in range(n_decode)]
    batch = W.assemble_batch(16, seqs, 1 if q_rows else 0, [], np.random.default_rng(n_decode))
    tens = W.make_tensors(shape, batch, 7, gains="random")
    check_step(lib, shape, batch, tens)


@pytest.mark.parametrize("d_model,d_ffn", [(256, 32768), (512, 33024)])
def test_rounds_of_full_tiles_in_gate_up(lib, d_model, d_ffn):
    # 512 rows and a wide FFN: the gate/up GEMM has two whole rounds of full 256x256 tiles (four and
    # eight k-tiles per tile); the second shape adds a last round that goes out on the small tiles
    shape = W.LayerShape(d_model, 4, 2, 64, d_ffn)
    batch = W.assemble_batch(16, [(300, 300, -1), (150, 180, -1)] + [(1, 20 + 3 * i, -1) for i in range(62)], 2,
                             [], np.random.default_rng(9))
    assert batch.n_rows == 512
    assert lib.Layer(shape, device=-1).gemm_division("gate_up", 512) == (1, 1)
    tens = W.make_tensors(shape, batch, 9)
    check_step(lib, shape, batch, tens)


def test_decode_only_and_prefill_only(lib):
    for batch in (W.batch_decode_only(33, 130, seed=2), W.batch_prefill_only(3, 75, seed=2)):
        tens = W.make_tensors(W.TINY, batch, 2)
        check_step(lib, W.TINY, batch, tens)


def test_degenerate_batches(lib):
    import torch
    shape = W.TINY
    layer = lib.Layer(shape, device=0)
    # an empty batch is accepted and touches nothing
    empty = W.assemble_batch(16, [], 0, [], None)
    tens = W.make_tensors(shape, W.batch_tiny(0), 0)
    dev = layer.upload(tens, W.batch_tiny(0))
    y = torch.full_like(dev.x, 7.0)
    layer.blend_step(dev, empty, y=y)
    torch.cuda.synchronize()
    assert bool((y == 7.0).all())
    # one decode sequence whose context is its own token: attention returns its value vector
    # (softmax over one score is 1), so this reduces to the dense part of the layer
    one = W.assemble_batch(16, [(1, 1, -1)], 0, [], None)
    check_step(lib, shape, one, W.make_tensors(shape, one, 1))
    # a one-row prefill chunk behind a cached context, contexts that end exactly on a page
    # boundary, and one that starts a fresh page with this step's row
    edge = W.assemble_batch(16, [(1, 48, -1), (16, 32, -1), (3, 35, -1), (1, 16, -1), (1, 17, -1), (1, 33, -1)], 3, [],
                            np.random.default_rng(5))
    check_step(lib, shape, edge, W.make_tensors(shape, edge, 2, gains="random"))


def test_ragged_prefill_segments(lib):
    # segments of 1, 31, 32, 33, 64, 65 and 97 rows (a wavefront of prefill attention owns 64) behind
    # cached contexts that end on and off page and block boundaries
    shape = W.LayerShape(512, 8, 2, 128, 256)
    segs = [(1, 48, -1), (31, 31, -1), (32, 96, -1), (33, 33, -1), (64, 200, -1), (65, 129, -1), (97, 1000, -1)]
    batch = W.assemble_batch(16, segs + [(1, 77, -1)], len(segs), [], np.random.default_rng(11))
    check_step(lib, shape, batch, W.make_tensors(shape, batch, 6, gains="random"))


def test_contexts_up_to_the_last_position(lib):
    # the longest contexts the default RoPE table (16384 positions) admits: a prefill chunk whose
    # last row sits at the last position, decode sequences there and one page short of it, two of
    # them behind a shared prefix of 1000 pages (split over many chunks of the decode kernel)
    shape = W.TINY
    top = 16384
    batch = W.assemble_batch(16, [(70, top, -1), (1, top, -1), (1, top, 0), (1, top - 16, 0), (1, 5000, -1)], 1,
                             [(-1, 1000)], np.random.default_rng(9))
    check_step(lib, shape, batch, W.make_tensors(shape, batch, 4, gains="random"))


@pytest.mark.parametrize("shape", [W.LayerShape(512, 16, 1, 64, 256), W.LayerShape(256, 4, 4, 64, 344)])
def test_group_sizes_sixteen_and_one(lib, shape):
    # 16 query heads per KV head (one member fills a decode work item) and plain multi-head attention
    batch = W.batch_random(8, n_prefill=2, n_decode=14, max_q=40, max_ctx=260, n_roots=2)
    check_step(lib, shape, batch, W.make_tensors(shape, batch, 8))


def test_shared_and_expanded_kv_agree(lib):
    batch = W.batch_random(21, n_prefill=2, n_decode=24, max_ctx=300, n_roots=3)
    tens = W.make_tensors(W.TINY, batch, 21)
    y, _ = check_step(lib, W.TINY, batch, tens)
    e, src = W.expand_batch(batch)
    te = W.make_tensors(W.TINY, batch, 21)
    te.k_pool = tens.k_pool[np.maximum(src, 0)]
    te.v_pool = tens.v_pool[np.maximum(src, 0)]
    y2, _, _, _ = run_step(lib, W.TINY, e, te)
    # same math, different grouping of the softmax partials: equal up to bf16 rounding of the output
    assert np.max(np.abs(y - y2)) / np.max(np.abs(y)) < 1e-2
    assert np.mean(np.abs(y - y2)) < MAE


def test_layers_back_to_back(lib):
    # three layers with their own weights and pools behind one descriptor; the activations passed
    # between layers are bf16 (that is the boundary's dtype), so the oracle chain rounds them too
    import dataclasses
    import torch
    shape = W.TINY
    batch = W.batch_random(11, n_prefill=3, n_decode=12, max_q=50, max_ctx=300)
    tens = [W.make_tensors(shape, batch, 20 + l, gains="random") for l in range(3)]
    layer = lib.Layer(shape, device=0)
    devs = [layer.upload(t, batch) for t in tens]
    y = layer.blend_layers(devs, batch)
    torch.cuda.synchronize()
    x = xd = tens[0].x
    for l, t in enumerate(tens):
        ref = O.layer_step(shape, dataclasses.replace(t, x=x), batch)
        diag = O.layer_step(shape, dataclasses.replace(t, x=xd), batch, storage="bf16")
        x = W.round_to_bf16(ref["y"].astype(np.float32))
        xd = diag["y"].astype(np.float32)
        k, v = layer.unpack_pool(devs[l].kv_pool, devs[l].n_pages)
        kn = to_np(k)[ref["dest"][:, 0], ref["dest"][:, 1]]
        assert errs(kn, ref["k_new"])[0] <= MAXREL, "layer %d keys" % l
    check(to_np(y), ref["y"], diag["y"], "3 layers")
    # one layer through the same entry point equals the single-step call bit for bit
    y1 = layer.blend_layers([layer.upload(tens[0], batch)], batch)
    y0 = layer.blend_step(layer.upload(tens[0], batch), batch)
    torch.cuda.synchronize()
    assert torch.equal(y0, y1)


@pytest.mark.parametrize("shape,n_layers", [(W.TINY, 4), (W.LayerShape(512, 8, 2, 128, 1288), 3)])
@pytest.mark.parametrize("knobs", [
    dict(head_cus_min=8, tail_workgroups=16, close_margin=2, ride_percent=100),
    dict(head_cus_min=48, tail_workgroups=208, close_margin=8, ride_percent=-1, attention_waves=4),
    dict(head_cus_min=0, tail_workgroups=24, close_margin=0, ride_percent=60),
])
def test_pipelined_layers_match_the_oracle_chain(lib, shape, n_layers, knobs):
    # BS_FLAG_PIPELINE: the decode rows run one stage ahead of the prefill rows across the layer
    # boundary, and the prefill rows' down projection of layer l carries decode attention of
    # layer l+1.  Every layer's appended keys and values and the final output against the oracle
    # chain (activations between layers are bf16, so the chain rounds them too).
    import dataclasses
    import torch
    rng = np.random.default_rng(31)
    seqs = [(130, 130, -1), (70, 200, -1), (45, 45, -1)] + [(1, 40 + 37 * i, -1) for i in range(40)]
    batch = W.assemble_batch(16, seqs, 3, [], rng)
    tens = [W.make_tensors(shape, batch, 40 + l, gains="random") for l in range(n_layers)]
    layer = lib.Layer(shape, device=0)
    layer.set_overlap(always=1, min_prefill_rows=1, **knobs)
    devs = [layer.upload(t, batch) for t in tens]
    layer.profile(True)
    y = layer.blend_layers(devs, batch, flags=lib.FLAG_OVERLAP | lib.FLAG_PIPELINE)
    torch.cuda.synchronize()
    prof = layer.profile_read()
    # the path was taken: the decode rows' GEMMs ran apart in every layer, and n_layers - 1 down
    # projections of the prefill rows were launches of their own
    assert prof["gemm_decode_rows"][1] > 0 and prof["gemm_down"][1] == n_layers
    x = xd = tens[0].x
    for l, t in enumerate(tens):
        ref = O.layer_step(shape, dataclasses.replace(t, x=x), batch)
        diag = O.layer_step(shape, dataclasses.replace(t, x=xd), batch, storage="bf16")
        x = W.round_to_bf16(ref["y"].astype(np.float32))
        xd = diag["y"].astype(np.float32)
        k, v = layer.unpack_pool(devs[l].kv_pool, devs[l].n_pages)
        k, v = to_np(k), to_np(v)
        assert errs(k[ref["dest"][:, 0], ref["dest"][:, 1]], ref["k_new"])[0] <= MAXREL, "layer %d keys" % l
        assert errs(v[ref["dest"][:, 0], ref["dest"][:, 1]], ref["v_new"])[0] <= MAXREL, "layer %d values" % l
        k0 = W.bf16_bits_to_f32(t.k_pool).astype(np.float64)
        written = np.zeros(k0.shape[:2], dtype=bool)
        written[ref["dest"][:, 0], ref["dest"][:, 1]] = True
        assert np.array_equal(k[~written], k0[~written]), "layer %d: a slot outside the append destinations changed" % l
    check(to_np(y), ref["y"], diag["y"], "%d pipelined layers" % n_layers)
    # and against the same layers co-scheduled one after the other (different tile shapes at most)
    devs2 = [layer.upload(t, batch) for t in tens]
    y2 = layer.blend_layers(devs2, batch, flags=lib.FLAG_OVERLAP)
    torch.cuda.synchronize()
    assert errs(to_np(y), to_np(y2))[0] <= MAXREL


def run_coscheduled(lib, shape, batch, tens, knobs, chunk_pages=0):
    import torch
    layer = lib.Layer(shape, device=0)
    layer.set_overlap(**knobs)
    if chunk_pages:
        layer.set_chunk_pages(chunk_pages)
    dev = layer.upload(tens, batch)
    layer.profile(True)
    y = layer.blend_step(dev, batch, flags=lib.FLAG_OVERLAP)
    torch.cuda.synchronize()
    run_coscheduled.taken = layer.profile_read()["gemm_decode_rows"][1] > 0   # the decode rows' GEMMs ran apart
    k, v = layer.unpack_pool(dev.kv_pool, dev.n_pages)
    return to_np(y), to_np(k), to_np(v)


@pytest.mark.parametrize("shape", [W.TINY, W.LayerShape(512, 8, 2, 128, 1288)])
@pytest.mark.parametrize("knobs", [
    dict(head_cus_min=8, tail_workgroups=16, close_margin=2, ride_percent=100),
    dict(head_cus_min=0, tail_workgroups=24, close_margin=0, ride_percent=60),
    dict(head_cus_min=16, tail_workgroups=0, close_margin=256, ride_percent=100, drain_in_last=0),
    dict(head_cus_min=48, tail_workgroups=208, close_margin=8, ride_percent=-1, attention_waves=4),
    dict(head_cus_min=8, tail_workgroups=8, close_margin=1, ride_percent=80, carry_down=0),
    dict(head_cus_min=8, tail_workgroups=8, close_margin=1, ride_percent=0)])
def test_coscheduled_step_matches_the_oracle(lib, shape, knobs):
    # decode attention of the 16-row units inside the prefill rows' GEMM launches: attention
    # workgroups ahead of the tiles only, behind them only, both; a queue that closes at once
    # (margin beyond the tile count) with everything left to a launch of its own; all units,
    # some or none of them waiting for the carrying launches; two or three carrying launches;
    # several chunks per tail, so the queue is longer than the workers are many
    knobs = dict(knobs, min_prefill_rows=1, always=1)
    batch = W.batch_random(17, n_prefill=4, n_decode=60, max_q=150, max_ctx=700, n_roots=3)
    tens = W.make_tensors(shape, batch, 17, gains="random")
    ref = O.layer_step(shape, tens, batch)
    diag = O.layer_step(shape, tens, batch, storage="bf16")
    y, k, v = run_coscheduled(lib, shape, batch, tens, knobs, chunk_pages=4)
    assert run_coscheduled.taken, "the step did not take the co-scheduled path"
    check(y, ref["y"], diag["y"], "co-scheduled %s" % knobs)
    kn = k[ref["dest"][:, 0], ref["dest"][:, 1]]
    assert errs(kn, ref["k_new"])[0] <= MAXREL


def test_coscheduled_step_agrees_with_the_serial_one(lib):
    # same arithmetic per output element; the GEMM tile shapes differ (the carrying launches use the
    # eight-wavefront tiles), so the fp32 sums may round differently: equal to within a bf16 step
    batch = W.batch_random(4, n_prefill=4, n_decode=30, max_q=120, max_ctx=500)
    tens = W.make_tensors(W.TINY, batch, 4)
    y0, _, _, _ = run_step(lib, W.TINY, batch, tens, 0)
    y1, _, _ = run_coscheduled(lib, W.TINY, batch, tens, dict(head_cus_min=8, tail_workgroups=16, min_prefill_rows=1, always=1))
    assert np.max(np.abs(y0 - y1)) <= 2.0 ** -7 * np.max(np.abs(y0))
    assert np.mean(np.abs(y0 - y1)) <= 1e-4


def test_coscheduled_flag_falls_back_where_nothing_can_overlap(lib):
    # no prefill rows, or no decode rows: the flag changes nothing
    for batch in (W.batch_decode_only(33, 130, seed=2), W.batch_prefill_only(3, 75, seed=2)):
        tens = W.make_tensors(W.TINY, batch, 2)
        y0, _, _, _ = run_step(lib, W.TINY, batch, tens, 0)
        y1, _, _ = run_coscheduled(lib, W.TINY, batch, tens, dict(head_cus_min=8, tail_workgroups=16, min_prefill_rows=1, always=1))
        assert not run_coscheduled.taken
        assert np.array_equal(y0, y1)


def test_cost_model_keeps_small_steps_serial(lib):
    # without `always` a tiny step is not expected to gain anything and runs the serial schedule
    batch = W.batch_random(4, n_prefill=4, n_decode=30, max_q=120, max_ctx=500)
    tens = W.make_tensors(W.TINY, batch, 4)
    y0, _, _, _ = run_step(lib, W.TINY, batch, tens, 0)
    y1, _, _ = run_coscheduled(lib, W.TINY, batch, tens, dict(min_prefill_rows=1))
    assert not run_coscheduled.taken and np.array_equal(y0, y1)


def test_repeated_calls_and_growing_workspace(lib):
    import torch
    layer = lib.Layer(W.TINY, device=0)
    for seed, (npf, ndec) in enumerate([(1, 4), (3, 40), (2, 9)]):
        batch = W.batch_random(30 + seed, n_prefill=npf, n_decode=ndec, max_q=200, max_ctx=300)
        tens = W.make_tensors(W.TINY, batch, seed)
        dev = layer.upload(tens, batch)
        y = layer.blend_step(dev, batch)
        torch.cuda.synchronize()
        ref = O.layer_step(W.TINY, tens, batch)["y"]
        maxrel, mae = errs(to_np(y), ref)
        assert maxrel <= MAXREL and mae <= MAE


def test_malformed_batch_is_an_error_code_on_the_gpu_path(lib):
    batch = W.batch_tiny(0)
    tens = W.make_tensors(W.TINY, batch, 0)
    layer = lib.Layer(W.TINY, device=0)
    dev = layer.upload(tens, batch)
    bad = batch.copy()
    bad.page_ids[0] = batch.n_pages + 5
    with pytest.raises(lib.BlendStepError) as ei:
        layer.blend_step(dev, bad)
    assert ei.value.code == -1
    # the context still works afterwards
    y = layer.blend_step(dev, batch)
    assert np.isfinite(to_np(y)).all()


def test_builder_batch_through_the_layer(lib):
    # host builder -> descriptor -> blended step, against the layer oracle on the same descriptor
    from paper_2411_16102_amd import binding
    rng = np.random.default_rng(5)
    b = binding.Builder(8_030_000_000, 131072, 2.5e15, 8.0e12, 600_000_000, 16)
    for g in range(3):
        prefix = [int(t) for t in rng.integers(0, 1000, int(rng.integers(40, 120)))]
        for _ in range(6):
            toks = prefix + [int(t) for t in rng.integers(0, 1000, int(rng.integers(1, 30)))]
            b.add(toks, int(rng.integers(50, 600)), len(toks) + int(rng.integers(0, 100)))
    for _ in range(4):
        b.add([int(t) for t in rng.integers(0, 1000, int(rng.integers(20, 90)))], 4, 0)
    b.finalize()
    info, d = b.next_batch(prefill_budget=128)
    assert info["n_prefill"] > 0 and info["n_decode"] > 0 and d["n_nodes"] > 0
    batch = W.Batch(page_size=16, n_seq=d["n_seq"], n_prefill=d["n_prefill"], n_rows=d["n_rows"],
                    row_start=d["row_start"], kv_len=d["kv_len"], page_start=d["page_start"], page_ids=d["page_ids"],
                    n_nodes=d["n_nodes"], node_parent=d["node_parent"], node_page_start=d["node_page_start"],
                    node_page_ids=d["node_page_ids"], node_seq_first=d["node_seq_first"],
                    node_seq_count=d["node_seq_count"], seq_leaf_node=d["seq_leaf_node"], n_pages=d["n_pages"] + 3)
    tens = W.make_tensors(W.TINY, batch, 5)
    check_step(lib, W.TINY, batch, tens)


def test_descriptors_of_calls_in_flight_do_not_overwrite_one_another(lib):
    # both halves of the staging buffer are filled several times over, and one descriptor is larger than either,
    # with no synchronisation between the calls
    import torch
    shape = W.LayerShape(256, 8, 2, 64, 256)
    rng = np.random.default_rng(3)
    batches = [W.assemble_batch(16, [(1, 16 * pages + 5 + i % 40, 0) for i in range(n)], 0, [(-1, pages)], rng)
               for n, pages in ((300, 700), (3, 2), (900, 333), (700, 1000), (301, 450), (40, 90))]
    assert max(4 * len(b.page_ids) for b in batches) > 2 << 20 > 4 * len(batches[2].page_ids) > 1 << 20
    layer = lib.Layer(shape, device=0)
    pages = max(b.n_pages for b in batches)
    gen = torch.Generator(device="cuda").manual_seed(1)
    pool = torch.randn(pages * (layer.page_bytes() // 2), generator=gen, device="cuda").to(torch.bfloat16)
    qs = [torch.randn((b.n_rows, 512), generator=gen, device="cuda").to(torch.bfloat16) for b in batches]
    alone = []
    for b, q in zip(batches, qs):
        alone.append(lib.Layer(shape, device=0).attention(b, q, pool, pages))
        torch.cuda.synchronize()
    order = [0, 1, 2, 4, 5, 2, 0, 3, 1, 2, 4, 0, 2, 5, 3, 0, 1]
    outs = [layer.attention(batches[i], qs[i], pool, pages) for i in order]
    for i, out in zip(order, outs):
        assert torch.equal(out, alone[i]), i


def test_a_half_of_the_staging_buffer_is_refilled_behind_its_copies(lib):
    # calls whose descriptors fill more than half of a half each, enqueued behind ordinary work that takes longer than
    # the host needs for all of them: the first turns to the other half at once, one of the next has to wait on the host
    # for copies that stand behind that work, so that it has passed when the last one returns
    import time
    import torch
    shape = W.LayerShape(256, 8, 2, 64, 256)
    rng = np.random.default_rng(4)
    batches = [W.assemble_batch(16, [(1, 16 * pages + 5 + i % 40, 0) for i in range(n)], 0, [(-1, pages)], rng)
               for n, pages in ((900, 333), (800, 400), (1000, 310), (700, 450))]
    layer = lib.Layer(shape, device=0)
    for b in batches:
        assert 1 << 20 < 4 * layer.attention_division(b).descriptor_words < 2 << 20
    pages = max(b.n_pages for b in batches)
    gen = torch.Generator(device="cuda").manual_seed(1)
    pool = torch.randn(pages * (layer.page_bytes() // 2), generator=gen, device="cuda").to(torch.bfloat16)
    qs = [torch.randn((b.n_rows, 512), generator=gen, device="cuda").to(torch.bfloat16) for b in batches]
    outs = [torch.zeros_like(q) for q in qs]
    work = torch.randn((8192, 8192), generator=gen, device="cuda").to(torch.bfloat16)
    product = work @ work
    alone = [layer.attention(b, q, pool, pages) for b, q in zip(batches, qs)]   # every workspace has its size
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for b, q in zip(batches, qs):
        layer.attention(b, q, pool, pages)
    host_s = time.perf_counter() - t0
    torch.cuda.synchronize()
    begun, passed = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    begun.record()
    for _ in range(200):   # 0.1 s and more: 1.1 TFLOP each
        torch.mm(work, work, out=product)
    passed.record()
    outs[0] = layer.attention(batches[0], qs[0], pool, pages)
    assert not passed.query(), "the work ended too early to show anything"
    for i in (1, 2, 3):
        outs[i] = layer.attention(batches[i], qs[i], pool, pages)
    assert passed.query(), "a half was refilled while a copy out of it was still to come"
    torch.cuda.synchronize()
    assert begun.elapsed_time(passed) * 1e-3 > 2 * host_s
    for i in range(4):
        assert torch.equal(outs[i], alone[i]), i


@pytest.mark.parametrize("shape,rows,division", [
    # one and two blocks of rows; columns in half a block, contractions with a partial last k-tile or less than one per
    # wavefront; several items per workgroup (gate/up of 513 units)
    (W.LayerShape(264, 3, 1, 64, 344), 1, (7, 7, 7, 7)), (W.LayerShape(520, 20, 2, 128, 4104), 7, (7, 7, 7, 7)),
    (W.LayerShape(4104, 5, 1, 128, 4104), 16, (7, 7, 7, 7)), (W.LayerShape(264, 3, 1, 64, 344), 17, (7, 7, 7, 7)),
    (W.LayerShape(520, 20, 2, 128, 4104), 32, (7, 7, 7, 7)), (W.LayerShape(520, 20, 2, 128, 4104), 33, (7, 7, 7, 8)),
    (W.LayerShape(1032, 8, 8, 64, 8200), 64, (7, 7, 3, 8)), (W.LayerShape(264, 3, 1, 64, 344), 136, (7, 7, 7, 7)),
    (W.LayerShape(256, 4, 4, 64, 760), 256, (7, 7, 7, 3)), (W.LayerShape(4096, 32, 8, 128, 1024), 32, (7, 7, 7, 7))])
def test_few_rows_stream_the_weights(lib, shape, rows, division):
    layer = lib.Layer(shape, device=-1)
    assert tuple(layer.gemm_division(p, rows)[0] for p in ("qkv", "o", "down", "gate_up")) == division
    n = max(1, rows // 2)
    seqs = ([(rows - n, rows - n + 21, -1)] if rows > n else []) + [(1, 20 + 9 * i, -1) for i in range(n)]
    batch = W.assemble_batch(16, seqs, 1 if rows > n else 0, [], np.random.default_rng(rows))
    check_step(lib, shape, batch, W.make_tensors(shape, batch, rows, gains="random"))


@pytest.mark.parametrize("d_model,d_ffn,rows,tiles", [
    (2048, 4104, 50, 8), (2048, 4104, 100, 9), (2048, 16648, 97, 4),  # 64x128, 128x128 and 128x256 tiles, begun at shifted k-tiles
    (1048, 4104, 64, 8), (1048, 4104, 65, 9)])                        # begun at the first, with a partial last one
def test_gate_up_of_few_rows(lib, d_model, d_ffn, rows, tiles):
    shape = W.LayerShape(d_model, 4, 2, 64, d_ffn)
    assert lib.Layer(shape, device=-1).gemm_division("gate_up", rows) == (tiles, 1)
    seqs = [(rows - 13, rows - 3, -1)] + [(1, 20 + 9 * i, -1) for i in range(13)]
    batch = W.assemble_batch(16, seqs, 1, [], np.random.default_rng(rows))
    check_step(lib, shape, batch, W.make_tensors(shape, batch, rows, gains="random"))


@pytest.mark.parametrize("d_model,d_ffn,rows,tiles", [
    (1024, 14336, 384, 10),  # one round of 192x256 tiles, all whole
    (136, 14280, 359, 10),   # ragged rows, columns and K
    (256, 8448, 1153, 10),   # a last row of tiles with one row
    (256, 8192, 1344, 10),   # more than one round
    (256, 8192, 577, 2)])    # (so few tiles that 160x256 ones are taken)
def test_gate_up_on_192_row_tiles(lib, d_model, d_ffn, rows, tiles):
    shape = W.LayerShape(d_model, 4, 2, 64, d_ffn)
    assert lib.Layer(shape, device=-1).gemm_division("gate_up", rows) == (tiles, 1)
    seqs = [(rows - 13, rows - 3, -1)] + [(1, 20 + 9 * i, -1) for i in range(13)]
    batch = W.assemble_batch(16, seqs, 1, [], np.random.default_rng(rows))
    check_step(lib, shape, batch, W.make_tensors(shape, batch, rows, gains="random"))


@pytest.mark.parametrize("dims,rows,product,want", [
    # QKV on whole 160x256, 192x256 and 128x256 tiles, a last row of tiles with one row or an odd number of them, K no multiple of 64
    ((264, 64, 64, 64, 1032), 700, "qkv", (2, 1)), ((264, 32, 8, 128, 1032), 1281, "qkv", (2, 1)),
    ((264, 32, 8, 128, 1032), 1700, "qkv", (10, 1)), ((264, 40, 8, 128, 1032), 1537, "qkv", (10, 1)),
    ((1032, 40, 8, 128, 1032), 513, "qkv", (11, 1)), ((776, 96, 8, 64, 1032), 700, "qkv", (11, 1)), ((264, 96, 8, 64, 1032), 1601, "qkv", (10, 1)),
    # output and down projection on 128x256 and 192x256 tiles, whole and cut along K
    ((1032, 24, 8, 64, 1032), 2049, "o", (11, 2)), ((2056, 4, 2, 64, 1032), 2049, "down", (11, 1)),
    ((520, 4, 2, 64, 8200), 1700, "down", (11, 6)), ((1032, 4, 2, 64, 8200), 1281, "down", (10, 7)),
    # gate/up on 128x256 tiles
    ((1032, 4, 2, 64, 4104), 300, "gate_up", (11, 1)), ((1048, 4, 2, 64, 4104), 257, "gate_up", (11, 1))])
def test_products_on_192_and_128_row_tiles(lib, dims, rows, product, want):
    shape = W.LayerShape(*dims)
    assert lib.Layer(shape, device=-1).gemm_division(product, rows) == want
    seqs = [(rows - 33, rows + 20, -1)] + [(1, 20 + 9 * i, -1) for i in range(33)]
    batch = W.assemble_batch(16, seqs, 1, [], np.random.default_rng(rows))
    check_step(lib, shape, batch, W.make_tensors(shape, batch, rows, gains="random"))


@pytest.mark.parametrize("d_model", [8, 64, 72, 128, 192, 200, 256, 320, 456])
@pytest.mark.parametrize("heads,dh", [((96, 8), 64), ((48, 4), 128)])
def test_qkv_on_192_row_tiles_around_the_look_ahead(lib, heads, dh, d_model):
    # one to eight k-tiles, whole and ragged, on the ring of two activation and three weight panels; the last row of tiles
    # has one row
    shape = W.LayerShape(d_model, heads[0], heads[1], dh, 64)
    assert lib.Layer(shape, device=-1).gemm_division("qkv", 1537) == (10, 1)
    batch = W.assemble_batch(16, [(53, 53, -1)] * 29, 29, [], np.random.default_rng(d_model))
    check_step(lib, shape, batch, W.make_tensors(shape, batch, d_model, gains="random"))


@pytest.mark.parametrize("heads,dh,segments,n_decode", [
    # contexts cut into ranges: one row, a row block that ends at, before and behind a block of 32 tokens, ranges that may not
    # begin behind a block's first row; 64, 128 and 256 rows to a workgroup; whole and cut blocks in one launch
    ((4, 1), 128, [(1, 520)], 0), ((8, 2), 128, [(64, 1088), (65, 1088), (33, 545), (5, 9)], 0), ((4, 1), 64, [(130, 641), (31, 2047)], 0),
    ((6, 3), 128, [(129, 1500)], 0), ((3, 1), 64, [(257, 1600), (40, 1040)], 0), ((8, 2), 128, [(200, 2000), (40, 40)], 3),
    ((4, 1), 64, [(96, 1024)], 2), ((3, 3), 128, [(70, 1100)], 3)])
def test_prefill_contexts_cut_into_ranges(lib, heads, dh, segments, n_decode):
    import torch
    shape = W.LayerShape(256, heads[0], heads[1], dh, 256)
    rng = np.random.default_rng(len(segments) * 10 + n_decode)
    seqs = [(q, kv, -1) for q, kv in segments] + [(1, 20 + i, -1) for i in range(n_decode)]
    batch = W.assemble_batch(16, seqs, len(segments), [], rng)
    tens = W.make_tensors(shape, batch, 13)
    q = W.round_to_bf16(rng.standard_normal((batch.n_rows, shape.n_q_heads * dh), dtype=np.float32))
    layer = lib.Layer(shape, device=0)
    division = layer.attention_division(batch)
    cut = division.states - n_decode   # (a decode sequence of one chunk has one state)
    assert cut > 0 and cut % division.prefill_rows == 0
    pool = layer.pack_pool(tens.k_pool, tens.v_pool)
    tq = torch.from_numpy(q).cuda().to(torch.bfloat16)
    out = layer.attention(batch, tq, pool, batch.n_pages)
    check_attention(shape, batch, q, tens, to_np(out))
    assert torch.equal(layer.attention_noalloc(batch, tq, pool, batch.n_pages, torch.zeros_like(out)), out)


def test_step_with_cut_prefill_contexts(lib):
    # the schedules of a step take the same ranges: serial, co-scheduled (the states of the prefill rows are merged apart
    # from those of the decode sequences), and pipelined layers
    shape = W.LayerShape(512, 8, 2, 128, 1032)
    prefill, decode = [(290, 1400, -1), (35, 900, -1)], [(1, 30 + 7 * i, -1) for i in range(40)]
    rng = np.random.default_rng(3)
    batch = W.assemble_batch(16, prefill + decode, 2, [], rng)
    host = lib.Layer(shape, device=-1)
    division = host.attention_division(batch)
    cut = division.states - host.attention_division(W.assemble_batch(16, decode, 0, [], rng)).states
    assert cut > 0 and cut % division.prefill_rows == 0
    tens = W.make_tensors(shape, batch, 3, gains="random")
    y, ref = check_step(lib, shape, batch, tens)
    layer = lib.Layer(shape, device=0)
    layer.set_overlap(head_cus_min=8, tail_workgroups=16, min_prefill_rows=1, always=1)
    layer.profile(True)
    y1 = layer.blend_step(layer.upload(tens, batch), batch, flags=lib.FLAG_OVERLAP)
    check(to_np(y1), ref["y"], O.layer_step(shape, tens, batch, storage="bf16")["y"], "co-scheduled")
    prof = layer.profile_read()
    assert prof["gemm_decode_rows"][1] > 0 and prof["attn_merge"][1] == 2
    out = []
    for flags in (lib.FLAG_SERIAL, lib.FLAG_OVERLAP | lib.FLAG_PIPELINE):
        devs = [layer.upload(W.make_tensors(shape, batch, 3 + l, gains="random"), batch) for l in range(3)]
        layer.profile(True)
        out.append(layer.blend_layers(devs, batch, flags=flags))
        prof = layer.profile_read()
        assert prof["attn_merge"][1] == (6 if flags else 3) and prof["gemm_down"][1] == 3
    assert errs(to_np(out[1]), to_np(out[0]))[0] <= MAXREL


def test_few_wide_items_among_many_narrow_ones(lib):
    # so few wide ones go first, alone and with prefill rows
    import torch
    shape = W.LayerShape(512, 8, 2, 128, 256)
    for n_prefill in (0, 1):
        rng = np.random.default_rng(7)
        seqs = [(7, 40, -1)] * n_prefill + [(1, 16 * 5 + 3 + i % 9, 0) for i in range(20)] + [(1, 30 + i, -1) for i in range(1100)]
        batch = W.assemble_batch(16, seqs, n_prefill, [(-1, 5)], rng)
        tens = W.make_tensors(shape, batch, 11)
        q = W.round_to_bf16(rng.standard_normal((batch.n_rows, shape.n_q_heads * shape.head_dim), dtype=np.float32))
        layer = lib.Layer(shape, device=0)
        division = layer.attention_division(batch)
        assert 0 < 4 * division.wide_items < division.items
        pool = layer.pack_pool(tens.k_pool, tens.v_pool)
        out = to_np(layer.attention(batch, torch.from_numpy(q).cuda().to(torch.bfloat16), pool, batch.n_pages))
        check_attention(shape, batch, q, tens, out)


@pytest.mark.parametrize("n_prefill,groups,loose", [(0, 112, 0), (0, 111, 0), (0, 64, 192), (0, 63, 200), (0, 130, 37), (1, 192, 3), (1, 191, 0)])
def test_wide_items_in_turn_with_narrow_ones(lib, n_prefill, groups, loose):
    # 8 KV heads; 3584 units and more of which 512 are wide alone, 1536 wide ones beside prefill rows: one wide in turn with two narrow
    # ones, the rest behind; one group less: wide ones first
    import torch
    shape = W.LayerShape(64, 64, 8, 128, 64)
    rng = np.random.default_rng(groups)
    seqs = [(7, 40, -1)] * n_prefill + [(1, 16 + 3 + (5 * i) % 29, i // 3) for i in range(3 * groups)] + [(1, 30 + i, -1) for i in range(loose)]
    batch = W.assemble_batch(16, seqs, n_prefill, [(-1, 1)] * groups, rng)
    layer = lib.Layer(shape, device=0)
    division = layer.attention_division(batch)
    assert division.wide_items == groups and 2 * groups <= division.items - groups
    assert (groups >= 192 if n_prefill else groups >= 64 and division.items >= 448) == (groups not in (63, 111, 191))
    tens = W.make_tensors(shape, batch, 12)
    q = W.round_to_bf16(rng.standard_normal((batch.n_rows, shape.n_q_heads * shape.head_dim), dtype=np.float32))
    pool = layer.pack_pool(tens.k_pool, tens.v_pool)
    tq = torch.from_numpy(q).cuda().to(torch.bfloat16)
    out = layer.attention(batch, tq, pool, batch.n_pages)
    check_attention(shape, batch, q, tens, to_np(out))
    assert torch.equal(layer.attention(batch, tq, pool, batch.n_pages), out)


@pytest.mark.parametrize("d_ffn,rows,tiles", [(8200, 907, 10), (14344, 800, 2), (14344, 805, 10), (6920, 1929, 1), (14344, 521, 2), (14344, 663, 10)])
def test_gate_up_columns_on_two_tile_shapes(lib, d_ffn, rows, tiles):
    # one round of 192x256, 160x256, 192x256 and 256x256 tiles, the other columns on 128x128, 256x256 (twice) and 192x256 ones, the last
    # of them partial; 521 and 663 rows on one shape, 4 to 10 % faster there than on two
    shape = W.LayerShape(1024, 4, 2, 64, d_ffn)
    assert lib.Layer(shape, device=-1).gemm_division("gate_up", rows) == (tiles, 1)
    seqs = [(rows - 13, rows - 3, -1)] + [(1, 20 + 9 * i, -1) for i in range(13)]
    batch = W.assemble_batch(16, seqs, 1, [], np.random.default_rng(rows))
    check_step(lib, shape, batch, W.make_tensors(shape, batch, rows, gains="random"))


def test_captured_step_cuts_into_what_the_context_holds(lib):
    # a fresh context whose first step has no prefill context to cut: captured, a step that would cut one allocates nothing,
    # leaves it whole and replays to the same result; eager, it is cut
    import torch
    shape = W.LayerShape(512, 8, 2, 128, 1032)
    rng = np.random.default_rng(5)
    warm = W.assemble_batch(16, [(40, 40, -1)], 1, [], rng)
    batch = W.assemble_batch(16, [(40, 1400, -1)], 1, [], rng)
    assert warm.n_pages <= batch.n_pages
    tens = W.make_tensors(shape, batch, 5)
    layer = lib.Layer(shape, device=0)
    assert layer.attention_division(batch).states > 0 and layer.attention_division(warm).states == 0
    dev = layer.upload(tens, batch)
    layer.blend_step(dev, batch)
    fresh = lib.Layer(shape, device=0)
    fresh.blend_step(dev, warm)        # every buffer but that of the states has its size
    eager = to_np(layer.blend_step(dev, batch))   # (the pool as that step left it)
    y, graph = torch.empty_like(dev.x), torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        fresh.blend_step(dev, batch, y=y)
    for _ in range(3):
        y.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert np.abs(to_np(y) - eager).max() <= 2e-2 * np.abs(eager).max()


def test_captured_attention_cuts_into_what_the_context_holds(lib):
    # a prefill-only call needs no states without cuts, and is captured on a context that has none; on one that a shorter
    # batch has grown, whose descriptor buffer or states are short, and on one that has all: each replays to the same result
    import torch
    shape = W.LayerShape(256, 8, 2, 128, 256)
    rng = np.random.default_rng(5)
    batch = W.assemble_batch(16, [(40, 1400, -1), (9, 2100, -1)], 2, [], rng)
    warm = [W.assemble_batch(16, [(40, 40, -1)], 1, [], rng), W.assemble_batch(16, [(1, 530, -1)], 1, [], rng), batch]
    host = lib.Layer(shape, device=-1)
    assert [host.attention_division(b).states > 0 for b in warm] == [False, True, True]
    assert host.attention_division(batch).states > 2 * host.attention_division(warm[1]).states
    tens = W.make_tensors(shape, batch, 5)
    q = W.round_to_bf16(rng.standard_normal((batch.n_rows, shape.n_q_heads * shape.head_dim), dtype=np.float32))
    tq = torch.from_numpy(q).cuda().to(torch.bfloat16)
    for first in warm:
        layer = lib.Layer(shape, device=0)
        pool = layer.pack_pool(tens.k_pool, tens.v_pool)
        layer.attention(first, tq[:first.n_rows], pool, batch.n_pages)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            out = layer.attention(batch, tq, pool, batch.n_pages)
        for _ in range(3):
            out.zero_()
            graph.replay()
            torch.cuda.synchronize()
            check_attention(shape, batch, q, tens, to_np(out))
            layer.attention(warm[2], tq, pool, batch.n_pages)  # grows the states between the replays


def test_cut_contexts_leave_captured_calls_their_workspace(lib):
    # a decode call and a cut prefill call are captured; calls that cut more grow the states between the replays
    import torch
    shape = W.LayerShape(256, 8, 2, 128, 256)
    rng = np.random.default_rng(6)
    decode = W.assemble_batch(16, [(1, 300 + 40 * i, -1) for i in range(6)], 0, [], rng)
    small = W.assemble_batch(16, [(9, 700, -1)], 1, [], rng)
    larger = [W.assemble_batch(16, [(33, 2500, -1)] * n, n, [], rng) for n in (1, 3)]
    layer = lib.Layer(shape, device=0)
    states = [layer.attention_division(b).states for b in [small] + larger]
    assert 0 < states[0] and 2 * states[0] + 64 < states[1] and 2 * states[1] < states[2]
    assert all(layer.attention_division(b).descriptor_words < 1024 for b in larger)  # (the descriptor's buffer stays)
    calls = []
    for b in [decode, small] + larger:
        t = W.make_tensors(shape, b, 6)
        q = W.round_to_bf16(rng.standard_normal((b.n_rows, shape.n_q_heads * shape.head_dim), dtype=np.float32))
        calls.append((b, t, q, torch.from_numpy(q).cuda().to(torch.bfloat16), layer.pack_pool(t.k_pool, t.v_pool)))
    graphs = []
    for b, t, q, tq, pool in calls[:2]:
        layer.attention(b, tq, pool, b.n_pages)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            out = layer.attention(b, tq, pool, b.n_pages)
        graphs.append((graph, out))
    for b, t, q, tq, pool in calls[2:]:
        check_attention(shape, b, q, t, to_np(layer.attention(b, tq, pool, b.n_pages)))
        for (graph, out), (cb, ct, cq, _, _) in zip(graphs, calls):
            out.zero_()
            graph.replay()
            torch.cuda.synchronize()
            check_attention(shape, cb, cq, ct, to_np(out))


def test_cut_contexts_on_a_context_whose_descriptor_buffer_holds_the_whole_ones(lib):
    # a short call leaves a descriptor buffer that would do for whole contexts: the same ranges as on a new context, and as
    # bs_attention_noalloc takes; a call that was captured with that buffer replays to the same result
    import torch
    shape = W.LayerShape(256, 8, 2, 128, 256)
    rng = np.random.default_rng(9)
    first, batch = W.assemble_batch(16, [(9, 9, -1)], 1, [], rng), W.assemble_batch(16, [(9, 1409, -1)] * 8, 8, [], rng)
    layer = lib.Layer(shape, device=0)
    held = (layer.attention_division(first).descriptor_words + 3) // 4 * 5 + 1024
    whole = lib.Layer(shape, device=-1)
    whole.set_chunk_pages(64)
    assert whole.attention_division(batch).descriptor_words <= held - 4 and held < layer.attention_division(batch).descriptor_words
    calls = []
    for b in (first, batch):
        t = W.make_tensors(shape, b, 9)
        q = W.round_to_bf16(rng.standard_normal((b.n_rows, shape.n_q_heads * shape.head_dim), dtype=np.float32))
        calls.append((b, t, q, torch.from_numpy(q).cuda().to(torch.bfloat16), layer.pack_pool(t.k_pool, t.v_pool)))
    (fb, ft, fq, ftq, fpool), (b, t, q, tq, pool) = calls
    layer.attention(fb, ftq, fpool, fb.n_pages)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        captured = layer.attention(fb, ftq, fpool, fb.n_pages)
    for _ in range(2):
        out = layer.attention(b, tq, pool, b.n_pages)
        check_attention(shape, b, q, t, to_np(out))
        assert torch.equal(lib.Layer(shape, device=0).attention(b, tq, pool, b.n_pages), out)
        assert torch.equal(layer.attention_noalloc(b, tq, pool, b.n_pages, torch.zeros_like(out)), out)
        captured.zero_()
        graph.replay()
        torch.cuda.synchronize()
        check_attention(shape, fb, fq, ft, to_np(captured))


@pytest.mark.parametrize("d_ffn,rows,launches", [(8200, 907, 2), (14344, 800, 2), (14344, 805, 2), (6920, 1929, 2),  # two shapes
                                                 (14344, 1216, 2), (14344, 1500, 1), (14344, 663, 1)])
def test_gate_up_in_as_many_launches_as_are_expected_to_be_shorter(lib, d_ffn, rows, launches):
    # 1216 rows: whole rounds of 256x256 tiles and 128x128 ones for the rest; 1500: these would take longer than whole tiles
    shape = W.LayerShape(1024, 4, 2, 64, d_ffn)
    layer = lib.Layer(shape, device=0)
    batch = W.assemble_batch(16, [(rows, rows, -1)], 1, [], np.random.default_rng(rows))
    dev = layer.upload(W.make_tensors(shape, batch, rows), batch)
    layer.profile(True)
    layer.blend_step(dev, batch)
    assert layer.profile_read()["gemm_gate_up"][1] == launches
