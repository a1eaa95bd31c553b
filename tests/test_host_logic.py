"""CPU-side checks of the library: exported symbols, descriptor validation and
bit-exact page resolution against the oracle's resolver.  No GPU is touched."""
import os

import numpy as np
import pytest

from oracle import layer as O
from paper_2411_16102_amd import binding, workloads as W


@pytest.fixture(scope="module")
def host_layer():
    return binding.Layer(W.TINY, device=-1)


def test_library_exports_every_declared_function():
    names = binding.declared_functions()
    assert "bs_blend_step" in names and "bs_create" in names and len(names) >= 15
    assert binding.check_symbols()


def test_gpu_entry_points_refuse_a_host_only_context(host_layer):
    b = W.batch_tiny()
    d, keep = binding.marshal_batch(b)
    import ctypes as C
    w = binding.Weights(*[C.c_void_p(8)] * 6)
    rc = host_layer.lib.bs_blend_step(host_layer.h, C.byref(w), C.byref(d), C.c_void_p(8), C.c_void_p(16),
                                      C.c_void_p(24), b.n_pages, None, 0)
    assert rc == -1 and "host-only" in host_layer.last_error()


@pytest.mark.parametrize("name", list(W.CONFIGS))
def test_generated_configs_validate(host_layer, name):
    shape, fn = W.CONFIGS[name]
    b = fn()
    lay = binding.Layer(shape, device=-1)
    assert lay.validate(b) == 0, lay.last_error()


@pytest.mark.parametrize("seed", range(6))
def test_row_resolution_is_bit_exact(host_layer, seed):
    b = W.batch_random(seed, n_prefill=4, n_decode=12, max_q=70, max_ctx=300)
    pg, sl = host_layer.resolve_rows(b)
    row = 0
    for s in range(b.n_seq):
        q = int(b.row_start[s + 1] - b.row_start[s])
        for j in range(q):
            want = O.resolve(b, s, int(b.kv_len[s]) - q + j)
            assert (int(pg[row]), int(sl[row])) == want
            row += 1
    assert row == b.n_rows


def test_row_resolution_full_size_config(host_layer):
    shape, fn = W.CONFIGS["blended_8b"]
    b = fn()
    lay = binding.Layer(shape, device=-1)
    pg, sl = lay.resolve_rows(b)
    rng = np.random.default_rng(0)
    row_seq = np.repeat(np.arange(b.n_seq), b.q_len())
    for r in rng.integers(0, b.n_rows, 300):
        s = int(row_seq[r])
        pos = int(b.kv_len[s]) - int(b.row_start[s + 1] - b.row_start[s]) + int(r - b.row_start[s])
        assert (int(pg[r]), int(sl[r])) == O.resolve(b, s, pos)


def _bad(host_layer, b, n_pages=None):
    rc = host_layer.validate(b, n_pages)
    return rc, host_layer.last_error()


def test_malformed_descriptors_are_error_codes(host_layer):
    good = W.batch_random(1, n_prefill=2, n_decode=8)
    assert host_layer.validate(good) == 0

    b = good.copy(); b.page_ids[3] = good.n_pages
    rc, msg = _bad(host_layer, b); assert rc == -1 and "outside the pool" in msg

    b = good.copy(); b.page_ids[0] = -1
    assert _bad(host_layer, b)[0] == -1

    b = good.copy(); b.kv_len[0] = int(np.diff(b.page_start)[0]) * 16 + 1
    rc, msg = _bad(host_layer, b); assert rc == -1 and "exceeds its" in msg

    b = good.copy(); b.row_start[1] = b.row_start[0]
    assert _bad(host_layer, b)[0] == -1

    b = good.copy(); b.n_rows += 1
    assert _bad(host_layer, b)[0] == -1

    b = good.copy(); b.page_start[2] = b.page_start[1] - 1
    assert _bad(host_layer, b)[0] == -1

    b = good.copy(); b.kv_len[b.n_prefill] = 0
    assert _bad(host_layer, b)[0] == -1

    # a decode sequence with two rows
    b = good.copy(); b.n_prefill = 0
    assert _bad(host_layer, b)[0] == -1

    # kv_len beyond the RoPE table
    b = W.assemble_batch(16, [(1, 20000, -1)], 0, [], None)
    rc, msg = _bad(host_layer, b); assert rc == -1 and "max_positions" in msg


def test_shared_page_may_not_be_written(host_layer):
    # two sequences whose last (written) page is the same physical page
    b = W.assemble_batch(16, [(1, 20, -1), (1, 20, -1)], 0, [], None)
    b.page_ids[3] = b.page_ids[1]
    rc, msg = _bad(host_layer, b)
    assert rc == -1 and "more than once" in msg
    # a node page may not be written even by its only member
    b = W.assemble_batch(16, [(1, 33, 0)], 0, [(-1, 2)], None)
    assert host_layer.validate(b) == 0
    b.kv_len[0] = 32
    rc, msg = _bad(host_layer, b)
    assert rc == -1


def test_inconsistent_nodes_are_rejected(host_layer):
    good = W.batch_tiny()
    assert host_layer.validate(good) == 0
    b = good.copy(); b.node_page_ids[2] = (b.node_page_ids[2] + 1) % good.n_pages
    rc, msg = _bad(host_layer, b); assert rc == -1 and "does not carry" in msg
    b = good.copy(); b.node_seq_count[0] = 7
    assert _bad(host_layer, b)[0] == -1
    b = good.copy(); b.node_seq_first[0] = 1   # run would include a prefill segment
    assert _bad(host_layer, b)[0] == -1
    b = good.copy(); b.seq_leaf_node[0] = 0    # prefill segment as a node member
    assert _bad(host_layer, b)[0] == -1
    b = good.copy(); b.node_parent[0] = 0
    assert _bad(host_layer, b)[0] == -1
    b = good.copy(); b.seq_leaf_node[5] = 3
    assert _bad(host_layer, b)[0] == -1


def test_empty_batch_is_valid(host_layer):
    b = W.assemble_batch(16, [], 0, [], None)
    assert host_layer.validate(b) == 0


def test_node_arrays_of_an_empty_batch_are_not_read(host_layer):
    import ctypes as C
    starts = (C.c_int32 * 4)(0, 0, 0, 0)
    d = binding.BatchDesc(n_seq=0, n_prefill=0, n_rows=0, n_nodes=3, node_page_start=C.cast(starts, C.POINTER(C.c_int32)))
    out = (C.c_int32 * 1)(7)
    assert host_layer.lib.bs_resolve_rows(host_layer.h, C.byref(d), out, out) == 0 and out[0] == 7
    div = binding.Division()
    assert host_layer.lib.bs_attention_division(host_layer.h, C.byref(d), 4, 1, C.byref(div)) == 0 and div.items == 0


def test_tuning_knobs_reject_values_outside_their_range(host_layer):
    for bad in (0, 1, 3, 66, -2):
        assert host_layer.lib.bs_set_chunk_pages(host_layer.h, bad) == -1 and "chunk_pages" in host_layer.last_error()
    for ok in (2, 32, 64):
        assert host_layer.lib.bs_set_chunk_pages(host_layer.h, ok) == 0
    assert host_layer.lib.bs_set_gemm_tiles(host_layer.h, 4) == -1
    assert host_layer.lib.bs_set_gemm_tiles(host_layer.h, 7) == -1
    assert host_layer.lib.bs_set_gemm_tiles(host_layer.h, 0) == 0
    good = host_layer.get_overlap()
    for bad in (dict(head_cus_min=4), dict(head_cus_min=200), dict(head_cus_min=-8), dict(tail_workgroups=257),
                dict(close_margin=-1), dict(min_prefill_rows=0), dict(ride_percent=101), dict(ride_percent=-2),
                dict(attention_waves=0), dict(attention_waves=9), dict(head_cus_max=7), dict(head_cus_max=200)):
        with pytest.raises(binding.BlendStepError):
            host_layer.set_overlap(**bad)
    assert host_layer.get_overlap() == good
    host_layer.set_overlap(head_cus_min=48, ride_percent=50)
    assert host_layer.get_overlap()["head_cus_min"] == 48 and host_layer.get_overlap()["ride_percent"] == 50
    host_layer.set_overlap(**good)


NOALLOC_WORDS = (1 << 20) // 4   # descriptor limit of bs_attention_noalloc, in 32-bit words


def _near_the_descriptor_limit(fill_pages):
    # one KV head: 80 contexts of 57 pages are cut into chunks of eight pages, 560 items more than chunks
    # of 64; prefill tables of `fill_pages` pages fill the descriptor
    seqs = []
    while fill_pages > 0:
        pages = min(1024, fill_pages)
        seqs.append((1, 16 * pages, -1))
        fill_pages -= pages
    n_prefill = len(seqs)
    return W.assemble_batch(16, seqs + [(1, 57 * 16, -1)] * 80, n_prefill, [], None)


def _fields(d):
    return (d.items, d.wide_items, list(d.longest_item_tokens), d.states, d.descriptor_words)


def test_noalloc_division_never_outgrows_the_descriptor_buffer():
    lay = binding.Layer(W.LayerShape(256, 16, 1, 64, 256), device=-1)
    empty = _near_the_descriptor_limit(0)
    coarse, fine = lay.attention_division(empty, noalloc=True), lay.attention_division(empty)
    assert fine.longest_item_tokens[0] == 128 and fine.items == 80 * 8
    assert (coarse.items, coarse.descriptor_words) == (fine.items, fine.descriptor_words)   # far from the limit: taken as it is
    lay.set_chunk_pages(8)
    fine_words = [lay.attention_division(_near_the_descriptor_limit(f)).descriptor_words for f in (248_000, 254_000)]
    assert fine_words[0] <= NOALLOC_WORDS < fine_words[1]   # the finer division stops fitting within the range
    lay = binding.Layer(W.LayerShape(256, 16, 1, 64, 256), device=-1)
    for fill in range(248_000, 254_001, 150):
        b = _near_the_descriptor_limit(fill)
        got = lay.attention_division(b, noalloc=True)
        assert got.descriptor_words <= NOALLOC_WORDS
        assert _fields(got) == _fields(lay.attention_division(b))
    # what the fixed division (chunks of 64 pages) fits is accepted, what it
    # does not fit is refused
    fixed = binding.Layer(W.LayerShape(256, 16, 1, 64, 256), device=-1)
    fixed.set_chunk_pages(64)
    spare = NOALLOC_WORDS - fixed.attention_division(_near_the_descriptor_limit(254_000)).descriptor_words
    for fill in range(254_000 + spare - 70, 254_000 + spare + 10, 10):   # (a prefill segment takes nine words beside its table)
        b = _near_the_descriptor_limit(fill)
        if fixed.attention_division(b).descriptor_words <= NOALLOC_WORDS:
            assert lay.attention_division(b, noalloc=True).descriptor_words <= NOALLOC_WORDS
        else:
            with pytest.raises(binding.BlendStepError, match="descriptor"):
                lay.attention_division(b, noalloc=True)


@pytest.mark.parametrize("seed", range(8))
def test_attention_division_counts(seed):
    # partial states and items of a batch against a plain count
    shape = [W.LayerShape(256, 4, 2, 64, 256), W.LayerShape(256, 16, 1, 64, 256), W.LayerShape(256, 8, 8, 64, 256)][seed % 3]
    grp = shape.n_q_heads // shape.n_kv_heads
    b = W.batch_random(seed, n_prefill=3, n_decode=60, max_q=200, max_ctx=3000, n_roots=3)
    lay = binding.Layer(shape, device=-1)
    lay.set_chunk_pages(4)
    got = lay.attention_division(b, noalloc=False)
    path = {-1: (0, 0)}   # node -> pages, chunks up to and including it
    items = wide = states = 0
    for n in range(b.n_nodes):
        pages = int(b.node_page_start[n + 1] - b.node_page_start[n])
        above = path[int(b.node_parent[n])]
        path[n] = (above[0] + pages, above[1] + -(-pages // 4))
        cnt, most = int(b.node_seq_count[n]), max(1, 64 // grp)
        groups = -(-cnt // most)
        for g in range(groups):
            members = cnt * (g + 1) // groups - cnt * g // groups
            items += -(-pages // 4)
            wide += -(-pages // 4) * (members * grp > 16)
    for s in range(b.n_prefill, b.n_seq):
        pages, chunks = path[int(b.seq_leaf_node[s])]
        tail = -(-(-(-int(b.kv_len[s]) // 16) - pages) // 4)
        items += tail
        states += chunks + tail
    assert (got.items, got.wide_items, got.states) == (items, wide, states)
    blocks = sum(-(-int(q) // got.prefill_rows) for q in b.q_len()[:b.n_prefill])
    assert got.prefill_rows in ((64,) if grp % 4 == 0 else (64, 256 if grp % 2 else 128))
    assert got.descriptor_words == 4 * b.n_seq + 3 + 3 * b.n_rows + 2 * blocks + 8 * items + b.node_page_ids.size + b.page_ids.size


@pytest.mark.parametrize("shape", [W.LLAMA3_8B, W.LLAMA3_70B, W.LayerShape(256, 16, 1, 64, 256)])
@pytest.mark.parametrize("members,prefix_pages,tails", [(60, 450, 20), (8, 4, 40), (40, 64, 300), (50, 256, 20), (70, 80, 100), (100, 64, 60),
                                                        (200, 100, 20), (16, 128, 2000), (300, 40, 30)])
def test_both_attention_entry_points_divide_alike(shape, members, prefix_pages, tails):
    # from steps cut into short chunks, over those whose short chunks the scratch array of bs_attention_noalloc
    # does not hold, to large ones with nodes of more than 16 query rows; refusals follow the fixed division
    lay = binding.Layer(shape, device=-1)
    seqs = [(1, 16 * prefix_pages + tails + 3 * i, 0) for i in range(members)] + [(1, 7 + tails, -1)] * 3
    b = W.assemble_batch(16, seqs, 0, [(-1, prefix_pages)], None)
    grp = shape.n_q_heads // shape.n_kv_heads
    groups = -(-members // max(1, 64 // grp))
    chunk = 32 if -(-members // groups) * grp > 16 else 64
    states = members * -(-prefix_pages // chunk) + sum(-(-(-(-int(k) // 16) - prefix_pages) // 64) for k in b.kv_len[:members]) + \
        3 * -(-(7 + tails) // 1024)
    hq = shape.n_q_heads
    fits = (states * hq + 3) // 4 * 4 * 8 + states * hq * shape.head_dim * 4 <= 15 << 20
    if fits:
        assert _fields(lay.attention_division(b, noalloc=True)) == _fields(lay.attention_division(b))
    else:
        with pytest.raises(binding.BlendStepError, match="partial softmax states"):
            lay.attention_division(b, noalloc=True)


@pytest.mark.parametrize("heads,dh,segments,rows,cached,want", [
    ((32, 32), 128, 128, 16, 0, 64), ((32, 32), 64, 128, 64, 0, 64), ((24, 8), 128, 32, 64, 1000, 64), ((16, 8), 64, 128, 64, 500, 64),
    ((8, 8), 128, 8, 16, 500, 64), ((32, 32), 128, 4, 1024, 0, 256), ((8, 8), 64, 1, 64, 2000, 256), ((16, 8), 128, 1, 2048, 2000, 128),
    ((24, 8), 64, 4, 1024, 0, 256), ((32, 8), 128, 128, 16, 0, 64), ((32, 8), 64, 4, 1024, 0, 64)])
def test_prefill_kernel_by_chunks(heads, dh, segments, rows, cached, want):
    # group sizes that are no multiple of four: many short chunks go 64 rows to a workgroup (without the LDS
    # ring), long or few ones 256 (128) to a ring; each choice is the faster side of a timed pair
    lay = binding.Layer(W.LayerShape(256, heads[0], heads[1], dh, 256), device=-1)
    b = W.assemble_batch(16, [(rows, rows + cached, -1)] * segments, segments, [], None)
    assert lay.attention_division(b).prefill_rows == want


@pytest.mark.parametrize("shape,product,rows,want", [
    (W.LayerShape(1024, 16, 4, 64, 4096), "o", 359, (3, 2)), (W.LayerShape(1024, 16, 4, 64, 4096), "qkv", 300, (3, 2)),
    (W.LayerShape(2048, 32, 8, 64, 8192), "down", 1000, (1, 8)), (W.LLAMA3_70B, "qkv", 359, (1, 3)),
    (W.LLAMA3_8B, "down", 1580, (1, 2)), (W.LLAMA3_8B, "o", 5120, (2, 1)), (W.LLAMA3_70B, "down", 5120, (6, 1)),
    (W.LLAMA3_70B, "qkv", 2200, (1, 1)), (W.LLAMA3_70B, "o", 77, (4, 8)), (W.LLAMA3_8B, "o", 77, (3, 8)), (W.TINY, "o", 257, (3, 1))])
def test_gemm_division_narrow_short_and_large(shape, product, rows, want):
    # the measured best or within 5 % of it (QKV of 2200 rows of the 70B layer: 7.6 %, 192x256 tiles are not offered to it):
    # narrow and short products that a cost fitted to large ones left whole, long ones cut, and the products that stay whole
    assert binding.Layer(shape, device=-1).gemm_division(product, rows) == want


@pytest.mark.parametrize("shape,product,rows,shared", [
    # tiles beyond whole rounds no multiple of a quarter round: slower on shared tiles by 5 to 20 %, in a step or alone
    (W.LayerShape(4096, 32, 32, 128, 11008), "qkv", 5600, False), (W.LLAMA3_70B, "down", 3170, False), (W.LLAMA3_70B, "down", 4782, False),
    (W.LLAMA3_70B, "qkv", 3584, False), (W.LLAMA3_70B, "o", 6695, False), (W.LayerShape(5120, 40, 8, 128, 13824), "down", 7300, False),
    # a multiple of a quarter round: slower where there are many rounds of a short K, ahead where K is long
    (W.LayerShape(4096, 32, 32, 128, 11008), "qkv", 7012, False), (W.LLAMA3_70B, "down", 3535, False),
    (W.LayerShape(4096, 32, 32, 128, 11008), "qkv", 3072, False), (W.LayerShape(5120, 40, 8, 128, 13824), "down", 4029, True),
    (W.LLAMA3_70B, "qkv", 2048, True), (W.LLAMA3_70B, "down", 7012, True), (W.LLAMA3_70B, "qkv", 4096, True)])
def test_shared_tiles_where_they_are_the_faster_ones(shape, product, rows, shared):
    assert (binding.Layer(shape, device=-1).gemm_division(product, rows) == (6, 1)) == shared


@pytest.mark.parametrize("heads,n,tail,groups,pages,want", [
    ((24, 8), 287, 32, 6, 151, (32, 512)), ((32, 8), 640, 400, 4, 128, (400, 1024)),   # large steps: by rounds of the wide units
    ((32, 8), 20, 16, 2, 64, (16, 128)), ((64, 8), 105, 181, 6, 5, (181, 80)),        # few: cut; tails beside wide nodes stay whole
    ((32, 8), 7, 2000, 0, 0, (224, 0)), ((32, 8), 256, 1024, 0, 0, (1024, 0)), ((16, 8), 8, 3000, 2, 100, (416, 0))])
def test_chunks_of_decode_attention(heads, n, tail, groups, pages, want):
    lay = binding.Layer(W.LayerShape(256, heads[0], heads[1], 128, 256), device=-1)
    b = W.assemble_batch(16, [(1, tail + 16 * pages, i * groups // n if groups else -1) for i in range(n)], 0, [(-1, pages)] * groups, None)
    assert tuple(lay.attention_division(b).longest_item_tokens) == want


def test_a_setting_of_a_device_is_made_on_each_device(tmp_path):
    # kernels whose launches need more than 64 KB of LDS are allowed it per device: from two devices, again after
    # a failure, and from threads that race for it
    import subprocess
    src = tmp_path / "once.cpp"
    src.write_text("""
#include <cstdio>
#include <thread>
#include <vector>
#include "once.hpp"
int main() {
  bs::OncePerDevice once;
  int made[3] = {0, 0, 0};
  for (int turn = 0; turn < 3; ++turn)
    for (int d = 0; d < 2; ++d)
      if (once(d, [&] { ++made[d]; return 0; })) return 1;
  if (made[0] != 1 || made[1] != 1) return 2;
  if (once(2, [&] { ++made[2]; return 7; }) != 7 || once(2, [&] { ++made[2]; return 0; }) != 0 || made[2] != 2) return 3;
  if (once(64, [&] { return 5; }) != 5) return 4;
  bs::OncePerDevice shared;
  std::atomic<int> seen{0};
  std::vector<std::thread> threads;
  for (int t = 0; t < 8; ++t)
    threads.emplace_back([&] {
      std::atomic<bool> mine{false};
      for (int i = 0; i < 1000; ++i)
        if (shared(i % 48, [&] { mine = true; return 0; })) seen = -1000000;
      if (mine) ++seen;
    });
  for (auto &t : threads) t.join();
  return seen >= 1 ? 0 : 5;
}
""")
    csrc = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2411_16102_amd", "csrc")
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-pthread", "-I", csrc, "-o", str(tmp_path / "once"), str(src)])
    assert subprocess.call([str(tmp_path / "once")]) == 0


def test_first_k_tile_of_a_tile(tmp_path):
    # evaluated by the compiler, which refuses what is undefined: within the k-tiles there are, and 0 where K is empty
    import subprocess
    src = tmp_path / "k.cpp"
    src.write_text("""
#include "k_order.hpp"
using bs::first_k_tile;
constexpr bool inside(int k, int ldb) {
  for (int tile = 0; tile < 600; ++tile)
    if (first_k_tile(tile, k, ldb) < 0 || first_k_tile(tile, k, ldb) >= (k + 63) / 64) return false;
  return true;
}
static_assert(inside(4096, 4096) && inside(2048, 2048) && inside(64, 2048) && inside(14336, 14336) && inside(8, 8), "");
static_assert(first_k_tile(1, 4096, 4096) == 16 && first_k_tile(5, 4096, 4096) == 16 && first_k_tile(3, 2048, 2048) == 16, "");
static_assert(first_k_tile(3, 4160, 4160) == 0 && first_k_tile(3, 2000, 2048) == 0, "");
static_assert(first_k_tile(0, 0, 0) == 0 && first_k_tile(3, 0, 0) == 0 && first_k_tile(3, 0, 2048) == 0, "");
int main() {}
""")
    csrc = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2411_16102_amd", "csrc")
    r = subprocess.run(["g++", "-std=c++17", "-fsyntax-only", "-I", csrc, str(src)], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    assert r.returncode == 0, r.stdout


@pytest.mark.parametrize("segments", [1, 2, 3, 6, 12])
def test_cut_prefill_contexts_keep_to_the_scratch_array(segments):
    # both entry points cut alike, and never into more states than the array of bs_attention_noalloc holds beside its
    # descriptor; host only
    lay = binding.Layer(W.LLAMA3_8B, device=-1)
    for rows, cached in ((64, 8000), (700, 3000)):
        b = W.assemble_batch(16, [(rows, rows + cached, -1)] * segments + [(1, 300, -1)] * 5, segments, [], None)
        d = lay.attention_division(b)
        assert _fields(d) == _fields(lay.attention_division(b, noalloc=True))
        assert d.states * 32 * (128 + 2) * 4 <= (63 << 20) and d.descriptor_words <= NOALLOC_WORDS
        if segments == 1:
            assert d.states > 5 * 3


@pytest.mark.parametrize("chunks,cut", [
    ([(909, 909), (1145, 1145)], False), ([(3662, 3746)], False), ([(n, n) for n in (332, 300, 274, 174, 80, 529, 258, 299, 1000, 147, 535)], False),
    ([(n, n) for n in (246, 646, 350, 1057, 455, 395, 418)], False),
    ([(32, 2000)], True), ([(134, 1362), (150, 843), (142, 2990)], True)])
def test_contexts_of_64_wide_heads_are_cut_where_that_is_shorter(chunks, cut):
    # many rows of 64-wide heads: 8 to 12 % slower cut, 8 heads in 32 query heads; few rows behind long contexts: 1.6 times as fast
    # and more
    b = W.assemble_batch(16, [(q, n, -1) for q, n in chunks], len(chunks), [], None)
    assert (binding.Layer(W.LayerShape(2048, 32, 8, 64, 8192), device=-1).attention_division(b).states > 0) == cut


@pytest.mark.parametrize("want,held,captured_words,capturing,free,got", [
    # want / held / got: states of cut contexts and descriptor words (the descriptor without cuts has 90); free: states that
    # the device has room for
    ((64, 120), (0, 100), 500, True, 0, (0, 90)),         # captured on a context without states: whole
    ((64, 120), (64, 128), 500, True, 0, (64, 120)),      # ... that holds them: cut as outside capture
    ((64, 120), (64, 100), 500, True, 0, (32, 100)),      # ... whose descriptor buffer is too short for that many
    ((64, 120), (64, 128), 100, True, 0, (32, 100)),      # ... whose ring of captured descriptors is
    ((64, 120), (0, 128), 500, False, 64, (64, 120)),     # outside capture the states grow
    ((64, 120), (0, 128), 500, False, 63, (0, 90)),       # ... and what the device has no room for stays whole
    ((64, 120), (0, 100), 500, False, 64, (64, 120)),     # ... and the descriptor's buffer, also where it would do without the cut
    ((64, 120), (64, 100), 500, False, 64, (64, 120)),
    ((64, 120), (64, 100), 500, False, 0, (0, 90)),
    ((64, 120), (64, 128), 100, False, 0, (64, 120)),     # the ring is for captured calls
    ((0, 90), (0, 0), 0, True, 0, (0, 90))])              # nothing to cut: nothing is asked
def test_what_a_call_cuts_into(tmp_path, want, held, captured_words, capturing, free, got):
    import subprocess
    src = tmp_path / "room.cpp"
    src.write_text("""
#include <cstdio>
#include "room.hpp"
struct Ops {
  long ws, ww, hs, hw, cw, free_slots;
  bool cap;
  long s = 0, w = 0;
  bool grew = false, asked = false, room = false;
  int build(bs::CutRoom r) {  // half of the cuts where all of them do not fit
    s = ws; w = ww;
    if (s > r.slots || w > r.words) { s = ws / 2; w = 100; }
    if (s > r.slots || w > r.words) { s = 0; w = 90; }
    return 0;
  }
  long slots() const { return s; }
  long words() const { return w; }
  long held_slots() const { return hs; }
  long held_words() const { return hw; }
  long captured_words() const { return cw; }
  bool capturing() { asked = true; return cap; }
  bool grow(long n, long words) { grew = true; return room = n <= free_slots && words == ww; }
};
int main() {
  Ops o{%d, %d, %d, %d, %d, %d, %s};
  if (bs::plan_within(o)) return 1;
  std::printf("%%ld %%ld %%d %%d", o.s, o.w, o.cap && o.grew, (o.asked && o.ws == 0) || (!o.cap && o.s > o.hs && !o.room));
}
""" % (*want, *held, captured_words, free, "true" if capturing else "false"))
    csrc = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2411_16102_amd", "csrc")
    subprocess.check_call(["g++", "-std=c++17", "-I", csrc, str(src), "-o", str(tmp_path / "room")])
    out = subprocess.check_output([str(tmp_path / "room")], text=True).split()
    assert out == [str(got[0]), str(got[1]), "0", "0"]


@pytest.mark.parametrize("rows,tiles", [(2606, 10), (4100, 10), (3300, 10), (5140, 1)])
def test_gate_up_on_one_shape_where_a_second_would_cost_more(rows, tiles):
    # K = 1024, 2 x 4096 columns: two shapes for an expected gain of 2 to 3 us take 3 to 5 us longer than the one shape (2606 and
    # 4100 rows: whole 192x256 tiles, not 160x256 ones first); an expected 4 us and more than
    # 3 % beside that cost pays
    assert binding.Layer(W.LayerShape(1024, 4, 2, 64, 4096), device=-1).gemm_division("gate_up", rows)[0] == tiles
