"""What the GPU tests' sizes reach: every kernel instance that the launch rules can choose is run by a test that compares
its results (no GPU: the rules are host code and are asked through the library)."""
import pytest

import test_gpu_attention_cuts as cuts
import test_gpu_projection_tiles as tiles
from paper_2605_07230_amd import binding


def _tiles(n, vocab, hidden, mode, packed):
    return binding.projection_tiles(n_nodes=n, hidden=hidden, vocab=vocab, guided=mode != "plain",
                                    w_layout=binding.W_PACKED32 if packed else binding.W_ROWMAJOR,
                                    cfg_mix=binding.CFG_MIX_HIDDEN if mode == "mixed" else binding.CFG_MIX_LOGITS)


def _streams(n, vocab, hidden, mode, packed):
    return binding.projection_streams(n_nodes=n, hidden=hidden, vocab=vocab, guided=mode != "plain",
                                      w_layout=binding.W_PACKED32 if packed else binding.W_ROWMAJOR,
                                      cfg_mix=binding.CFG_MIX_HIDDEN if mode == "mixed" else binding.CFG_MIX_LOGITS)


def _marked(test, names):
    return next(m.args[1] for m in test.pytestmark if m.name == "parametrize" and m.args[0] == names)


def test_every_projection_kernel_is_tested():
    reached = set()     # (tile, rows in pairs, packed weights)
    sizes = [(max(1, r // 2) if mode == "pairs" else r, v, h, mode, packed)
             for r, v, h in tiles.SHAPES for mode in ("plain", "pairs", "mixed") for packed in (True, False)]
    sizes += [(n, v, 2048, mode, packed) for n, v, mode, packed, _ in tiles.SPLITS]
    sizes += [(n, v, h, mode, True) for n, v, h, mode, _ in _marked(tiles.test_large_tiles_short_hidden, "n,vocab,hidden,mode,tile")]
    for n, vocab, hidden, mode, packed in sizes:
        tile, rest, _ = _tiles(n, vocab, hidden, mode, packed)
        pairs = mode == "pairs" or (mode == "mixed" and not packed)
        reached |= {(tile, pairs, packed), (rest, pairs, packed)}
    assert reached == {(t, c, p) for t in range(5) for c in (False, True) for p in (False, True)} | {(5, False, True), (6, False, True), (6, True, True)}


def test_both_ways_of_loading_weights_are_tested_in_every_tile():
    reached = set()     # (tile, rows in pairs, packed weights, streamed)
    for shapes in (tiles.SHAPES, tiles.STREAMED):
        for r, vocab, hidden in shapes:
            for mode in ("plain", "pairs", "mixed"):
                for packed in (True, False):
                    n = max(1, r // 2) if mode == "pairs" else r
                    pairs = mode == "pairs" or (mode == "mixed" and not packed)
                    used = zip(_tiles(n, vocab, hidden, mode, packed)[:2], _streams(n, vocab, hidden, mode, packed))
                    reached |= {(tile, pairs, packed, streamed) for tile, streamed in used}
    ring = {(t, c, p, s) for t in range(5) for c in (False, True) for p in (False, True) for s in (False, True)}
    assert ring <= reached and {s for t, _, _, s in reached if t == 5} == {True, False} and {s for t, _, _, s in reached if t == 6} <= {False}


@pytest.mark.parametrize("rows", [1, 33, 64])
@pytest.mark.parametrize("vocab", [63552, 65536])
@pytest.mark.parametrize("hidden", [3072, 4096, 5120])
def test_few_mixed_rows_are_cut_like_plain_ones(rows, vocab, hidden):
    """Up to 64 rows, mixed or not, fill one row tile of 64: what their weights divide into does not lead past the costs of the tiles."""
    assert _tiles(rows, vocab, hidden, "mixed", True) == _tiles(rows, vocab, hidden, "plain", True) == (2, 2, vocab)


@pytest.mark.parametrize("head_dim", [64, 128])
def test_every_attention_cut_is_tested(head_dim):
    reached, loads = set(), set()
    for name, (kv_heads, group, sizes, prefix) in cuts.CASES.items():
        cut = binding.attention_cut(n_rows=len(sizes), n_nodes_total=sum(sizes), max_nodes_per_tree=max(sizes), max_prefix_len=max(prefix),
                                    n_heads=kv_heads * group, n_kv_heads=kv_heads, head_dim=head_dim)
        assert cut == cuts.CUTS[name][head_dim == 128], name
        reached.add((cut[0], cut[1] > 1))
        loads.add((cut[0], cut[1] == 1 and max(sizes) * group <= cut[0]))    # one block and one part: the prefix is streamed
    assert {r for r, _ in reached} == {16, 64, 80, 96, 128, 256} and {(64, True), (64, False), (128, True), (128, False)} <= reached
    assert {(rows, streamed) for rows in (64, 80, 96, 128) for streamed in (True, False)} <= loads


def test_queries_refuse_what_they_do_not_describe():
    lib, n = binding.load_library(), binding.C.c_int32()
    a, b = binding.tree_attn_args(), binding.lmhead_args()
    assert lib.cascade_attention_cut(None, a, n, n) == binding.EDTYPE and lib.cascade_projection_tiles(None, b, n, n, n) == binding.EDTYPE
    a.dtype = b.dtype = binding.BF16
    assert lib.cascade_attention_cut(None, a, n, n) == binding.EINVAL and lib.cascade_projection_tiles(None, b, n, n, n) == binding.EINVAL
    assert lib.cascade_projection_streams(None, b, n, n) == binding.EINVAL and lib.cascade_projection_streams(None, None, n, n) == binding.EINVAL
    assert lib.cascade_attention_cut(None, None, n, n) == binding.EINVAL and lib.cascade_projection_tiles(None, None, n, n, n) == binding.EINVAL
