"""Every tile of the bf16 projection at its edges (ragged last row and column tiles, one- and two-stage hidden sizes,
guidance pairs, packed and row-major weights) against the same product in float64.

Bound: the kernels sum K exact bf16 products in float32 in some order, so an element is off by at most
K 2^-24 sum |h| |w| (and the guidance mix adds its own two roundings, which the same bound covers with the factor of
the mix applied to |h|); rows mixed before the product carry one bf16 rounding (2^-8 of the element) in addition."""
import pytest
import torch

from paper_2605_07230_amd import binding

pytestmark = pytest.mark.gpu

# rows of the product, vocabulary, hidden: the tile that 256 compute units choose for plain rows (mixed rows and row-major
# weights may take a neighbour; tests/test_dispatch.py counts what these lists reach)
SHAPES = [
    (1, 64, 128), (33, 16384, 128), (64, 16320, 384),          # 64 x 64
    (65, 16384, 256), (127, 16320, 640),                       # 128 x 64
    (3, 65536, 256), (64, 33088, 384), (120, 65472, 128),      # 64 x 256, the last column tile ragged
    (129, 16384, 256), (230, 16320, 384),                      # 128 x 128
    (257, 16384, 256), (700, 33088, 256), (256, 65472, 128),   # 256 x 128 (mixed rows: 128 x 256)
    (490, 16448, 128), (513, 33088, 256),                      # 128 x 128 again: whole rounds
]


@pytest.mark.parametrize("rows,vocab,hidden", SHAPES)
@pytest.mark.parametrize("mode", ["plain", "pairs", "mixed"])
@pytest.mark.parametrize("packed", [True, False])
def test_projection_tiles(rows, vocab, hidden, mode, packed):
    _check(max(1, rows // 2) if mode == "pairs" else rows, vocab, hidden, mode, packed)


# the same with weights that are loaded past the caches (85 MiB and more, at most two row tiles): every tile of the ring kernel, for
# pairs or not, packed or row-major weights, and 128 x 256 (mixed rows; tests/test_dispatch.py counts these too)
STREAMED = [(33, 16384, 2816), (61, 16384, 2816), (120, 16384, 2816), (60, 65472, 768), (200, 16448, 2816), (200, 65472, 768), (300, 16384, 2816)]


@pytest.mark.parametrize("rows,vocab,hidden", STREAMED)
@pytest.mark.parametrize("mode", ["plain", "pairs", "mixed"])
@pytest.mark.parametrize("packed", [True, False])
def test_projection_tiles_with_streamed_weights(rows, vocab, hidden, mode, packed):
    _check(max(1, rows // 2) if mode == "pairs" else rows, vocab, hidden, mode, packed)


# the large tiles, with one row in the last of them, at hidden sizes of one, three and five rounds of their rings (and the
# 256 x 128 ring tile at as many): nodes, vocabulary, hidden, mode, tile
@pytest.mark.parametrize("n,vocab,hidden,mode,tile", [
    (129, 24576, 128, "plain", 4), (129, 24576, 384, "plain", 4), (129, 24576, 640, "plain", 4),
    (257, 16448, 128, "mixed", 5), (257, 16448, 384, "mixed", 5), (257, 16448, 640, "mixed", 5),
    (257, 24576, 128, "mixed", 6), (257, 24576, 384, "mixed", 6), (257, 24576, 640, "mixed", 6), (257, 65536, 384, "plain", 6),
    (513, 49152, 128, "pairs", 6), (257, 33024, 384, "pairs", 6), (257, 33024, 640, "pairs", 6),
])
def test_large_tiles_short_hidden(n, vocab, hidden, mode, tile):
    _check(n, vocab, hidden, mode, True, tiles=(tile, tile))


# columns cut into whole rounds of one tile and a rest in another (tiles by number, as the launcher counts them)
SPLITS = [
    (65, 33024, "plain", True, (3, 0)), (200, 33024, "plain", True, (4, 0)), (257, 33088, "plain", True, (5, 2)), (461, 24000, "plain", True, (4, 3)),
    (600, 33024, "plain", True, (6, 5)), (343, 24000, "plain", True, (5, 0)),
    (257, 33088, "mixed", True, (5, 2)), (200, 41024, "mixed", True, (5, 3)), (600, 41024, "mixed", True, (5, 1)), (257, 33024, "mixed", True, (6, 0)),
    (65, 33024, "pairs", True, (2, 3)), (343, 24000, "pairs", True, (4, 1)), (300, 33024, "pairs", True, (6, 3)), (461, 33024, "pairs", True, (6, 0)),
    (65, 33024, "pairs", False, (2, 3)), (100, 33024, "pairs", False, (4, 0)), (200, 41024, "pairs", False, (4, 2)),
]


@pytest.mark.parametrize("n,vocab,mode,packed,tiles", SPLITS)
def test_projection_split_columns(n, vocab, mode, packed, tiles):
    _check(n, vocab, 2048, mode, packed, tiles=tiles)


# buffers that start 2, 8 and 14 bytes past a 16-byte boundary: sizes that take one ring tile, two, packed rows, and both
@pytest.mark.parametrize("n,vocab,hidden", [(1, 64, 128), (60, 4096, 384), (200, 16448, 128), (257, 33088, 256), (520, 16384, 128)])
@pytest.mark.parametrize("mode", ["plain", "pairs", "mixed"])
@pytest.mark.parametrize("packed", [True, False])
@pytest.mark.parametrize("shift_h,shift_w", [(1, 0), (0, 4), (7, 1)])
def test_projection_of_buffers_off_the_16_byte_grid(n, vocab, hidden, mode, packed, shift_h, shift_w):
    _check(n, vocab, hidden, mode, packed, shift_h, shift_w)


def _shifted(x, elements):
    y = torch.empty(x.numel() + 8, dtype=x.dtype, device=x.device)[elements:elements + x.numel()].view(x.shape)
    return y.copy_(x)


def _check(n, vocab, hidden, mode, packed, shift_h=0, shift_w=0, tiles=None):
    print(f"[projection] nodes={n} vocab={vocab} hidden={hidden} {mode} packed={packed} shift={shift_h},{shift_w}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(n * 131 + vocab + hidden)
    w = (0.02 * torch.randn(vocab, hidden, device="cuda", generator=gen)).bfloat16()
    c = torch.randn(n, hidden, device="cuda", generator=gen).bfloat16()
    u = (c.float() + 0.5 * torch.randn(n, hidden, device="cuda", generator=gen)).bfloat16()
    ctx = binding.Context(max_rows=1, max_nodes_total=n, max_nodes_per_tree=1, max_prefix=0, n_heads=1, head_dim=64, hidden=hidden, vocab=vocab)
    if tiles:
        got = binding.projection_tiles(n_nodes=n, hidden=hidden, vocab=vocab, guided=mode != "plain", ctx=ctx,
                                       w_layout=binding.W_PACKED32 if packed else binding.W_ROWMAJOR,
                                       cfg_mix=binding.CFG_MIX_HIDDEN if mode == "mixed" else binding.CFG_MIX_LOGITS)
        assert got[:2] == tiles and (got[2] == vocab) == (tiles[0] == tiles[1])
    logits = torch.full((n, vocab), float("nan"), device="cuda")
    stats = [torch.empty(n, device="cuda") for _ in range(3)]
    s, temp = 3.0, 0.8
    wp = binding.cascade_pack_lmhead_w(ctx, w) if packed else w
    if shift_h or shift_w:
        c, u, wp = _shifted(c, shift_h), _shifted(u, shift_h), _shifted(wp, shift_w)
        assert c.data_ptr() % 16 == 2 * shift_h and wp.data_ptr() % 16 == 2 * shift_w
    binding.lmhead_softmax_cfg(ctx, h_cond=c, h_uncond=None if mode == "plain" else u, w=wp,
                               w_layout=binding.W_PACKED32 if packed else binding.W_ROWMAJOR, cfg_scale=s, temperature=temp, top_k=50,
                               logits=logits, row_max=stats[0], row_thr=stats[1], row_lse=stats[2],
                               cfg_mix=binding.CFG_MIX_HIDDEN if mode == "mixed" else binding.CFG_MIX_LOGITS)
    cd, ud = c.double(), u.double()
    x = cd if mode == "plain" else ud + s * (cd - ud)
    mag = cd.abs() if mode == "plain" else ud.abs() + s * (cd.abs() + ud.abs())
    ref, bound = x @ w.double().t() / temp, hidden * 2.0 ** -24 * (mag @ w.double().abs().t()) / temp
    if mode == "mixed" and packed:
        bound = bound + 2.0 ** -8 * (x.abs() @ w.double().abs().t()) / temp
    bad = ~((logits.double() - ref).abs() <= bound + 1e-6)      # NaN (an unwritten element) is bad
    assert not bad.any(), (int(bad.sum()), torch.nonzero(bad)[0].tolist())
    assert torch.equal(stats[0], logits.max(1).values)


# one size per tile; a 256 x 256 tile (more rows) sums in one chain
@pytest.mark.parametrize("rows,vocab,tile", [(60, 16384, 0), (120, 16384, 1), (60, 65536, 2), (230, 16384, 3), (250, 32768, 4), (250, 65536, 5)])
def test_projection_sums_in_four_chains(rows, vocab, tile):
    """2-norm distance from float64.  A chain of n accumulations whose partial sums grow as a random walk rounds with an
    rms of at most 2^-24 / sqrt(3) of each partial sum: sqrt(n / 2) / sqrt(3) 2^-24 of the result, n = K / 16 / 4; an
    undivided chain of the same terms measures twice that."""
    print(f"[projection chains] rows={rows} vocab={vocab}", flush=True)
    hidden = 4096
    gen = torch.Generator(device="cuda")
    gen.manual_seed(rows + vocab)
    w = (0.02 * torch.randn(vocab, hidden, device="cuda", generator=gen)).bfloat16()
    c = torch.randn(rows, hidden, device="cuda", generator=gen).bfloat16()
    ctx = binding.Context(max_rows=1, max_nodes_total=rows, max_nodes_per_tree=1, max_prefix=0, n_heads=1, head_dim=64, hidden=hidden, vocab=vocab)
    assert binding.projection_tiles(n_nodes=rows, hidden=hidden, vocab=vocab, guided=False, w_layout=binding.W_PACKED32, ctx=ctx) == (tile, tile, vocab)
    logits = torch.empty(rows, vocab, device="cuda")
    stats = [torch.empty(rows, device="cuda") for _ in range(3)]
    binding.lmhead_softmax_cfg(ctx, h_cond=c, h_uncond=None, w=binding.cascade_pack_lmhead_w(ctx, w), w_layout=binding.W_PACKED32, cfg_scale=1.0,
                               temperature=1.0, top_k=50, logits=logits, row_max=stats[0], row_thr=stats[1], row_lse=stats[2])
    num = den = 0.0
    for v in range(0, vocab, 8192):
        ref = c.double() @ w[v:v + 8192].double().t()
        num += float(((logits[:, v:v + 8192].double() - ref) ** 2).sum())
        den += float((ref ** 2).sum())
    assert (num / den) ** 0.5 <= (hidden / 64 / 6) ** 0.5 * 2.0 ** -24
