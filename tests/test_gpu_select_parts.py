"""Path selection with the vocabulary of a prompt dealt to several workgroups: rows around the 4096-entry passes, the most
prompts that still share a row and the first count that does not, repeated calls on one context (the counters of arrival are
zero between calls), and rows of which every kept entry was removed (the workgroup that finishes sums them again by itself).
Bounds and margins are those of test_gpu_select_edges."""
import numpy as np
import pytest
import torch

import test_gpu_select_edges as edges
from oracle import verify_oracle as vo
from paper_2605_07230_amd import binding

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", [binding.WALK_SEQUENTIAL, binding.WALK_LONGEST])
@pytest.mark.parametrize("vocab", [4095, 4096, 4097, 4100, 8192, 8196, 33088, 61444])
def test_passes_of_a_row(vocab, mode):
    sizes = (40, 3, 65)
    inp, ref = next(r for r in (edges._inputs(vocab, sizes, True, mode, seed) for seed in range(40)) if r is not None)
    print(f"[select] vocab={vocab} mode={mode}", flush=True)
    edges._check(inp, ref, vocab, sizes, mode)


@pytest.mark.parametrize("prompts", [127, 128, 129])    # 4 workgroups of a prompt, 4, 1
@pytest.mark.parametrize("vocab", [16384, 16388, 20000, 24580, 33088, 65532])    # alone, passes x chunks per wave: 1 x 8, 2 x 6, 2 x 6, 2 x 8, 3 x 6, 4 x 8
def test_many_prompts(prompts, vocab):
    sizes = (3,) * prompts
    inp, ref = next(r for r in (edges._inputs(vocab, sizes, False, binding.WALK_SEQUENTIAL, seed) for seed in range(40)) if r is not None)
    print(f"[select] prompts={prompts} vocab={vocab}", flush=True)
    edges._check(inp, ref, vocab, sizes, binding.WALK_SEQUENTIAL)


@pytest.mark.parametrize("vocab", [4096, 20000, 65536])
def test_repeated_calls_and_rows_with_nothing_left(vocab):
    rng = np.random.default_rng(vocab)
    B, n = 5, 4                                   # a root and three children each, all rejected
    off, parent = (n * np.arange(B + 1)).astype(np.int32), np.tile(np.array([-1, 0, 0, 0], np.int32), B)
    token = np.stack([rng.choice(vocab, n, replace=False) for _ in range(B)]).astype(np.int32).reshape(-1)
    g = rng.standard_normal((B * n, vocab)).astype(np.float32)
    thr = np.full(B * n, 20.0, np.float32)
    for b in range(B):                            # only the children's tokens are kept, except in prompt 2
        g[n * b, token[n * b + 1:n * b + n]] = 21.0
    thr[2 * n] = -np.inf
    lse = np.log(np.where(g >= thr[:, None], np.exp(g.astype(np.float64)), 0).sum(1) + 1e-30).astype(np.float32)
    z = np.zeros(B * n, np.float32)
    acc = vo.AcceptScalars(q_tok=z, m_int=z, m_conv=z, n_int=z.astype(np.int32), n_conv=z.astype(np.int32), cos_parent=z, min_cos_margin=1.0)
    u, ub = np.full(B * n, 0.5, np.float32), np.array([0.1, 0.4, 0.6, 0.9, 0.5], np.float32)
    ref = vo.select_path(off, parent, token, acc, None, u, ub, 0.1, g, thr, lse, 3, binding.WALK_SEQUENTIAL)
    assert (ref.accept_len == 0).all() and ref.min_margin > edges.MARGIN / 100
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()  # noqa: E731
    ctx = binding.Context(max_rows=B, max_nodes_total=B * n, max_nodes_per_tree=n, max_prefix=0, n_heads=1, head_dim=64, hidden=128, vocab=vocab)
    kw = dict(node_off=dev(off), parent=dev(parent), token=dev(token), q_tok=dev(z), m_int=dev(z), m_conv=dev(z), n_int=dev(acc.n_int),
              n_conv=dev(acc.n_conv), draft_prob=None, u=dev(u), u_bonus=dev(ub), eps_tvd=0.1, logits=dev(g), row_thr=dev(thr), row_lse=dev(lse),
              max_depth=3, mode=binding.WALK_SEQUENTIAL)
    for _ in range(4):
        out = {k: torch.full(s, -7, dtype=torch.int32, device="cuda") for k, s in dict(accept_len=(B,), path_nodes=(B, 3), emitted=(B, 4), terminal=(B,)).items()}
        binding.select_path(ctx, tvd_used=torch.empty(B, device="cuda"), **out, **kw)
        for k, got in out.items():
            assert np.array_equal(got.cpu().numpy(), getattr(ref, k)), (k, got.cpu().numpy(), getattr(ref, k))
