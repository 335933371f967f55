"""Acceptance on wide rows that several workgroups share: around the widths at which there are more parts (8192 elements: four of
floats, two of bf16, 16384: four, 32768: eight) and the node counts that limit them (256, 128, 64), widths whose last part is
short, rows that 16-byte loads cannot read, nodes beside each other that meet and that are done by one workgroup (one sweep of
less than 16384 elements); called on one context with other widths in turn (the counters of arrival are zero between calls).
Gram tiles beside them, at hidden sizes of one and several steps per wave.
Cosines are off by at most (h + 16) 2^-24, as in test_gpu_accept_widths; bf16 products are exact in float32, their sums are not."""
import numpy as np
import pytest
import torch

import test_gpu_accept_widths as widths
from oracle import verify_oracle as vo
from paper_2605_07230_amd import binding
from paper_2605_07230_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,hidden", [("f32", 4096), ("f32", 6001), ("f32", 8188), ("f32", 8192), ("f32", 8193), ("f32", 16380), ("f32", 16384),
                                          ("f32", 16388), ("f32", 33000), ("bf16", 8184), ("bf16", 8200), ("bf16", 16392), ("bf16", 32776)])
@pytest.mark.parametrize("kids", [1, 4, 8, 31, 60])
def test_wide_rows(dtype, hidden, kids):
    widths.test_acceptance_on_generic_rows(dtype, hidden, kids)


def _call(trees, features, dtype, repeats):
    """Calls of one context, the feature rows of every width in turn."""
    off = np.concatenate([[0], np.cumsum([len(t) for t in trees])]).astype(np.int32)
    n, vocab, rng = int(off[-1]), 128, np.random.default_rng(1)
    parent, token = np.concatenate(trees).astype(np.int32), rng.integers(0, vocab, n).astype(np.int32)
    logits = rng.standard_normal((n, vocab)).astype(np.float32)
    thr, lse = np.full(n, -np.inf, np.float32), np.log(np.exp(logits.astype(np.float64)).sum(1)).astype(np.float32)
    accs = [vo.cascade_accept(off, parent, token, h, logits.astype(np.float64), thr.astype(np.float64), lse.astype(np.float64), 0.9, 0.9) for h in features]
    assert min(acc.min_cos_margin for acc in accs) > 1e-3
    dev = lambda x: torch.from_numpy(x).cuda()  # noqa: E731
    ctx = binding.Context(max_rows=len(trees), max_nodes_total=n, max_nodes_per_tree=max(map(len, trees)), max_prefix=0, n_heads=1, head_dim=64,
                          hidden=max(h.shape[1] for h in features), vocab=vocab)
    rows = [dev(h) if dtype == "f32" else dev(h).bfloat16() for h in features]
    for _ in range(repeats):
        for h, acc in zip(rows, accs):
            f = {k: torch.full((n,), float("nan"), device="cuda") for k in ("q_tok", "m_int", "m_conv", "cos_parent")}
            i = {k: torch.full((n,), -7, dtype=torch.int32, device="cuda") for k in ("n_int", "n_conv")}
            binding.cascade_accept(ctx, node_off=dev(off), parent=dev(parent), token=dev(token), h_cond=h, logits=dev(logits), row_thr=dev(thr),
                                   row_lse=dev(lse), tau_pos=0.9, tau_seq=0.9, **f, **i)
            np.testing.assert_array_equal(i["n_int"].cpu().numpy(), acc.n_int)
            np.testing.assert_array_equal(i["n_conv"].cpu().numpy(), acc.n_conv)
            np.testing.assert_allclose(f["cos_parent"].cpu().numpy(), acc.cos_parent, rtol=0, atol=(h.shape[1] + 16) * 2.0 ** -24)
    assert ctx.device_status() == binding.OK


def _rows(rng, trees, hidden, dtype):
    """Near-duplicates (cosine 0.98) of the parent or the node before, and strangers."""
    rows = []
    for t in trees:
        h = rng.standard_normal((len(t), hidden)).astype(np.float32)
        for i in range(1, len(t)):
            if i % 3:
                h[i] = h[t[i] if i % 2 else i - 1] + 0.2 * h[i]
        rows.append(h)
    h = np.concatenate(rows)
    return wl.round_bf16(h) if dtype == "bf16" else h


@pytest.mark.parametrize("nodes", [40, 44, 45, 108, 109, 236, 237])    # with the two small trees 60 to 257 nodes: up to eight parts, four from 65 on, two from 129, one from 257
def test_repeated_calls_on_ragged_trees(nodes):
    rng = np.random.default_rng(nodes)
    trees = [wl.grow_tree(rng, n, d) for n, d in ((nodes, 6), (3, 2), (17, 4))]
    print(f"[accept] f32, {nodes} + 20 nodes, widths in turn", flush=True)
    _call(trees, [_rows(rng, trees, hidden, "f32") for hidden in (33000, 8192, 4096, 16384, 12000)], "f32", 2)


@pytest.mark.parametrize("hidden", [128, 256, 384, 1152, 2176, 4096])
@pytest.mark.parametrize("nodes", [30, 129])
def test_gram_tiles_over_the_waves(hidden, nodes):
    rng = np.random.default_rng(hidden + nodes)
    trees = [wl.grow_tree(rng, nodes, 6) for _ in range(2)]
    print(f"[accept] bf16 hidden={hidden} nodes={2 * nodes}", flush=True)
    h = _rows(rng, trees, max(hidden, 512), "bf16")[:, :hidden] if hidden >= 512 else _rows(rng, trees, hidden, "bf16")
    _call(trees, [np.ascontiguousarray(h)], "bf16", 2)
