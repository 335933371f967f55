"""Row statistics at the edges of the register frames (4 to 64 values per thread) and of their 4096-entry chunks: rows that
fill a frame exactly, rows one vector longer or shorter, and top-k at both ends.  Maximum and k-th largest are selections
of the kernel's own logits and must be exact; the log-sum-exp adds at most 65536 float32 exponentials whose relative
errors (a few 2^-24 each, all of one sign at worst) and summation stay below 1e-5 of the sum."""
import pytest
import torch

from paper_2605_07230_amd import binding

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("vocab", [4, 4096, 4100, 8192, 8196, 12292, 16384, 16388, 24576, 24580, 32768, 33088, 40956, 40964, 49152, 49156, 61444, 65532, 65536])
@pytest.mark.parametrize("law", ["normal", "equal_tail"])
def test_row_statistics_frames(vocab, law):
    n, hidden = 3, 4
    print(f"[row stats] vocab={vocab} {law}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(vocab)
    w = torch.randn(vocab, hidden, device="cuda", generator=gen)
    if law == "equal_tail":
        w[vocab // 2:] = w[0]            # thousands of ties, up to the very end of the row
    h = torch.randn(n, hidden, device="cuda", generator=gen)
    ctx = binding.Context(max_rows=1, max_nodes_total=n, max_nodes_per_tree=1, max_prefix=0, n_heads=1, head_dim=64, hidden=hidden, vocab=vocab)
    logits = torch.empty(n, vocab, device="cuda")
    mx, thr, lse = (torch.full((n,), float("nan"), device="cuda") for _ in range(3))
    for k in sorted({1, min(50, vocab), min(2000, vocab), max(1, vocab - 1), vocab}):
        binding.lmhead_softmax_cfg(ctx, h_cond=h, h_uncond=None, w=w, cfg_scale=1.0, temperature=1.0, top_k=k, logits=logits, row_max=mx,
                                   row_thr=thr, row_lse=lse)
        kth = torch.topk(logits, k, dim=1).values[:, -1] if k < vocab else torch.full((n,), -float("inf"), device="cuda")
        assert torch.equal(mx, logits.max(1).values) and torch.equal(thr, kth), (k, thr.tolist(), kth.tolist())
        g = logits.double()
        ref = torch.logsumexp(g.masked_fill(g < kth.double()[:, None], -float("inf")), 1)
        assert torch.all((lse.double() - ref).abs() <= 1e-5 + 2.0 ** -23 * ref.abs()), (k, lse.tolist(), ref.tolist())
