"""Row statistics of long rows, where a sample of the row (the first load of each of the sixteen waves, 256 entries each) tells which
entries are looked at: samples that promise too many entries, none of the largest ones, only equal ones, -inf, and rows that end inside a
chunk.  Bounds are those of test_gpu_row_stats_frames."""
import pytest
import torch

from paper_2605_07230_amd import binding

pytestmark = pytest.mark.gpu


def _sampled(vocab):
    """Entries of the sample: wave w begins with its 256 entries of chunk w / 16 of the whole 4096-entry ones."""
    full = vocab // 4096
    return torch.cat([torch.arange(256) + ((w * full) // 16 * 16 + w) * 256 for w in range(16)]).cuda()


@pytest.mark.parametrize("vocab", [33088, 45060, 57344, 65532, 65536])
@pytest.mark.parametrize("law", ["sample_high", "sample_low", "sample_equal", "outside_masked", "sample_masked", "normal"])
def test_rows_whose_sample_misleads(vocab, law):
    n = 130
    print(f"[row stats] vocab={vocab} {law}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(vocab)
    row = torch.randn(vocab, device="cuda", generator=gen)
    at = _sampled(vocab)
    rest = torch.ones(vocab, dtype=torch.bool, device="cuda")
    rest[at] = False
    if law == "sample_high":
        row[at] += 20.0
    elif law == "sample_low":
        row[at] -= 20.0
    elif law == "sample_equal":
        row[at] = 0.5
    elif law == "outside_masked":
        row[rest] = -float("inf")
    elif law == "sample_masked":
        row[at] = -float("inf")
    scale = torch.linspace(0.5, 2.0, n, device="cuda")
    ctx = binding.Context(max_rows=1, max_nodes_total=n, max_nodes_per_tree=1, max_prefix=0, n_heads=1, head_dim=64, hidden=1, vocab=vocab)
    logits = torch.empty(n, vocab, device="cuda")
    mx, thr, lse = (torch.full((n,), float("nan"), device="cuda") for _ in range(3))
    for k in (1, 50, 2000, 3000, 4100):
        binding.lmhead_softmax_cfg(ctx, h_cond=scale[:, None].contiguous(), h_uncond=None, w=row[:, None].contiguous(), cfg_scale=1.0, temperature=1.0,
                                   top_k=k, logits=logits, row_max=mx, row_thr=thr, row_lse=lse)
        kth = torch.topk(logits, k, dim=1).values[:, -1]
        assert torch.equal(mx, logits.max(1).values) and torch.equal(thr, kth), k
        g = logits.double()
        ref = torch.logsumexp(g.masked_fill(g < kth.double()[:, None], -float("inf")), 1)
        assert torch.all((lse.double() - ref).abs() <= 1e-5 + 2.0 ** -23 * ref.abs()), k
