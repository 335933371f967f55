"""Row statistics of more rows than compute units: two rows on each at a time, in workgroups of 512 threads.  Rows at the edges
of those frames (8 to 48 values per thread) and of their 2048-entry chunks, one row more than the compute units and a few more than one
pass of all of them takes.  Bounds are those of test_gpu_row_stats_frames."""
import pytest
import torch

from paper_2605_07230_amd import binding

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("vocab", [4, 2048, 2052, 4096, 4100, 8192, 8196, 12292, 16384, 16388, 22532, 24576, 24580])
@pytest.mark.parametrize("per_cu", [1, 2])
def test_more_rows_than_compute_units(vocab, per_cu):
    n, hidden = per_cu * torch.cuda.get_device_properties(0).multi_processor_count + 1 + 4 * (per_cu - 1), 4
    print(f"[row stats] vocab={vocab} rows={n}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(vocab + n)
    w = torch.randn(vocab, hidden, device="cuda", generator=gen)
    h = torch.randn(n, hidden, device="cuda", generator=gen)
    h[n // 2] = 0.0                      # a row of equal entries
    ctx = binding.Context(max_rows=1, max_nodes_total=n, max_nodes_per_tree=1, max_prefix=0, n_heads=1, head_dim=64, hidden=hidden, vocab=vocab)
    logits = torch.empty(n, vocab, device="cuda")
    mx, thr, lse = (torch.full((n,), float("nan"), device="cuda") for _ in range(3))
    for k in sorted({0, 1, min(50, vocab), min(2000, vocab), max(1, vocab - 1)}):
        binding.lmhead_softmax_cfg(ctx, h_cond=h, h_uncond=None, w=w, cfg_scale=1.0, temperature=1.0, top_k=k, logits=logits, row_max=mx,
                                   row_thr=thr, row_lse=lse)
        kth = torch.topk(logits, k, dim=1).values[:, -1] if 0 < k < vocab else torch.full((n,), -float("inf"), device="cuda")
        assert torch.equal(mx, logits.max(1).values) and torch.equal(thr, kth), k
        g = logits.double()
        ref = torch.logsumexp(g.masked_fill(g < kth.double()[:, None], -float("inf")), 1)
        assert torch.all((lse.double() - ref).abs() <= 1e-5 + 2.0 ** -23 * ref.abs()), k


@pytest.mark.parametrize("vocab", [4, 2052, 6000, 8192, 12292, 16384, 20000, 24576])
@pytest.mark.parametrize("law", ["sorted", "one_range"])
def test_rows_whose_entries_are_ordered(vocab, law):
    """Entries that fall along the row, and -inf outside one range of them that does not begin with the row: the first load of every wave,
    whose range bins the row, lies elsewhere in it, also where the row holds fewer whole chunks than there are waves."""
    n = torch.cuda.get_device_properties(0).multi_processor_count + 9
    print(f"[row stats] vocab={vocab} rows={n} {law}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(vocab)
    w = torch.randn(vocab, 2, device="cuda", generator=gen)
    if law == "sorted":
        w[:, 1] = torch.sort(3 * w[:, 1], descending=True).values
    else:
        w[:, 1] = -3e38      # twice that is -inf
        w[vocab // 4:vocab // 4 + (vocab + 3) // 4, 1] = 0.0
    h = torch.stack([torch.linspace(-1.0, 1.0, n, device="cuda"), torch.full((n,), 2.0, device="cuda")], dim=1)
    ctx = binding.Context(max_rows=1, max_nodes_total=n, max_nodes_per_tree=1, max_prefix=0, n_heads=1, head_dim=64, hidden=2, vocab=vocab)
    logits = torch.empty(n, vocab, device="cuda")
    mx, thr, lse = (torch.full((n,), float("nan"), device="cuda") for _ in range(3))
    for k in sorted({1, min(50, max(1, vocab // 4)), min(2000, max(1, vocab // 4))}):
        binding.lmhead_softmax_cfg(ctx, h_cond=h, h_uncond=None, w=w, cfg_scale=1.0, temperature=1.0, top_k=k, logits=logits, row_max=mx,
                                   row_thr=thr, row_lse=lse)
        kth = torch.topk(logits, k, dim=1).values[:, -1]
        assert torch.equal(mx, logits.max(1).values) and torch.equal(thr, kth), k
        g = logits.double()
        ref = torch.logsumexp(g.masked_fill(g < kth.double()[:, None], -float("inf")), 1)
        assert torch.all((lse.double() - ref).abs() <= 1e-5 + 2.0 ** -23 * ref.abs()), k
