"""Row statistics whose kept entries all belong to one wave: its list holds 704 entries before the exact rounds take over
(768 less the 64 that one step may add), so counts around that and around the 64 lanes, in the first and the last wave, in
rows of one and of several chunks per thread.  Bounds are those of test_gpu_row_stats_frames."""
import pytest
import torch

from paper_2605_07230_amd import binding

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("vocab", [16384, 33088, 65536])
@pytest.mark.parametrize("wave", [0, 15])
@pytest.mark.parametrize("kept", [63, 64, 65, 639, 640, 641, 703, 704, 705, 768, 769])
def test_kept_entries_of_one_wave(vocab, wave, kept):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(vocab + kept)
    row = torch.randn(vocab, device="cuda", generator=gen)
    at = torch.arange(vocab, device="cuda")
    mine = torch.nonzero((at % 4096) // 256 == wave).flatten()    # thread t holds entries 4 t .. 4 t + 3 of every 4096
    row[mine[torch.randperm(len(mine), device="cuda", generator=gen)[:kept]]] += 10.0
    ctx = binding.Context(max_rows=1, max_nodes_total=1, max_nodes_per_tree=1, max_prefix=0, n_heads=1, head_dim=64, hidden=1, vocab=vocab)
    logits = torch.empty(1, vocab, device="cuda")
    mx, thr, lse = (torch.full((1,), float("nan"), device="cuda") for _ in range(3))
    print(f"[row stats] vocab={vocab} wave={wave} kept={kept}", flush=True)
    for k in (kept, kept + 1):
        binding.lmhead_softmax_cfg(ctx, h_cond=torch.ones(1, 1, device="cuda"), h_uncond=None, w=row[:, None].contiguous(), cfg_scale=1.0, temperature=1.0,
                                   top_k=k, logits=logits, row_max=mx, row_thr=thr, row_lse=lse)
        assert torch.equal(logits[0], row) and torch.equal(mx, row.max()[None])
        kth = torch.topk(row, k).values[-1]
        assert torch.equal(thr, kth[None]), (k, thr.item(), kth.item())
        ref = torch.logsumexp(row.double().masked_fill(row < kth, -float("inf")), 0)
        assert abs(lse.item() - ref.item()) <= 1e-5 + 2.0 ** -23 * abs(ref.item())
