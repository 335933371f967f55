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


# entries that are not -inf, how many of them the sample holds, k
FEW_FINITE = {"few": (128, 6, (20, 50)), "thousands": (2400, 100, (2000,))}


def _delta(law, vocab, at, gen):
    """What a misled row has added to the values of the ordinary ones."""
    delta = torch.zeros(vocab, device="cuda")
    if law in FEW_FINITE:
        finite, sampled, _ = FEW_FINITE[law]
        rest = torch.ones(vocab, dtype=torch.bool, device="cuda")
        rest[at] = False
        rest = torch.nonzero(rest).flatten()
        keep = torch.cat([at[torch.randperm(len(at), device="cuda", generator=gen)[:sampled]],
                          rest[torch.randperm(len(rest), device="cuda", generator=gen)[:finite - sampled]]])
        delta[:] = -3e38      # twice that is -inf
        delta[keep] = 0.0
    elif law == "one_large":
        delta[at[1234]] = 1e6
    else:
        delta[at] = 10.0 if law == "sample_high" else -10.0
    return delta


def _bins(row, at, k):
    """The bins, of 4096 over the finite range of the sample, of the sample's entry that makes the cut and of the row's k-th largest."""
    sample = row[at].double()
    lo, hi = sample[sample > -float("inf")].min(), sample.max()
    mean = k * 4096 / len(row)
    rank = int(mean + 4 * mean ** 0.5 + 8)
    return [int(torch.nan_to_num((torch.topk(x.double(), n).values[-1] - lo) * 4096 / (hi - lo), neginf=0.0).clamp(0, 4095)) for x, n in ((sample, rank), (row, k))]


@pytest.mark.parametrize("vocab", [33088, 45060, 57344, 65532, 65536])
@pytest.mark.parametrize("law", ["few", "thousands", "one_large", "sample_high", "sample_low"])
def test_misled_and_ordinary_rows_in_turn(vocab, law):
    """More rows than compute units, so that a workgroup takes a misled row and then an ordinary one, or the other way round.  "few",
    "thousands" and "one_large" are samples whose cut lies in their lowest bin, which says nothing, while the k-th largest entry of the row does not."""
    units = torch.cuda.get_device_properties(0).multi_processor_count
    n = 2 * units + 5
    print(f"[row stats] vocab={vocab} rows={n} {law}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(vocab)
    at = _sampled(vocab)
    w = torch.stack([torch.randn(vocab, device="cuda", generator=gen), _delta(law, vocab, at, gen)], dim=1)
    rows = torch.arange(n, device="cuda")
    misled = (rows + rows // units) % 2 == 0
    h = torch.stack([torch.linspace(0.5, 2.0, n, device="cuda"), 2.0 * misled], dim=1)
    ctx = binding.Context(max_rows=1, max_nodes_total=n, max_nodes_per_tree=1, max_prefix=0, n_heads=1, head_dim=64, hidden=2, vocab=vocab)
    logits = torch.empty(n, vocab, device="cuda")
    mx, thr, lse = (torch.full((n,), float("nan"), device="cuda") for _ in range(3))
    for k in FEW_FINITE[law][2] if law in FEW_FINITE else (1,) if law == "one_large" else (50, 2000):
        binding.lmhead_softmax_cfg(ctx, h_cond=h, h_uncond=None, w=w, cfg_scale=1.0, temperature=1.0, top_k=k, logits=logits, row_max=mx,
                                   row_thr=thr, row_lse=lse)
        if law in FEW_FINITE or law == "one_large":
            sample_bin, row_bin = _bins(logits[0], at, k)
            assert sample_bin == 0 < row_bin
        kth = torch.topk(logits, k, dim=1).values[:, -1]
        assert torch.equal(mx, logits.max(1).values) and torch.equal(thr, kth), k
        g = logits.double()
        ref = torch.logsumexp(g.masked_fill(g < kth.double()[:, None], -float("inf")), 1)
        assert torch.all((lse.double() - ref).abs() <= 1e-5 + 2.0 ** -23 * ref.abs()), k
