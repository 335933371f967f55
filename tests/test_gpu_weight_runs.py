"""convergence_weights where its split changes: row widths around every number of waves that share a row, sequence lengths
around the run length, and runs at their longest."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,B,K,h", [
    ("bf16", 3, 2, 8),              # the narrowest row, one pair
    ("bf16", 2, 5, 512), ("bf16", 2, 6, 520),        # 1 KiB, one piece more (two waves per row)
    ("f32", 2, 37, 512), ("f32", 1, 38, 516),        # 2 KiB, one piece more (four waves per row)
    ("bf16", 5, 1000, 2048), ("bf16", 3, 1001, 2056),   # 4 KiB, one piece more (two KiB per wave)
    ("f32", 8, 700, 2048), ("f32", 2, 777, 2052),    # 8 KiB, one piece more (four KiB per wave)
    ("bf16", 1, 515, 8192),         # 16 KiB, the widest row
    ("f32", 2, 150001, 64),         # runs at their longest (128 pairs)
])
def test_weights_over_widths_and_run_lengths(dtype, B, K, h):
    from paper_2605_07230_amd import binding
    print(f"[weight runs] dtype={dtype} B={B} K={K} h={h}", flush=True)
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(K + h)
    x = torch.randn(B, K, h, device=dev, generator=gen)
    x[:, 1:] += 1.5 * x[:, :-1].clone()
    x = x.to(torch.bfloat16 if dtype == "bf16" else torch.float32).contiguous()
    w, cs = torch.full((B, K), -5.0, device=dev), torch.full((B, K), -5.0, device=dev)
    ctx = binding.Context(max_rows=1, max_nodes_total=1, max_nodes_per_tree=1, max_prefix=0, n_heads=1, head_dim=64, hidden=64, vocab=64)
    binding.convergence_weights(ctx, features=x, tau_seq=0.6, c=2.0, weights=w, cos_next=cs)
    assert ctx.device_status() == binding.OK
    # float32 sums of exact float32 / bf16 products: a rounding error of a few 2^-24 sqrt(terms per lane) each
    ref = torch.nn.functional.cosine_similarity(x[:, :-1].double(), x[:, 1:].double(), dim=-1)
    assert (cs[:, :-1].double() - ref).abs().max().item() <= 2e-6
    assert (cs[:, -1] == 0).all() and (w[:, -1] == 1).all()
    torch.testing.assert_close(w[:, :-1], torch.where(cs[:, :-1] >= 0.6, 2.0, 1.0), rtol=0, atol=0)
