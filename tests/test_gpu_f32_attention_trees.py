"""f32 tree attention where the parents move from the lanes of a wave to LDS (128 nodes), where a wave takes several tiles of keys (more than
sixteen, eight or four of them by head width) and with values off the 16-byte grid, against float64.  Bounds are those of test_gpu_f32_kernels."""
import numpy as np
import pytest
import torch

from paper_2605_07230_amd import binding
from paper_2605_07230_amd import workloads as wl
from test_gpu_f32_kernels import _attend

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("head_dim", [32, 64, 128, 256])
@pytest.mark.parametrize("sizes,prefix,depth", [([127], [0], 60), ([128], [129], 9), ([129, 64], [240, 250], 9), ([65, 200], [700, 17], 12), ([16, 1], [272, 1024], 4)])
@pytest.mark.parametrize("off_grid", [False, True])
def test_f32_attention_trees(head_dim, sizes, prefix, depth, off_grid):
    print(f"[f32 attention] d={head_dim} sizes={sizes} prefix={prefix} off_grid={off_grid}", flush=True)
    rng = np.random.default_rng(head_dim + sum(sizes))
    gen = torch.Generator(device="cuda")
    gen.manual_seed(head_dim + sum(sizes))
    heads, kv_heads = 4, 2
    trees = [wl.grow_tree(rng, n, min(depth, n - 1)) if n > 1 else np.full(1, -1, np.int32) for n in sizes]
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    n, S, cap = int(off[-1]), len(sizes), max(max(prefix), 1)

    def rand(*shape, shift=0):
        flat = torch.empty(int(np.prod(shape)) + shift, device="cuda").normal_(generator=gen)
        return flat[shift:].view(*shape)

    q, kt, kc = rand(n, heads, head_dim), rand(n, kv_heads, head_dim), rand(S, kv_heads, cap, head_dim)
    vt, vc = rand(n, kv_heads, head_dim, shift=int(off_grid)), rand(S, kv_heads, cap, head_dim, shift=int(off_grid))
    out, lse = torch.full_like(q, float("nan")), torch.full((n, heads), float("nan"), device="cuda")
    ctx = binding.Context(max_rows=S, max_nodes_total=n, max_nodes_per_tree=max(sizes), max_prefix=cap, n_heads=heads, head_dim=head_dim, hidden=64, vocab=64)
    dev = lambda x: torch.from_numpy(np.asarray(x, np.int32)).cuda()  # noqa: E731
    binding.tree_verify_attn(ctx, node_off=dev(off), parent=dev(np.concatenate(trees)), prefix_len=dev(prefix), q=q, k_tree=kt, v_tree=vt,
                             k_cache=kc, v_cache=vc, out=out, lse=lse, max_nodes_per_tree=max(sizes), max_prefix_len=max(prefix))
    assert ctx.device_status() == binding.OK
    for s, tree in enumerate(trees):
        lo, T, P = int(off[s]), len(tree), prefix[s]
        see = torch.zeros(T, P + T, dtype=torch.bool)
        see[:, :P] = True
        for i in range(T):
            a = i
            while a >= 0:
                see[i, P + a] = True
                a = int(tree[a])
        see = see.cuda()
        for h in range(heads):
            kv = h // (heads // kv_heads)
            k = torch.cat([kc[s, kv, :P], kt[lo:lo + T, kv]])
            v = torch.cat([vc[s, kv, :P], vt[lo:lo + T, kv]])
            ref, l = _attend(q[lo:lo + T, h], k, v, see, head_dim ** -0.5)
            d = head_dim * 2.0 ** -24 * float((q[lo:lo + T, h].double().abs() @ k.double().abs().t()).max()) * head_dim ** -0.5
            bound = (2 * d + (P + T + 8) * 2.0 ** -24) * float(v.abs().max())
            assert (out[lo:lo + T, h].double() - ref).abs().max() <= bound
            assert (lse[lo:lo + T, h].double() - l).abs().max() <= d + (P + T + 8) * 2.0 ** -24 + 2.0 ** -23 * float(l.abs().max())
