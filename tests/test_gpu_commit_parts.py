"""kv_commit around the 2 KiB parts a node row is copied in: rows of one piece, of an odd number of pieces, one part exactly, one
piece more, several parts with a short last one; no slot but the root, and the longest path (65 slots), around the groups of
eight slots that few rows and layers are cut into and with more layers, which make fewer groups.  Bit for bit."""
import numpy as np
import pytest
import torch

from oracle import commit_oracle as co
from paper_2605_07230_amd import binding

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("depth,layers", [(0, 2), (1, 2), (5, 2), (7, 2), (8, 2), (15, 2), (23, 1), (64, 2), (64, 25), (17, 40)])
@pytest.mark.parametrize("dtype,heads,dim", [("bf16", 1, 8), ("bf16", 5, 24), ("bf16", 8, 128), ("bf16", 43, 24), ("f32", 33, 20), ("f32", 7, 100)])
def test_parts_of_a_node_row(dtype, heads, dim, depth, layers):
    rng = np.random.default_rng(heads * dim + depth)
    prompts, T, cap = 3, 70, 100
    S, dt = 2 * prompts, torch.bfloat16 if dtype == "bf16" else torch.float32
    off = (T * np.arange(S + 1)).astype(np.int32)
    accept = np.array([depth, 0, depth // 2], np.int32)
    path = rng.integers(0, T, (prompts, depth)).astype(np.int32)
    row_prompt, plen = (np.arange(S) // 2).astype(np.int32), rng.integers(0, cap - 65, S).astype(np.int32)
    r = lambda *s: torch.from_numpy(rng.standard_normal(s).astype(np.float32)).to(dt)  # noqa: E731
    kt, vt, kc, vc = r(layers, S * T, heads, dim), r(layers, S * T, heads, dim), r(layers, S, heads, cap, dim), r(layers, S, heads, cap, dim)
    ek, ev, elen, over = co.kv_commit(kt.float().numpy(), vt.float().numpy(), kc.float().numpy(), vc.float().numpy(), off, row_prompt, plen, cap, accept, path)
    assert not over.any()
    ctx = binding.Context(max_rows=S, max_nodes_total=S * T, max_nodes_per_tree=T, max_prefix=cap, n_heads=heads, head_dim=128, hidden=128, vocab=64)
    dev = lambda x: torch.from_numpy(x).cuda()  # noqa: E731
    kc, vc, out = kc.cuda(), vc.cuda(), torch.full((S,), -7, dtype=torch.int32, device="cuda")
    print(f"[commit] {dtype} heads {heads} x {dim}, depth {depth}, {layers} layers", flush=True)
    binding.kv_commit(ctx, node_off=dev(off), row_prompt=dev(row_prompt), accept_len=dev(accept), path_nodes=dev(path) if depth else None,
                      k_tree=kt.cuda(), v_tree=vt.cuda(), k_cache=kc, v_cache=vc, prefix_len=dev(plen), prefix_len_out=out)
    assert ctx.device_status() == binding.OK
    assert np.array_equal(out.cpu().numpy(), elen)
    assert np.array_equal(kc.float().cpu().numpy(), ek) and np.array_equal(vc.float().cpu().numpy(), ev)
