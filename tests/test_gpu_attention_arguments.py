"""Calls of tree_verify_attn that the host can tell to be unusual: a bound of no nodes per tree."""
import ctypes as C

import pytest
import torch

from paper_2605_07230_amd import binding

pytestmark = pytest.mark.gpu


def _call(dtype, max_nodes_per_tree):
    """One row of three nodes behind a five-key prefix: (context, args, keep-alive, out)."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(3)
    r = lambda *s: torch.randn(*s, device="cuda", generator=gen).to(dtype)  # noqa: E731
    q, kt, vt, kc, vc = r(3, 2, 64), r(3, 2, 64), r(3, 2, 64), r(1, 2, 5, 64), r(1, 2, 5, 64)
    i32 = lambda x: torch.tensor(x, dtype=torch.int32, device="cuda")  # noqa: E731
    out = torch.full_like(q, 7.0)
    t = dict(node_off=i32([0, 3]), parent=i32([-1, 0, 0]), prefix_len=i32([5]), q=q, k_tree=kt, v_tree=vt, k_cache=kc, v_cache=vc, out=out)
    ctx = binding.Context(max_rows=1, max_nodes_total=3, max_nodes_per_tree=3, max_prefix=5, n_heads=2, head_dim=64, hidden=64, vocab=64)
    return ctx, binding._tree_attn_args(**t, lse=None, scale=0.0, max_nodes_per_tree=max_nodes_per_tree, max_prefix_len=5), t, out


def test_a_bound_of_no_nodes_is_refused_for_bf16():
    ctx, a, _keep, out = _call(torch.bfloat16, 0)
    assert ctx.lib.tree_verify_attn(ctx.handle, C.byref(a)) == binding.ESHAPE
    assert ctx.lib.tree_verify_attn_static(None, C.byref(a), None) == binding.ESHAPE
    torch.cuda.synchronize()
    assert torch.all(out == 7.0)


def test_the_f32_path_does_not_use_the_bound():
    (ctx, a, _k0, out), (_, b, _k1, ref) = _call(torch.float32, 0), _call(torch.float32, 3)
    assert ctx.lib.tree_verify_attn(ctx.handle, C.byref(a)) == binding.OK and ctx.lib.tree_verify_attn(ctx.handle, C.byref(b)) == binding.OK
    assert ctx.device_status() == binding.OK
    assert torch.equal(out, ref) and not torch.any(out == 7.0)
