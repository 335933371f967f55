"""Acceptance on feature rows that do not go through the matrix cores (f32 of any width, bf16 widths that are no multiple
of 128): the others of a node are swept eight at a time by the workgroup, or four at a time by each wave where rows are
narrow, so nodes with 1 to 60 relatives and widths around the workgroup's stride (512 threads x 4 floats), around the
narrow rows' limit (1024 elements, 128 where a row cannot be read 16 bytes at a time) and not divisible by a 16-byte
piece are compared with the checker.

Cosines are float32 dot products in some order: off by at most h 2^-24 sum|a||b| / (|a||b|) <= h 2^-24, the quotient adds a
few 2^-24; set sizes are exact because the constructed cosines stay 1e-3 away from the thresholds."""
import numpy as np
import pytest
import torch

from oracle import verify_oracle as vo
from paper_2605_07230_amd import binding
from paper_2605_07230_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,hidden", [("f32", 1), ("f32", 99), ("f32", 129), ("f32", 260), ("f32", 516), ("f32", 1024), ("f32", 1028), ("f32", 2048), ("f32", 2052), ("f32", 5000), ("bf16", 136), ("bf16", 1016), ("bf16", 1032), ("bf16", 4104)])
@pytest.mark.parametrize("kids", [1, 7, 8, 17, 60])
def test_acceptance_on_generic_rows(dtype, hidden, kids):
    rng = np.random.default_rng(hidden * 64 + kids)
    # a root with `kids` children, the first of which has `kids` children of its own
    parent = np.array([-1] + [0] * kids + [1] * kids, np.int32)
    n, vocab = len(parent), 256
    h = rng.standard_normal((n, hidden)).astype(np.float32)
    for i in range(2, n):
        if i % 3:
            h[i] = h[parent[i] if i % 2 else i - 1] + 0.2 * h[i]
    if dtype == "bf16":
        h = wl.round_bf16(h)
    off, token = np.array([0, n], np.int32), rng.integers(0, vocab, n).astype(np.int32)
    logits = rng.standard_normal((n, vocab)).astype(np.float32)
    thr, lse = np.full(n, -np.inf, np.float32), np.log(np.exp(logits.astype(np.float64)).sum(1)).astype(np.float32)
    c = np.abs(h.astype(np.float64) @ h.astype(np.float64).T / np.outer(*[np.linalg.norm(h.astype(np.float64), axis=1)] * 2))
    tau = 0.9 + 0.002 * min(range(25), key=lambda k: -np.abs(c - 0.9 - 0.002 * k).min())   # the widest gap near 0.9
    acc = vo.cascade_accept(off, parent, token, h, logits.astype(np.float64), thr.astype(np.float64), lse.astype(np.float64), tau, tau)
    if hidden == 1:                       # every cosine is 1 or -1: all the same
        tau = 0.5
        acc = vo.cascade_accept(off, parent, token, h, logits.astype(np.float64), thr.astype(np.float64), lse.astype(np.float64), tau, tau)
    print(f"[accept] {dtype} hidden={hidden} kids={kids} tau={tau}", flush=True)
    dev = lambda x: torch.from_numpy(x).cuda()  # noqa: E731
    ctx = binding.Context(max_rows=1, max_nodes_total=n, max_nodes_per_tree=n, max_prefix=0, n_heads=1, head_dim=64, hidden=hidden, vocab=vocab)
    f = {k: torch.full((n,), float("nan"), device="cuda") for k in ("q_tok", "m_int", "m_conv", "cos_parent")}
    i = {k: torch.full((n,), -7, dtype=torch.int32, device="cuda") for k in ("n_int", "n_conv")}
    hd = dev(h) if dtype == "f32" else dev(h).bfloat16()
    binding.cascade_accept(ctx, node_off=dev(off), parent=dev(parent), token=dev(token), h_cond=hd, logits=dev(logits), row_thr=dev(thr),
                           row_lse=dev(lse), tau_pos=tau, tau_seq=tau, **f, **i)
    assert ctx.device_status() == binding.OK
    np.testing.assert_array_equal(i["n_int"].cpu().numpy(), acc.n_int)
    np.testing.assert_array_equal(i["n_conv"].cpu().numpy(), acc.n_conv)
    np.testing.assert_allclose(f["cos_parent"].cpu().numpy(), acc.cos_parent, rtol=0, atol=(hidden + 16) * 2.0 ** -24)
    for k in ("q_tok", "m_int", "m_conv"):
        np.testing.assert_allclose(f[k].cpu().numpy(), getattr(acc, k), rtol=1e-5, atol=1e-9)
