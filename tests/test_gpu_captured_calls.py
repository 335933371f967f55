"""Graphs captured from one context whose replays overlap with each other and with further calls of that context: acceptance on
wide rows and path selection on long rows share a node or a prompt among workgroups when they are called, and must not when they
are recorded, where nothing orders the workgroups of two replays.

Chunk sums do not depend on how passes are dealt, so a recorded walk equals the called one bit for bit; cosines are off by at
most (h + 16) 2^-24, as in test_gpu_accept_widths."""
import numpy as np
import pytest
import torch

from paper_2605_07230_amd import binding
from paper_2605_07230_amd import workloads as wl

pytestmark = pytest.mark.gpu

VOCAB, HIDDEN, NODES, PROMPTS, DEPTH = 65536, 16384, 30, 4, 8


def _problem(seed):
    rng = np.random.default_rng(seed)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    n = NODES * PROMPTS
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).cuda()  # noqa: E731
    rand = lambda *s: torch.rand(*s, device="cuda", generator=gen)  # noqa: E731
    logits = 2.0 * torch.randn(n, VOCAB, device="cuda", generator=gen)
    thr = torch.topk(logits, 2000, dim=1).values[:, -1].contiguous()
    tree = dict(node_off=dev((NODES * np.arange(PROMPTS + 1)).astype(np.int32)),
                parent=dev(np.concatenate([wl.grow_tree(rng, NODES, 6) for _ in range(PROMPTS)]).astype(np.int32)),
                token=dev(rng.integers(0, VOCAB, n).astype(np.int32)), logits=logits, row_thr=thr,
                row_lse=torch.logsumexp(logits.masked_fill(logits < thr[:, None], -float("inf")), 1))
    zero = torch.zeros(n, dtype=torch.int32, device="cuda")
    walk = dict(q_tok=0.5 * rand(n), m_int=0.1 * rand(n), m_conv=0.1 * rand(n), n_int=zero, n_conv=zero, draft_prob=None, u=rand(n),
                u_bonus=rand(PROMPTS), eps_tvd=0.12, max_depth=DEPTH, mode=binding.WALK_SEQUENTIAL)
    return tree, walk, torch.randn(n, HIDDEN, device="cuda", generator=gen)


class _Call:
    """One acceptance and one walk with outputs of their own."""

    def __init__(self, ctx, seed):
        self.ctx, (self.tree, self.walk, self.rows) = ctx, _problem(seed)
        n = NODES * PROMPTS
        self.scalars = dict({k: torch.empty(n, device="cuda") for k in ("q_tok", "m_int", "m_conv", "cos_parent")},
                            **{k: torch.empty(n, dtype=torch.int32, device="cuda") for k in ("n_int", "n_conv")})
        self.path = {k: torch.empty(s, dtype=torch.int32, device="cuda") for k, s in dict(
            accept_len=(PROMPTS,), path_nodes=(PROMPTS, DEPTH), emitted=(PROMPTS, DEPTH + 1), terminal=(PROMPTS,)).items()}
        self.tvd = torch.empty(PROMPTS, device="cuda")

    def __call__(self):
        binding.cascade_accept(self.ctx, h_cond=self.rows, tau_pos=0.005, tau_seq=0.005, **self.scalars, **self.tree)
        binding.select_path(self.ctx, tvd_used=self.tvd, **self.path, **self.walk, **self.tree)

    def clear(self):
        for t in (*self.scalars.values(), *self.path.values(), self.tvd):
            t.fill_(-7)

    def result(self):
        return {k: t.clone() for k, t in dict(self.scalars, **self.path, tvd=self.tvd).items()}


def test_replays_that_overlap():
    stream, sides = torch.cuda.Stream(), [torch.cuda.Stream() for _ in range(2)]
    n = NODES * PROMPTS
    with torch.cuda.stream(stream):
        ctx = binding.Context(max_rows=PROMPTS, max_nodes_total=n, max_nodes_per_tree=NODES, max_prefix=0, n_heads=32, head_dim=128,
                              hidden=HIDDEN, vocab=VOCAB, stream=stream)
        calls = [_Call(ctx, seed) for seed in range(3)]
        expect = []
        for call in calls:
            call()
            expect.append(call.result())
    torch.cuda.synchronize()
    graphs = []
    for call in calls[:2]:
        graphs.append(torch.cuda.CUDAGraph())
        with torch.cuda.graph(graphs[-1], stream=stream):
            call()
    for replay in range(20):
        for call in calls:
            call.clear()
        torch.cuda.synchronize()
        for _ in range(3):
            for graph, side in zip(graphs, sides):
                with torch.cuda.stream(side):
                    graph.replay()
            with torch.cuda.stream(stream):
                calls[2]()
        torch.cuda.synchronize()
        print(f"[captured] replay {replay}", flush=True)
        for call, want in zip(calls, expect):
            for k, got in call.result().items():
                if k == "cos_parent":
                    assert (got - want[k]).abs().max() <= 2 * (HIDDEN + 16) * 2.0 ** -24
                else:
                    assert torch.equal(got, want[k]), (replay, k)
    assert ctx.device_status() == binding.OK
