"""bf16 tree attention in every way the dispatcher cuts it (64 / 80 / 96 / 128 / 256 query rows per workgroup, keys split or
whole, query-split) at head_dim 64 and 128: ragged trees around the cuts' edges, empty prefixes, one-node trees, prefixes
around the 64-key tiles; every output against float64.

Bound per output, with m = sum p |v|: rounding to bf16 (8 significant bits, to nearest) moves a value by at most u = 2^-8 of
it.  Probabilities are rounded before the second product (u m), their sum may be taken after that rounding (u m), the output
is rounded (u m), and a score's float32 error d moves every probability by at most 2 d.  The log-sum-exp carries d, the
rounded sum (u) and L 2^-24.

That bound would not see probabilities rounded more coarsely, so the 2-norm distance from float64 is compared with that of a
copy of the finest rounding: every tile of 64 keys refers to its own maximum, probabilities are rounded once, the output is
rounded once.  float32 instead of float64 before a rounding flips 2^-24 / 2^-9 of them, 3e-5, so both distances agree to 3e-3
where the kernel rounds like that (steps of few workgroups, head_dim 64, and the query split up to eight tiles).  A reference
that is not the tile's spreads the mantissas of the heavy probabilities, at worst evenly over an octave: sqrt(2) times the
distance of a copy without rounded probabilities, 1.17 times this one's; a running maximum measures 1.03 to 1.08."""
import numpy as np
import pytest
import torch

from paper_2605_07230_amd import binding
from paper_2605_07230_amd import workloads as wl

pytestmark = pytest.mark.gpu

CASES = {   # kv heads, query heads per kv head, tree sizes, prefix lengths (cuts: CUTS, below)
    "64 rows, keys in 8 parts": (2, 1, [60, 41, 64, 17, 55], [1500, 37, 700, 1100, 260]),
    "64 rows, keys in 16 parts": (1, 1, [60, 31], [4000, 900]),
    "64 rows, whole": (32, 1, [60, 41, 64, 17, 55], [800, 0, 64, 513, 300]),
    "64 rows, grouped heads, ragged blocks": (2, 3, [100, 33, 64], [1900, 130, 0]),
    "80 rows": (32, 1, [70, 80, 65, 3, 64, 63, 79, 16, 1], [90, 200, 64, 0, 333, 128, 1, 65, 63]),
    "96 rows": (32, 1, [90, 96, 81, 3, 64, 63, 79, 16, 1], [90, 200, 64, 0, 333, 128, 1, 65, 63]),
    "128 rows": (32, 1, [100, 128, 97, 33, 64, 63, 79, 16, 1, 2, 127, 65, 17, 111, 20, 7],
                 [90, 20, 64, 0, 133, 128, 1, 65, 63, 10, 5, 70, 30, 100, 40, 200]),
    "128 rows, keys in parts": (32, 1, [256, 130], [4000, 64]),
    "128 rows, long keys in parts": (32, 1, [256, 240], [4200, 4100]),
    "256 rows": (32, 1, [256, 255, 130, 200, 140, 199, 250, 256], [70, 1, 0, 64, 65, 130, 200, 31]),
    "query split": (2, 1, [20, 17], [400, 63]),
    "query split, one node": (1, 1, [1], [0]),
    # the cuts above with several blocks of query rows or several parts where they had one (prefixes are not streamed then), and
    # with fewer or more workgroups (the tile's own maximum, or the running one)
    "64 rows, grouped heads, full chip": (8, 4, [80, 80, 66, 3, 80, 79, 41, 1, 80], [24, 0, 64, 65, 1, 20, 70, 13, 5]),
    "80 rows, grouped heads, several blocks": (16, 2, [70] * 8 + [69], [24, 0, 24, 1, 20, 24, 13, 5, 24]),
    "80 rows, grouped heads, few workgroups": (8, 4, [40] * 15 + [39], [24, 0, 24, 1, 20, 24, 13, 5, 24, 24, 7, 23, 19, 24, 2, 24]),
    "80 rows, one block, few workgroups": (16, 2, [33, 40, 5, 33, 40, 40, 21, 1, 40, 38, 40, 40], [24, 0, 64, 65, 1, 20, 70, 13, 5, 24, 24, 7]),
    "96 rows, grouped heads, several blocks": (8, 4, [70] * 8 + [69], [24, 0, 24, 1, 20, 24, 13, 5, 24]),
    "96 rows, keys in parts": (8, 1, [90] * 5 + [89], [513, 90, 400, 64, 0, 130]),
    "96 rows, few workgroups": (32, 1, [90, 96, 81, 3, 64, 95], [24, 0, 64, 65, 1, 20]),
    "128 rows, grouped heads, several blocks": (8, 4, [60] * 15 + [59], [24, 0, 24, 1, 20, 24, 13, 5, 24, 24, 7, 23, 19, 24, 2, 24]),
    "128 rows, one block, few workgroups": (32, 1, [15, 20, 7, 15, 20, 19, 3, 20, 15, 20, 1, 20], [24, 0, 64, 65, 1, 20, 70, 13, 5, 24, 24, 7]),
    "128 rows, grouped heads, keys in parts": (16, 2, [60, 64, 33, 60, 60, 21, 64, 64], [2000, 1300, 64, 1900, 2000, 7, 1000, 2000]),
}

# (query rows per workgroup, parts of the keys) that 256 compute units choose, at head_dim 64 and 128
CUTS = {
    "64 rows, keys in 8 parts": ((64, 8), (64, 8)), "64 rows, keys in 16 parts": ((64, 16), (64, 16)), "64 rows, whole": ((64, 1), (64, 1)),
    "64 rows, grouped heads, ragged blocks": ((64, 8), (64, 8)), "80 rows": ((80, 1), (80, 1)), "96 rows": ((96, 1), (96, 1)),
    "128 rows": ((128, 1), (128, 1)), "128 rows, keys in parts": ((64, 3), (128, 4)), "128 rows, long keys in parts": ((128, 4), (128, 4)),
    "256 rows": ((256, 1), (256, 1)), "query split": ((16, 1), (16, 1)), "query split, one node": ((16, 1), (16, 1)),
    "64 rows, grouped heads, full chip": ((64, 1), (64, 1)), "80 rows, grouped heads, several blocks": ((80, 1), (80, 1)),
    "80 rows, grouped heads, few workgroups": ((80, 1), (80, 1)), "80 rows, one block, few workgroups": ((80, 1), (80, 1)),
    "96 rows, grouped heads, several blocks": ((96, 1), (96, 1)), "96 rows, keys in parts": ((96, 4), (96, 4)), "96 rows, few workgroups": ((96, 1), (96, 1)),
    "128 rows, grouped heads, several blocks": ((64, 1), (128, 1)), "128 rows, one block, few workgroups": ((64, 1), (128, 1)),
    "128 rows, grouped heads, keys in parts": ((128, 3), (128, 3)),
}
FULL_CHIP = ("256 rows", "128 rows, keys in parts", "128 rows, long keys in parts", "64 rows, grouped heads, full chip",
             "80 rows, grouped heads, several blocks", "96 rows, grouped heads, several blocks")


@pytest.mark.parametrize("name", CASES)
@pytest.mark.parametrize("head_dim", [64, 128])
def test_attention_cuts(name, head_dim):
    full_chip = name in FULL_CHIP or (head_dim == 128 and name in ("80 rows", "96 rows", "128 rows"))
    _check(head_dim, *CASES[name], further=(1.17 if name == "256 rows" else 1.08) if full_chip else 1.003)


# buffers 2, 8 and 14 bytes past a 16-byte boundary, and positions further apart than a 32-bit offset of a tile reaches:
# loads that need neither, in the cuts they come in (64 and 128 query rows per workgroup, keys whole and in parts, query split)
LOADS = {
    "64 rows, keys in parts": (2, 1, [60, 41, 64, 17, 55], [1500, 37, 700, 1100, 260]),
    "64 rows, grouped heads": (2, 3, [100, 33, 64], [900, 130, 0]),
    "128 rows": (32, 1, [100, 128, 97, 33, 64, 63, 79, 16, 1, 2, 127, 65, 17, 111, 20, 7], [90, 20, 64, 0, 133, 128, 1, 65, 63, 10, 5, 70, 30, 100, 40, 200]),
    "128 rows, keys in parts": (32, 1, [256, 130], [2000, 64]),
    "query split": (2, 1, [20, 17], [400, 63]),
}


@pytest.mark.parametrize("name", LOADS)
@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("shift", [1, 4, 7])
def test_attention_of_buffers_off_the_16_byte_grid(name, head_dim, shift):
    _check(head_dim, *LOADS[name], shift=shift)


@pytest.mark.parametrize("sizes,prefix", [([20, 70], [5, 66]), ([150], [40])])
@pytest.mark.parametrize("head_dim", [64, 128])
def test_attention_of_positions_far_apart(sizes, prefix, head_dim):
    _check(head_dim, 2, 1, sizes, prefix, pos_stride=(1 << 25) + 8)


def _check(head_dim, kv_heads, group, sizes, prefix, shift=0, pos_stride=None, further=None):
    print(f"[attention cuts] heads {kv_heads} x {group}, trees {sizes}, prefixes {prefix}, head_dim {head_dim}, shift {shift}", flush=True)
    rng = np.random.default_rng(head_dim + len(sizes))
    gen = torch.Generator(device="cuda")
    gen.manual_seed(head_dim + kv_heads)
    trees = [wl.grow_tree(rng, n, min(7, n - 1)) for n in sizes]
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    n, S, cap, heads = int(off[-1]), len(sizes), max(max(prefix), 1), kv_heads * group
    r = lambda *s: torch.randn(*s, device="cuda", generator=gen).bfloat16()  # noqa: E731
    q, kt, vt = r(n, heads, head_dim), r(n, kv_heads, head_dim), r(n, kv_heads, head_dim)
    kc, vc = r(S, kv_heads, cap, head_dim), r(S, kv_heads, cap, head_dim)
    if shift:
        def moved(x):
            y = torch.empty(x.numel() + 8, dtype=x.dtype, device="cuda")[shift:shift + x.numel()].view(x.shape)
            assert y.data_ptr() % 16 == 2 * shift
            return y.copy_(x)
        q, kt, vt, kc, vc = (moved(x) for x in (q, kt, vt, kc, vc))
    if pos_stride:   # [position][row][head][head_dim] with a gap behind every position
        def spread(x):
            size = (S, kv_heads, cap, head_dim)
            y = torch.empty(cap * pos_stride, dtype=x.dtype, device="cuda").as_strided(size, (kv_heads * head_dim, head_dim, pos_stride, 1))
            return y.copy_(x)
        kc, vc = spread(kc), spread(vc)
    out, lse = torch.full_like(q, float("nan")), torch.full((n, heads), float("nan"), device="cuda")
    ctx = binding.Context(max_rows=S, max_nodes_total=n, max_nodes_per_tree=max(sizes), max_prefix=cap, n_heads=heads, head_dim=head_dim, hidden=128, vocab=64)
    if (kv_heads, group, sizes, prefix) in CASES.values() and not shift:
        name = next(k for k, c in CASES.items() if c == (kv_heads, group, sizes, prefix))
        assert binding.attention_cut(n_rows=S, n_nodes_total=n, max_nodes_per_tree=max(sizes), max_prefix_len=max(prefix), n_heads=heads,
                                     n_kv_heads=kv_heads, head_dim=head_dim, ctx=ctx) == CUTS[name][head_dim == 128]
    dev = lambda x: torch.from_numpy(np.asarray(x, np.int32)).cuda()  # noqa: E731
    binding.tree_verify_attn(ctx, node_off=dev(off), parent=dev(np.concatenate(trees)), prefix_len=dev(prefix), q=q, k_tree=kt, v_tree=vt,
                             k_cache=kc, v_cache=vc, out=out, lse=lse, max_nodes_per_tree=max(sizes), max_prefix_len=max(prefix))
    assert ctx.device_status() == binding.OK
    scale = head_dim ** -0.5
    far = far_copy = 0.0
    for s in range(S):
        lo, hi, T, P = int(off[s]), int(off[s + 1]), sizes[s], prefix[s]
        see = torch.zeros(T, P + T, dtype=torch.bool)
        see[:, :P] = True
        for i in range(T):
            a = i
            while a >= 0:
                see[i, P + a] = True
                a = int(trees[s][a])
        see = see.cuda()
        for kv in range(kv_heads):
            k, v = torch.cat([kc[s, kv, :P], kt[lo:hi, kv]]).double(), torch.cat([vc[s, kv, :P], vt[lo:hi, kv]]).double()
            for h in range(kv * group, (kv + 1) * group):
                qd = q[lo:hi, h].double()
                z = ((qd @ k.t()) * scale).masked_fill(~see, -float("inf"))
                rl = torch.logsumexp(z, 1)
                p = torch.exp(z - rl[:, None])
                d = head_dim * 2.0 ** -24 * scale * float(qd.norm(dim=1).max() * k.norm(dim=1).max())
                bound = (3 * 2.0 ** -8 + 2 * d) * (p @ v.abs()) + 1e-30
                assert torch.all((out[lo:hi, h].double() - p @ v).abs() <= bound), (s, h)
                assert torch.all((lse[lo:hi, h].double() - rl).abs() <= 2 * d + 2.0 ** -8 + (P + T) * 2.0 ** -24), (s, h)
                if further:
                    num = torch.zeros_like(p @ v)
                    for first, end in [(i, min(i + 64, P)) for i in range(0, P, 64)] + [(P + i, min(P + i + 64, P + T)) for i in range(0, T, 64)]:
                        m = z[:, first:end].max(1, keepdim=True).values.clamp(min=-1e30)     # a tile without visible keys adds nothing
                        num += torch.exp(m - rl[:, None]) * (torch.exp(z[:, first:end] - m).bfloat16().double() @ v[first:end])
                    far += float(((out[lo:hi, h].double() - p @ v) ** 2).sum())
                    far_copy += float(((num.bfloat16().double() - p @ v) ** 2).sum())
    assert not further or far ** 0.5 <= further * far_copy ** 0.5, (far ** 0.5 / max(far_copy, 1e-30) ** 0.5)
