"""Path selection at the edges of its register frames: vocabularies around the 16384- and 65536-entry frames and the 256-entry
chunks (rows that 16-byte loads can and cannot read), trees around the 64-node chunks and the 256-node frame.

Integers are compared with the float64 checker.  The kernel's float32 masses, scans and target are off by at most a few
2^-24 of the row's mass per addition along a chain of ~30 additions, 2e-6; the inputs keep every decision further away."""
import numpy as np
import pytest
import torch

from oracle import verify_oracle as vo
from paper_2605_07230_amd import binding
from paper_2605_07230_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _inputs(vocab, sizes, limited, seed):
    rng = np.random.default_rng(seed)
    trees = [wl.grow_tree(rng, n, min(6, n - 1)) for n in sizes]
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    n = int(off[-1])
    f32 = lambda x: np.asarray(x, np.float32)  # noqa: E731
    g = f32(2.0 * rng.standard_normal((n, vocab)))
    thr = np.full(n, -np.inf, np.float32)
    if limited:
        k = min(2000, vocab)
        thr = np.partition(g, vocab - k, axis=1)[:, vocab - k]
    kept = np.where(g >= thr[:, None], np.exp(g.astype(np.float64)), 0.0)
    m = f32(np.where(rng.random(n) < 0.5, 0.1 * rng.random(n), 0.0))
    acc = vo.AcceptScalars(q_tok=f32(0.5 * rng.random(n)), m_int=m, m_conv=f32(m[::-1]), n_int=(m > 0).astype(np.int32),
                           n_conv=(m[::-1] > 0).astype(np.int32), cos_parent=np.zeros(n), min_cos_margin=1.0)
    return dict(off=off, parent=np.concatenate(trees).astype(np.int32), token=rng.integers(0, vocab, n).astype(np.int32), acc=acc, g=g, thr=thr,
                lse=f32(np.log(kept.sum(1))), draft=f32(rng.random(n)), u=f32(rng.random(n)), ub=f32(rng.random(len(sizes))))


@pytest.mark.parametrize("mode", [binding.WALK_SEQUENTIAL, binding.WALK_LONGEST])
@pytest.mark.parametrize("vocab", [4, 250, 256, 16380, 16384, 16385, 16388, 65532, 65533, 65536])
@pytest.mark.parametrize("sizes", [(2, 64, 65), (256, 17, 193), (257, 2, 300)])
def test_select_path_edges(vocab, sizes, mode):
    print(f"[select] vocab={vocab} trees={sizes} mode={mode}", flush=True)
