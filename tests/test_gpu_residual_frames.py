"""The residual walk around its register frames (1, 4, 8, 12 and 16 four-wide vectors per lane; 4096 to 65536 entries): rows that
fill a frame, one vector more, a few entries, trees of one and several 64-node chunks.  Checked as in test_gpu_next."""
import numpy as np
import pytest

import test_gpu_next as nxt
from paper_2605_07230_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("vocab", [128, 4096, 4100, 12300, 16384, 16388, 32768, 32772, 49152, 49156])
@pytest.mark.parametrize("sizes", [(3, 20), (65, 130)])
def test_residual_walk_frames(vocab, sizes):
    for seed in range(20):
        rng = np.random.default_rng(seed)
        inp = wl.make_inputs(seed=seed, name=f"frame{vocab}", dtype="f32", n_prompts=2, cfg=False, n_heads=2, n_kv_heads=2, head_dim=32,
                             hidden=64, vocab=vocab, prefix_lens=[5, 9], trees=[wl.grow_tree(rng, n, min(4, n - 1)) for n in sizes],
                             cfg_scale=1.0, temperature=1.0, top_k=min(50, vocab - 1), tau_pos=2.0, tau_seq=2.0, eps_tvd=0.5, token_law="zipf")
        try:
            nxt._check_residual(inp, seed, 0.7)
            return
        except AssertionError as e:
            if "min walk margin" not in str(e) or "not equal" in str(e).lower():
                raise
    raise AssertionError("no seed keeps its decisions apart")
