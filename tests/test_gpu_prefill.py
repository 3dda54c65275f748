"""The prefill-shaped tree attention where its launch shapes and its softmax shift can go wrong:
launches of more than 512 row blocks (one group of waves per workgroup), with one unit per XCD
(the folded block order), row blocks that end inside a tile, and scores whose range makes the
shift move again and again.  Against the CPU oracle, at its bf16 tolerance."""
import pytest

import test_gpu_tree_attn
from gpu_harness import Run
from test_gpu_tree_attn import every_node, run_tree, small

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [64, 96, 128])
@pytest.mark.parametrize("window", [0, 90])
def test_many_row_blocks(d, window):
    # 2 x 4 x 8 units of 10 row blocks: 640 blocks
    run_tree(small(n_tries=2, n_layers=4, prompt_min=250, prompt_max=290, n_q_heads=32, n_kv_heads=8, head_dim=d,
                   beam_width=4, steps=3, window=window), seed=21, pick=every_node)


def test_one_unit_per_xcd():
    # 8 units of 65 or more row blocks of 128 rows (16 query heads per KV head)
    run_tree(small(n_layers=1, prompt_min=530, prompt_max=530, n_q_heads=128, n_kv_heads=8, head_dim=64,
                   beam_width=4, steps=3), seed=22, pick=every_node)


@pytest.mark.parametrize("d,prompt", [(64, 127), (96, 129), (128, 65)])
def test_large_scores(d, prompt, monkeypatch):
    # twelve times the usual scale: scores of a row over tens of powers of two
    class Steep(Run):
        def __init__(self, *args, **kw):
            super().__init__(*args, **kw)
            self.scale *= 12.0

    monkeypatch.setattr(test_gpu_tree_attn, "Run", Steep)
    run_tree(small(prompt_min=prompt, prompt_max=prompt, n_q_heads=16, n_kv_heads=4, head_dim=d, beam_width=6,
                   steps=4), seed=23, pick=every_node)
