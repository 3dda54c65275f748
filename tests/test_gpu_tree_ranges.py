"""Prefill-shaped tree attention over key ranges beyond the compact kernel's, where the rule of
the kernels and of the groups of waves per workgroup changes: one or two groups, several tiles
past the shared prefix, a window, dead nodes, scores that move the softmax shift.  Against the CPU
oracle, at its bf16 tolerance."""
import pytest

import test_gpu_tree_attn
from gpu_harness import Run
from test_gpu_tree_attn import every_node, run_tree, small

pytestmark = pytest.mark.gpu


# (KV heads, layers, prompt, window): 16 to 640 row blocks of 128 rows; tries of 544 to 800 nodes,
# below and above both limits of the rule
@pytest.mark.parametrize("d", [64, 96, 128])
@pytest.mark.parametrize("hkv,layers,prompt,window", [(2, 1, 528, 0), (2, 1, 600, 0), (2, 1, 640, 520), (8, 2, 576, 0),
                                                      (8, 2, 770, 0)])
def test_long_ranges(d, hkv, layers, prompt, window):
    g = 8 if layers > 1 else 4
    run_tree(small(n_layers=layers, prompt_min=prompt, prompt_max=prompt, n_q_heads=g * hkv, n_kv_heads=hkv, head_dim=d,
                   beam_width=6, steps=7, window=window, gc_interval=4), seed=24, pick=every_node)


# 257 to 512 row blocks: one group where the blocks are not those of every node, or have no XCD of
# their own (12 units), two where they are and have
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("tries,hkv,layers,g,prompt,n", [(1, 8, 4, 4, 600, 300), (3, 4, 1, 8, 570, None), (1, 8, 2, 4, 600, None)])
def test_groups(d, tries, hkv, layers, g, prompt, n):
    run_tree(small(n_tries=tries, n_layers=layers, prompt_min=prompt, prompt_max=prompt, n_q_heads=g * hkv, n_kv_heads=hkv,
                   head_dim=d, beam_width=6, steps=3), seed=27, pick=lambda tr, r: every_node(tr, r)[-(n or 10 ** 6):])


# a window over a trie of many nodes per level, queries in no order: a row block's keys are many more
# than its window's levels hold on average (the estimate that chooses the kernel)
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("window", [30, 100])
def test_diverged_trie_with_unsorted_queries(d, window):
    def shuffled(tr, g):
        assert len(tr.order) > 900
        return g.permutation(every_node(tr, g))

    run_tree(small(n_layers=1, prompt_min=40, prompt_max=40, n_q_heads=8, n_kv_heads=2, head_dim=d, beam_width=16,
                   steps=78, window=window, gc_interval=60, alpha=0.0), seed=28, pick=shuffled)


@pytest.mark.parametrize("d,hkv", [(64, 2), (96, 4), (128, 2)])
def test_large_scores(d, hkv, monkeypatch):
    # twelve times the usual scale: scores of a row over tens of powers of two
    class Steep(Run):
        def __init__(self, *args, **kw):
            super().__init__(*args, **kw)
            self.scale *= 12.0

    monkeypatch.setattr(test_gpu_tree_attn, "Run", Steep)
    run_tree(small(prompt_min=790, prompt_max=790, n_layers=1, n_q_heads=4 * hkv, n_kv_heads=hkv, head_dim=d, beam_width=6,
                   steps=4), seed=25, pick=every_node)
