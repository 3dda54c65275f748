"""The prefill-shaped tree attention where its launch shapes and its softmax shift can go wrong:
launches of more than 512 row blocks (one group of waves per workgroup), with one unit per XCD,
row blocks that end inside a tile, and scores whose range makes the
shift move again and again.  Against the CPU oracle, at its bf16 tolerance.  And NaN scores."""
import numpy as np
import pytest
import torch

import test_gpu_tree_attn
from gpu_harness import Run, from_dev, log
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


# The compact kernel; beyond its key range one and two groups of waves per workgroup
@pytest.mark.parametrize("d,hkv,layers,prompt", [(64, 2, 1, 90), (96, 2, 1, 90), (128, 2, 1, 90), (64, 2, 1, 780), (128, 2, 1, 600),
                                                 (64, 8, 2, 780), (96, 8, 2, 600), (128, 8, 2, 600)])
@pytest.mark.parametrize("where", ["k", "q"])
def test_nan_scores_stay_nan(d, hkv, layers, prompt, where):
    """A NaN key, or a query with an infinite element: the rows that see it are NaN, the others as
    they were, those of empty queries zero."""
    w = small(n_layers=layers, prompt_min=prompt, prompt_max=prompt, n_q_heads=8 * hkv, n_kv_heads=hkv, head_dim=d,
              beam_width=6, steps=7, alpha=0.0)
    log(f"nan scores d={d} Hkv={hkv} L={layers} P={prompt} {where}")
    r = Run(w, seed=26, oracle=False)
    for _ in range(w.steps):
        r.step(check=False)
    q, kn, vn, logits, _, _ = r.inputs(w.steps + 1)
    qd, knd, vnd, _ = r.dev_inputs(w.steps + 1, q, kn, vn, logits)
    r.dec.attn_decode(0, layers, qd, knd, vnd, torch.empty_like(qd), r.scale)  # stores the leaves
    st = r.dec.read_state(0)
    n = st["n_nodes"]
    slots = np.concatenate([np.arange(n), [-1, -1, -1]]).astype(np.int32)
    qs = torch.from_numpy(slots[None]).cuda()
    x = torch.randn((layers, 1, n + 3, 8 * hkv, d), device="cuda", generator=torch.Generator("cuda").manual_seed(3))
    x = x.to(torch.bfloat16)
    out = [torch.full_like(x, 5.0) for _ in range(2)]
    r.dec.tree_attn(0, layers, qs, x, out[0], r.scale)
    hit = np.zeros((n + 3, 8 * hkv), bool)
    bad = n - 3  # a leaf, or a node on the way to one
    if where == "k":
        bad = int(st["parent_slot"][bad])
        r.dec.k_pool[:, :, 1, st["base"] + bad, 5] = float("nan")
        for i in range(n):
            p = i
            while p > bad:
                p = st["parent_slot"][p]
            hit[i, 8:16] = p == bad and st["mask"][i] != 0
    else:
        x[:, :, bad, 3, 7] = float("inf")
        x[:, :, n + 1] = float("nan")
        hit[bad, 3] = True
    r.dec.tree_attn(0, layers, qs, x, out[1], r.scale)
    a, b = (from_dev(o)[:, 0] for o in out)
    assert hit.any() and np.isnan(b[:, hit]).all()
    assert np.array_equal(a[:, ~hit], b[:, ~hit]) and np.isfinite(a).all() and not a[:, n:].any()
    r.dec.close()
