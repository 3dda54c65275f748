"""One-layer attention calls over the ranges of the node-split rule (4-wave and 8-wave workgroups,
one to 32 splits, one to four row blocks, the row blocks of a range on one XCD or not), against the
CPU oracle: tries of one tile, of a tile more or less than a workgroup's share, and larger."""
import pytest

import paper_2502_00085_amd.binding as B
import test_gpu_tree_attn as tree
from gpu_harness import Run, log
from test_gpu_parity import small

pytestmark = pytest.mark.gpu


# (tries, beams, q heads, KV heads, prompt, window): units of 1 .. 160, rows of 1 .. 96 per KV head
@pytest.mark.parametrize("T,b,hq,hkv,P,W", [
    (1, 1, 1, 1, 5, 0), (1, 4, 4, 1, 31, 0), (1, 4, 8, 2, 127, 0), (1, 8, 32, 8, 1025, 0), (1, 8, 8, 2, 4200, 0),
    (1, 16, 8, 2, 700, 0), (2, 24, 8, 2, 129, 0), (2, 24, 8, 2, 90, 33), (1, 3, 8, 8, 2300, 1100),
    (16, 4, 8, 8, 70, 0), (20, 4, 16, 8, 150, 0)])
@pytest.mark.parametrize("d", [64, 128])
def test_decode(T, b, hq, hkv, P, W, d):
    w = small(n_tries=T, beam_width=b, n_q_heads=hq, n_kv_heads=hkv, prompt_min=max(1, P - 3 * (T - 1)), prompt_max=P,
              window=W, head_dim=d, n_layers=2, steps=3, vocab=700)
    log(f"splits decode T={T} b={b} Hq={hq} Hkv={hkv} P={P} W={W} d={d}")
    r = Run(w, seed=31, layer_calls=[0, 1, 2])
    for _ in range(w.steps):
        errs, _ = r.step()
        assert not errs, errs[:5]
    assert r.dec.status() == B.TD_OK
    r.dec.close()


@pytest.mark.parametrize("hq,hkv,P,W,n", [(2, 2, 20, 0, 3), (8, 2, 300, 0, 9), (32, 8, 1100, 0, 24), (8, 2, 600, 100, 31)])
def test_small_query_sets(hq, hkv, P, W, n):
    tree.run_tree(tree.small(prompt_min=P, prompt_max=P, n_q_heads=hq, n_kv_heads=hkv, window=W, steps=4, beam_width=6),
                  seed=32, pick=lambda tr, g: tree.every_node(tr, g)[-n:], layer_calls=[0, 1, 2])
