"""One-layer attention calls over the ranges of the node-split rule (4-wave and 8-wave workgroups,
one to 32 splits, one to four row blocks, the row blocks of a range on one XCD or not), against the
CPU oracle: tries of one tile, of a tile more or less than a workgroup's share, and larger."""
import numpy as np
import pytest

import paper_2502_00085_amd.binding as B
import synth
import test_gpu_tree_attn as tree
from gpu_harness import Run, log
from test_gpu_parity import small

pytestmark = pytest.mark.gpu


# (tries, beams, q heads, KV heads, prompt, window): units of 1 .. 160, rows of 1 .. 96 per KV head;
# tries that grow past the unsplit ones (256 nodes, 192 under two row blocks per workgroup); three and
# four row blocks over 5, 6 and 12 ranges, which do not divide over the XCDs by themselves
@pytest.mark.parametrize("T,b,hq,hkv,P,W", [
    (1, 1, 1, 1, 5, 0), (1, 4, 4, 1, 31, 0), (1, 4, 8, 2, 127, 0), (1, 8, 32, 8, 1025, 0), (1, 8, 8, 2, 4200, 0),
    (1, 16, 8, 2, 700, 0), (2, 24, 8, 2, 129, 0), (2, 24, 8, 2, 90, 33), (1, 3, 8, 8, 2300, 1100),
    (16, 4, 8, 8, 70, 0), (20, 4, 16, 8, 150, 0), (1, 8, 8, 2, 245, 0), (1, 16, 8, 2, 180, 0), (1, 24, 24, 6, 700, 0),
    (5, 25, 4, 1, 400, 0), (3, 24, 16, 4, 330, 200)])
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


@pytest.mark.parametrize("hq,hkv,P,W,n", [(2, 2, 20, 0, 3), (8, 2, 300, 0, 9), (32, 8, 1100, 0, 24), (8, 2, 600, 100, 31),
                                          (8, 2, 225, 0, 20), (24, 6, 700, 0, 30)])
def test_small_query_sets(hq, hkv, P, W, n):
    tree.run_tree(tree.small(prompt_min=P, prompt_max=P, n_q_heads=hq, n_kv_heads=hkv, window=W, steps=4, beam_width=6),
                  seed=32, pick=lambda tr, g: tree.every_node(tr, g)[-n:], layer_calls=[0, 1, 2])


@pytest.mark.parametrize("beams,q_heads,kv_heads,dtype,d,P,steps", [
    (16, 16, 8, "bf16", 128, 100, 260), (8, 8, 2, "f32", 64, 100, 100), (4, 4, 1, "bf16", 192, 20, 150)])
def test_reading_the_state_changes_no_output(beams, q_heads, kv_heads, dtype, d, P, steps):
    """A trie that collections keep far below b nodes per step: the attention before and after
    td_read_state is the same, bit for bit (over the layers: another order of sums would change
    several bf16 roundings)."""
    import torch
    L = 24
    w = small(beam_width=beams, n_q_heads=q_heads, n_kv_heads=kv_heads, prompt_min=P, prompt_max=P, head_dim=d,
              dtype=dtype, n_layers=L, steps=steps, vocab=200, alpha=2.0)
    log(f"read_state b={beams} Hq={q_heads} Hkv={kv_heads} {dtype} d={d}")
    r = Run(w, seed=33, oracle=False, input_period=1)
    q, kn, vn, logits, _, _ = r.inputs(1)
    qd, knd, vnd, ld = r.dev_inputs(1, q, kn, vn, logits)
    sel = [torch.empty((1, beams), dtype=t, device="cuda") for t in (torch.int32, torch.int32, torch.float32, torch.float32, torch.float32)]
    out = [torch.empty_like(qd) for _ in range(2)]
    for s in range(w.steps):  # (the harness reads the state at every step: these do not)
        r.dec.attn_decode(0, L, qd, knd if s else None, vnd if s else None, out[0], r.scale)
        par, tok = (torch.from_numpy(x).cuda() for x in synth.step_script(w, s + 1, 33))
        r.dec.topk_append(ld, *sel, par, tok, torch.empty((1, beams), device="cuda"))
    r.dec.attn_decode(0, L, qd, knd, vnd, out[0], r.scale)  # stores the leaves

    def layers(o):
        for l in range(L):
            r.dec.attn_decode(l, 1, qd[l:l + 1], None, None, o[l:l + 1], r.scale)

    layers(out[0])
    assert r.dec.read_state(0)["n_nodes"] < P + steps * beams - 400
    layers(out[1])
    assert torch.equal(out[0], out[1])
    assert r.dec.status() == B.TD_OK
    r.dec.close()


@pytest.mark.parametrize("window", [0, 60])
def test_a_captured_step_on_a_growing_trie(window):
    """One step, captured on a trie of few nodes and replayed while it grows to many tiles per
    wave, against the same steps launched one by one."""
    import torch
    w = small(beam_width=8, n_q_heads=8, n_kv_heads=2, prompt_min=20, prompt_max=20, n_layers=2, steps=130, vocab=300,
              alpha=0.0, window=window)
    log(f"captured step W={window}")
    runs = [Run(w, seed=34, oracle=False, fused=True, input_period=1, mode="driven", capacity=3000) for _ in range(2)]
    for r in runs:
        r.step(check=False)
    q, kn, vn, logits, _, _ = runs[0].inputs(1)
    qd, knd, vnd, ld = runs[0].dev_inputs(1, q, kn, vn, logits)
    sel = [torch.empty((1, 8), dtype=t, device="cuda") for t in (torch.int32, torch.int32, torch.float32, torch.float32, torch.float32)]
    out = [torch.empty_like(qd) for _ in range(2)]

    def step(r, o):
        for l in range(2):
            r.dec.attn_decode(l, 1, qd[l:l + 1], knd[l:l + 1], vnd[l:l + 1], o[l:l + 1], r.scale)
        r.dec.topk_append(ld, *sel)

    step(runs[0], out[0])
    graph, cs = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    with torch.cuda.graph(graph, stream=cs):
        step(runs[1], out[1])
    for i in range(w.steps - 2):
        if i:
            step(runs[0], out[0])
        graph.replay()
        torch.cuda.synchronize()
        a, b = (o.float() for o in out)
        assert float((a - b).abs().max()) <= 2.0 ** -7 * float(a.abs().max())  # (bf16 outputs; sums in another order)
    a, b = (r.dec.read_state(0) for r in runs)
    for k in ("n_nodes", "node_id", "parent_slot", "token", "depth", "mask", "leaf_slot", "leaf_score"):
        assert np.array_equal(np.asarray(a[k]), np.asarray(b[k])), k
    for r in runs:
        assert r.dec.status() == B.TD_OK
        r.dec.close()
