"""The fp32 matrix-instruction attention (fp32, and bf16 beyond the matrix-core head dims) at
the sizes where its tiling can go wrong, against the CPU oracle, and its treatment of
non-finite values in nodes that a beam does not see."""
import numpy as np
import pytest

import paper_2502_00085_amd.binding as B
import synth
from gpu_harness import Run, from_dev, log

pytestmark = pytest.mark.gpu


def small(**kw):
    base = dict(name="small", cfg_id=410, n_layers=2, n_q_heads=8, n_kv_heads=2, head_dim=64, dtype="f32",
                n_tries=1, prompt_min=47, prompt_max=47, beam_width=4, steps=4, vocab=600, window=0, alpha=1.0,
                qkv_std=1.0, logit_std=3.0, gc_interval=1)
    base.update(kw)
    return synth.Workload(**base)


# (prompt, beams, q heads): 16-node tiles with 1, 15, 16, 17 nodes and several per wave; 1, 16,
# 17, 32 and 33 query rows per KV head (one and two 16-row tiles, a second block)
@pytest.mark.parametrize("dtype,d", [("f32", 32), ("f32", 96), ("f32", 128), ("f32", 224), ("f32", 256),
                                     ("bf16", 32), ("bf16", 160), ("bf16", 192), ("bf16", 256)])
@pytest.mark.parametrize("prompt,beams,q_heads", [(1, 1, 2), (15, 4, 8), (16, 17, 2), (260, 8, 8), (1061, 11, 6)])
def test_tiles_and_row_blocks(dtype, d, prompt, beams, q_heads):
    w = small(dtype=dtype, head_dim=d, prompt_min=prompt, prompt_max=prompt, beam_width=beams, n_q_heads=q_heads)
    log(f"mfma32 {dtype} d={d} P={prompt} b={beams} Hq={q_heads}")
    r = Run(w, seed=3, layer_calls=[0, 1, 2] if prompt == 260 else None)
    for _ in range(w.steps):
        errs, _ = r.step()
        assert not errs, errs[:5]
    assert r.dec.status() == B.TD_OK
    r.dec.close()


@pytest.mark.parametrize("dtype,d,beams", [("f32", 64, 4), ("f32", 128, 8), ("bf16", 160, 4)])
def test_hidden_nodes_with_non_finite_values(dtype, d, beams):
    """NaN and infinite K/V in the nodes of some beams' paths leave the other beams' outputs as
    they were (their tiles take another order of additions: a few fp32 roundings)."""
    import torch
    w = small(dtype=dtype, head_dim=d, beam_width=beams, n_q_heads=8, alpha=0.0, steps=6)
    r = Run(w, seed=5, oracle=False)
    for _ in range(w.steps):
        r.step(check=False)
    st = r.dec.read_state(0)
    q, kn, vn, logits, _, _ = r.inputs(w.steps + 1)
    qd, knd, vnd, _ = r.dev_inputs(w.steps + 1, q, kn, vn, logits)
    out = [torch.empty_like(qd) for _ in range(2)]
    r.dec.attn_decode(0, w.n_layers, qd, knd, vnd, out[0], r.scale)  # stores the leaves
    r.dec.attn_decode(0, w.n_layers, qd, None, None, out[0], r.scale)
    some = [i for i in range(st["n_nodes"]) if st["mask"][i] & np.uint64(1) and not st["mask"][i] & np.uint64(2)]
    assert some
    seen = np.uint64(0)
    for i, bad in zip(some, [float("nan"), float("inf")] * len(some)):
        r.dec.v_pool[:, :, :, st["base"] + i, ::3] = bad
        r.dec.k_pool[:, :, :, st["base"] + i, 1::5] = bad
        seen |= st["mask"][i]
    r.dec.attn_decode(0, w.n_layers, qd, None, None, out[1], r.scale)
    a, b = (from_dev(x) for x in out)
    clean = [j for j in range(beams) if not int(seen) >> j & 1]
    assert 1 in clean and 0 not in clean
    assert not np.array_equal(a[:, :, 0], b[:, :, 0])
    tol = 2.0 ** -20 if dtype == "f32" else 2.0 ** -7  # roundings of one order of sums; of bf16 outputs
    assert np.all(np.abs(a[:, :, clean] - b[:, :, clean]) <= tol * np.abs(a).max())
    r.dec.close()
