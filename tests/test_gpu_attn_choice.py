"""The choice between the two fp32-arithmetic decode kernels (the fp32 matrix instructions and the
vector ALU) on both sides of its line, against the CPU oracle: nodes, query rows, units, types and
head dims, with a window, deferred collections, moved rows and calls per layer.  A run that forces
the vector ALU gives the same bits where it is the choice, and other ones where it is not."""
import numpy as np
import pytest

import paper_2502_00085_amd.binding as B
import synth
from gpu_harness import Run, log

pytestmark = pytest.mark.gpu


def case(dtype, d, beams, q_heads, kv_heads, prompt, layers, **kw):
    base = dict(name="choice", cfg_id=420, n_layers=layers, n_q_heads=q_heads, n_kv_heads=kv_heads, head_dim=d, dtype=dtype,
                n_tries=1, prompt_min=prompt, prompt_max=prompt, beam_width=beams, steps=4, vocab=500, window=0, alpha=1.0,
                qkv_std=1.0 / np.sqrt(d), logit_std=3.0, gc_interval=1)
    base.update(kw)
    return synth.Workload(**base)


VALU, MFMA = True, False
LAYERS = "one call per layer"
CASES = [
    # bf16 at d = 160: one workgroup's round, a few nodes more, more than the vector ALU is good for
    (case("bf16", 160, 3, 2, 1, 100, 12), LAYERS, MFMA),
    (case("bf16", 160, 3, 2, 1, 200, 3), LAYERS, VALU),
    (case("bf16", 192, 4, 8, 2, 400, 2), LAYERS, VALU),
    (case("bf16", 160, 4, 8, 2, 1500, 12, steps=2), LAYERS, MFMA),
    # 4 waves per workgroup (d past 192; 17 and more rows past 128)
    (case("bf16", 256, 4, 4, 1, 50, 12), LAYERS, MFMA),
    (case("bf16", 256, 4, 4, 1, 70, 3), LAYERS, VALU),
    (case("bf16", 224, 4, 16, 4, 800, 12, steps=2), LAYERS, MFMA),
    (case("bf16", 256, 6, 4, 1, 50, 3), LAYERS, VALU),
    (case("bf16", 192, 20, 4, 2, 300, 2), LAYERS, VALU),
    (case("f32", 256, 12, 16, 4, 900, 2, steps=2), LAYERS, MFMA),
    # few rows, many units: unsplit launches, moved rows and leaves stored by the attention itself
    (case("bf16", 256, 4, 32, 32, 66, 6, alpha=0.0, steps=8), None, VALU),
    (case("f32", 224, 2, 32, 32, 90, 6, alpha=0.0, steps=8, window=80, gc_interval=3), None, VALU),
    (case("f32", 160, 4, 32, 32, 60, 6, alpha=0.0, steps=8), None, MFMA),
    # a window and deferred collections, split
    (case("bf16", 192, 8, 8, 4, 260, 3, steps=9, window=150, gc_interval=4, alpha=0.0), LAYERS, VALU),
    # several tries
    (case("f32", 256, 5, 4, 2, 90, 2, n_tries=3, prompt_min=40), LAYERS, VALU),
    # fp32 at the bf16 kernel's head dims: 17 and more rows in small calls
    (case("f32", 128, 8, 16, 4, 150, 2), LAYERS, VALU),
    (case("f32", 128, 8, 16, 4, 900, 2, steps=2), LAYERS, MFMA),
    (case("f32", 128, 4, 16, 4, 150, 2), LAYERS, MFMA),
    (case("f32", 96, 8, 16, 4, 150, 2), LAYERS, VALU),
    (case("f32", 96, 8, 16, 4, 400, 2), LAYERS, MFMA),
    (case("bf16", 32, 8, 16, 4, 150, 6), LAYERS, MFMA),
]


@pytest.mark.parametrize("w,calls,choice", CASES, ids=lambda x: f"{x.dtype}-d{x.head_dim}-b{x.beam_width}-q{x.n_q_heads}-P{x.prompt_max}"
                         if isinstance(x, synth.Workload) else None)
def test_both_sides(w, calls, choice):
    log(f"choice {w.dtype} d={w.head_dim} b={w.beam_width} Hq={w.n_q_heads} Hkv={w.n_kv_heads} P={w.prompt_max} L={w.n_layers}")
    calls = list(range(w.n_layers + 1)) if calls else None
    auto = Run(w, seed=41, layer_calls=calls, layers=[0, w.n_layers - 1])
    valu = Run(w, seed=41, layer_calls=calls, oracle=False, attn_impl=B.TD_ATTN_VALU)
    same = True
    for _ in range(w.steps):
        errs, res = auto.step()
        assert not errs, errs[:5]
        _, ref = valu.step()
        same = same and np.array_equal(res["o"], ref["o"])
    assert same == choice
    for r in (auto, valu):
        assert r.dec.status() == B.TD_OK
        r.dec.close()
