"""The chunk pass of the selection on logits where its per-value shortcuts can go wrong: both zeros,
equal largest logits in one sub-chunk (one lane, one run, several runs), values far below the
row's maximum (of any magnitude) and -inf, against the oracle's ranking of every candidate.  Bit
for bit."""
import numpy as np
import pytest

import oracle.beam as obeam
import paper_2502_00085_amd.binding as B

pytestmark = pytest.mark.gpu


def run(logits, scores, b):
    import torch
    T, n, V = logits.shape
    i32, f32 = dict(dtype=torch.int32, device="cuda"), dict(dtype=torch.float32, device="cuda")
    sel = [torch.empty((T, b), **i32), torch.empty((T, b), **i32), torch.empty((T, b), **f32), torch.empty((T, b), **f32)]
    lse, status = torch.empty((T, b), **f32), torch.empty(2, **i32)
    B.beam_topk_static(T, b, V, torch.from_numpy(logits).cuda(), torch.full((T,), n, **i32),
                       torch.from_numpy(scores).cuda(), *sel, lse, status)
    torch.cuda.synchronize()
    assert status.tolist() == [0, 0]
    par, tok, sc, lp, lse = (x.cpu().numpy() for x in (*sel, lse))
    for t in range(T):
        ref = obeam.select(logits[t], scores[t], b)
        assert np.array_equal(par[t], ref["sel_parent"]) and np.array_equal(tok[t], ref["sel_token"])
        for got, want in ((sc[t], ref["sel_score"]), (lp[t], ref["sel_logprob"]), (lse[t], ref["lse"])):
            assert np.array_equal(got.view(np.uint32), want.view(np.uint32))


# (tries, beams, V): chunk passes of 16-wave and 4-wave workgroups, whole chunks and a ragged last one
@pytest.mark.parametrize("T,b,V", [(1, 4, 4096), (2, 3, 8200), (9, 16, 16384), (8, 16, 20000)])
@pytest.mark.parametrize("kind", ["ties", "zeros", "deep", "peaks"])
def test_edges(T, b, V, kind):
    g = np.random.default_rng(7)
    x = (g.standard_normal((T, b, V)) * 3).astype(np.float32)
    if kind == "ties":  # few distinct values: equal logits in every sub-chunk
        x = np.round(x * 2) / 2
    elif kind == "zeros":  # the largest logits are -0 and +0
        x = -np.abs(np.round(x)) * np.float32(1.0)
        x[..., ::7] = 0.0
        x[..., ::11] = -0.0
    elif kind == "deep":  # far below the maximum, and masked
        x = x * np.float32(200.0)
        x[..., ::3] = -np.inf
        x[..., 5::8] = np.float32(-3e38)
    else:  # one lane's four logits of a sub-chunk, and one run's, are the largest and equal
        x[:, :, 70] = x[:, :, 1094] = x[:, :, 2118] = x[:, :, 3142] = np.float32(12.5)
        x[:, :, 128:192] = np.float32(12.0)
    run(np.ascontiguousarray(x, np.float32), -np.sort(g.random((T, b)) * 4).astype(np.float32), b)


def test_one_finite_logit():
    # lse = 0: the sign of a zero logit reaches the log-probability
    for zero in (0.0, -0.0):
        x = np.full((1, 1, 4096), -np.inf, np.float32)
        x[0, 0, 2055] = zero
        run(x, np.zeros((1, 1), np.float32), 1)


# Around these maxima the floats are 32, 256, 1,024, 2,048 and far more apart: 700 below the
# maximum is no float.  Chunks with lower logits just below, far below, of the type's lowest and -inf.
@pytest.mark.parametrize("T,b,V", [(1, 4, 4096), (2, 3, 8200), (9, 16, 16384)])
@pytest.mark.parametrize("m", [5e8, 3e9, 1e10, 2e10, 3e38, -5e8, -3e9, -1e10, -2e10, -3e38])
@pytest.mark.parametrize("rest", ["near", "far", "masked"])
def test_large_maxima(T, b, V, m, rest):
    g = np.random.default_rng(11)
    top = np.float32(m)
    if rest == "near":  # up to 40 floats below
        x = (top.view(np.int32) + (-1 if m > 0 else 1) * g.integers(0, 40, (T, b, V), dtype=np.int32)).view(np.float32)
    elif rest == "far":
        x = np.minimum(top - np.float32(1000.0), np.float32(-abs(m)) * g.uniform(1, 1.1, (T, b, V)).astype(np.float32))
        x[..., ::5] = np.finfo(np.float32).min
    else:
        x = np.full((T, b, V), -np.inf, np.float32)
    x[..., 17::509] = top  # several of the largest in every chunk
    x[..., 3::64] = -np.inf
    run(np.ascontiguousarray(x, np.float32), -np.sort(g.random((T, b)) * 4).astype(np.float32), b)
