"""td_init_prompt over its launch shapes: prompts shorter and longer than one workgroup's slots, and
more tries than one launch takes; a second prompt replaces the first and empties the pool of
finished hypotheses."""
import numpy as np
import pytest

import paper_2502_00085_amd.binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,lengths", [(1, [1]), (1, [1024]), (2, [1025, 3]), (3, [2049, 1023, 4096]), (64, [5]), (70, [9, 1500])])
def test_states(T, lengths):
    import torch
    g = np.random.default_rng(T)
    dec = B.TrieDecoder(T, 2, 4200, 50, 1, 1, 1, 32, eos_token=7)
    for shift in (0, 1):
        lens = [lengths[(t + shift) % len(lengths)] for t in range(T)]
        tokens = g.integers(0, 50, (T, max(lens) + shift)).astype(np.int32)
        dec.init_prompt(lens, torch.from_numpy(tokens).cuda())
        for t in range(T):
            st, n = dec.read_state(t), lens[t]
            assert (st["n_nodes"], st["n_live"], st["n_shared"], st["next_id"], st["step"], st["base"]) == (n, 1, n, n, 0, 0)
            for k, want in (("node_id", np.arange(n)), ("parent_slot", np.arange(n) - 1), ("depth", np.arange(n)),
                            ("token", tokens[t, :n]), ("mask", np.ones(n, np.uint64)), ("leaf_slot", [n - 1])):
                assert np.array_equal(st[k], want), k
            assert st["leaf_score"].tolist() == [0.0]
            f = dec.read_finished(t)
            assert f["count"] == 0 and not f["done"]
    dec.close()
