"""The tree steps on rows of large finite logits: beside a maximum of 4e10 or 1e30 every lower logit, and every
filtered one, has no mass at all, and tokens at the maximum share the row.  Both sibling rules against the oracle, on
the vocabularies at which the kernel that walks or ends the step changes, large rows on either side in turn."""
import numpy as np
import pytest
import torch

from parity_utils import random_trees

pytestmark = pytest.mark.gpu

K, DELTA, B, M = 40, 0.0523, 6, 12


def _large(rng, rows, V, top, dtype):
    """Nothing at -inf is above `top`; about 30 % of the tokens lie at it or, where it has units left, around it."""
    kind = rng.random((rows, V))
    low = rng.normal(0.0, 2.0, (rows, V)) + (2 * top if top < 0 else 0.0)
    x = np.where(kind < 0.3, top + np.minimum(rng.normal(-2.0, 1.0, (rows, V)), 0.0), np.where(kind < 0.5, -np.inf, low))
    return torch.from_numpy(x.astype(np.float32)).to(dtype)


def _inputs(V, dtype, top, seed):
    rng = np.random.default_rng(seed)
    parent = random_trees(rng, B, M, max_children=4)
    R = B * (M + 1)
    tl = torch.from_numpy(rng.normal(0, 2.0, (R, V)).astype(np.float32)).to(dtype)
    dl = torch.from_numpy((tl.float().numpy() + rng.normal(0, 1.5, (R, V))).astype(np.float32)).to(dtype)
    large = _large(rng, R, V, top, dtype), _large(rng, R, V, top, dtype)
    side = np.arange(B).repeat(M + 1) % 3                     # per tree: the target, the drafter, both
    tl[torch.from_numpy(side != 1)] = large[0][torch.from_numpy(side != 1)]
    dl[torch.from_numpy(side != 0)] = large[1][torch.from_numpy(side != 0)]
    row_index = (np.arange(B, dtype=np.int64)[:, None] * (M + 1) + parent + 1).astype(np.int32).reshape(-1)
    top4 = torch.topk(dl.float(), 4, dim=1).indices.numpy()
    tokens = top4[row_index, rng.integers(0, 4, B * M)].astype(np.int32)
    table = ((np.arange(V, dtype=np.int64)[:, None] + 3 * np.arange(K, dtype=np.int64)[None, :]) % V).astype(np.int32)
    un = torch.from_numpy(rng.random((B * M, 2)).astype(np.float32))
    un[:, 0] = 0.9 + 0.1 * un[:, 0]
    dev = [t.cuda() for t in (tl, dl, torch.from_numpy(row_index), torch.from_numpy(parent.reshape(-1).copy()),
                              torch.from_numpy(tokens), torch.from_numpy(table), un)]
    return (tl, dl, row_index, parent, tokens, table, un), dev


@pytest.mark.parametrize("top", [1e6, 4e10, 1e30, -1e30])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("V", [1003, 8192, 8200, 16384, 19200, 19201])
def test_large_logits(oracle_mod, lantern_gpu, V, dtype, top):
    drawn = 0
    for seed in range(2):
        (tl, dl, row_index, parent, tokens, table, un), (t, d, ri, par, tok, tab, u) = _inputs(V, dtype, top, 100 * V + seed)
        want = oracle_mod.verify_trees_sequential(tl, dl, row_index, parent, M, tokens, table, K, DELTA, un, threads=8)
        got = lantern_gpu.verify_trees_sequential(t, d, ri, par, M, tok, tab, DELTA, u)
        drawn += int((np.asarray(want[2]) >= 0).sum())
        for name, g, w in zip(("len", "path", "next"), got, want):
            np.testing.assert_array_equal(g.cpu().numpy().reshape(-1), np.asarray(w).reshape(-1), err_msg=f"sequential {name}")
        acc, res, _ = oracle_mod.verify_rows(tl, dl, row_index, tokens, table, K, DELTA, un, threads=8)
        want = (acc, *oracle_mod.accept_trees(acc.reshape(B, M), res.reshape(B, M), parent, M))
        got = lantern_gpu.verify_trees(t, d, ri, par, M, tok, tab, DELTA, u)
        for name, g, w in zip(("accept", "len", "path", "next"), got, want):
            np.testing.assert_array_equal(g.cpu().numpy().reshape(-1), np.asarray(w).reshape(-1), err_msg=f"plain {name}")
    assert drawn > 0
