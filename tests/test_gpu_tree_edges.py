"""GPU parity of the tree steps at the sizes where their kernels change: one and two tokens, odd
vocabularies, the edges of a wavefront's step (128 tokens), of a workgroup's step count and of what fits
in LDS, trees around the staged size, table widths around one slot per thread, rows at odd addresses.
Lengths, paths and tokens are whole numbers, defined by fp64 evaluation of the rule: compared exactly."""
import numpy as np
import pytest
import torch

from parity_utils import random_trees

pytestmark = pytest.mark.gpu


def _step(V, k, B, M, dtype, offset, seed):
    rng = np.random.default_rng(seed)
    parent = random_trees(rng, B, M, max_children=4)
    R = B * (M + 1)
    tl = torch.from_numpy(rng.normal(0, 2.0, (R, V)).astype(np.float32)).to(dtype)
    dl = torch.from_numpy((tl.float().numpy() + rng.normal(0, 1.5, (R, V))).astype(np.float32)).to(dtype)
    row_index = (np.arange(B, dtype=np.int64)[:, None] * (M + 1) + parent + 1).astype(np.int32).reshape(-1)
    top = torch.topk(dl.float(), min(4, V), dim=1).indices.numpy()
    tokens = top[row_index, rng.integers(0, min(4, V), B * M)].astype(np.int32)
    table = ((np.arange(V, dtype=np.int64)[:, None] * 3 + np.arange(k, dtype=np.int64)[None, :]) % V).astype(np.int32)
    un = torch.from_numpy(rng.random((B * M, 2)).astype(np.float32))
    un[:, 0] = 0.5 + 0.5 * un[:, 0]

    def device(x):
        room = torch.zeros((R, V + offset), dtype=dtype, device="cuda")
        room[:, offset:].copy_(x)
        return room[:, offset:]

    rest = [torch.from_numpy(v).cuda() for v in (row_index, parent.reshape(-1), tokens, table)]
    return (tl, dl, row_index, parent, tokens, table, un), (device(tl), device(dl), *rest, un.cuda())


SHAPES = [  # V, k, B, M, dtype, first column
    (1, 1, 2, 3, torch.float32, 1), (2, 2, 3, 5, torch.bfloat16, 0), (127, 5, 4, 9, torch.bfloat16, 1),
    (129, 64, 4, 128, torch.float32, 1), (2049, 1025, 3, 129, torch.bfloat16, 3), (4096, 1024, 3, 20, torch.float32, 0),
    (4097, 1023, 3, 20, torch.bfloat16, 1), (16384, 300, 3, 12, torch.float32, 0), (16385, 65, 3, 12, torch.bfloat16, 1),
    (19200, 64, 3, 9, torch.float32, 0), (19201, 64, 3, 9, torch.bfloat16, 1)]


@pytest.mark.parametrize("divergence", ["tvd", "jsd"])
@pytest.mark.parametrize("V,k,B,M,dtype,offset", SHAPES)
def test_sequential_rule(oracle_mod, lantern_gpu, V, k, B, M, dtype, offset, divergence):
    (tl, dl, row_index, parent, tokens, table, un), dev = _step(V, k, B, M, dtype, offset, seed=V + k)
    want = oracle_mod.verify_trees_sequential(tl, dl, row_index, parent, M, tokens, table, k, 0.05, un, threads=8,
                                              divergence=divergence)
    t, d, ri, par, tok, tab, u = dev
    got = lantern_gpu.verify_trees_sequential(t, d, ri, par, M, tok, tab, 0.05, u, divergence=divergence)
    for g, w in zip(got, want):
        np.testing.assert_array_equal(g.cpu().numpy().reshape(-1), np.asarray(w).reshape(-1))


@pytest.mark.parametrize("divergence", ["tvd", "jsd"])
@pytest.mark.parametrize("V,k,B,M,dtype,offset", SHAPES)
def test_plain_rule(oracle_mod, lantern_gpu, V, k, B, M, dtype, offset, divergence):
    (tl, dl, row_index, parent, tokens, table, un), dev = _step(V, k, B, M, dtype, offset, seed=V + k)
    acc, res, _ = oracle_mod.verify_rows(tl, dl, row_index, tokens, table, k, 0.05, un, threads=8,
                                         divergence=divergence)
    want = (acc, *oracle_mod.accept_trees(acc.reshape(B, M), res.reshape(B, M), parent, M))
    t, d, ri, par, tok, tab, u = dev
    got = lantern_gpu.verify_trees(t, d, ri, par, M, tok, tab, 0.05, u, divergence=divergence)
    for g, w in zip(got, want):
        np.testing.assert_array_equal(g.cpu().numpy().reshape(-1), np.asarray(w).reshape(-1))
