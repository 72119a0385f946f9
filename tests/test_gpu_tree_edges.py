"""GPU parity of the tree steps at the sizes where their kernels change: one and two tokens, odd
vocabularies, the edges of a wavefront's step (128 tokens), of a workgroup's step count and of what fits
in LDS, trees around the staged size, table widths around one slot per thread, rows at odd addresses.
Lengths, paths and tokens are whole numbers, defined by fp64 evaluation of the rule: compared exactly."""
import numpy as np
import pytest
import torch

from parity_utils import random_trees, replay_us

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


@pytest.mark.parametrize("divergence", ["tvd", "jsd"])
@pytest.mark.parametrize("V,k,B,M,dtype,offset", [
    # the lines between the two kernels that end a plain step: aligned rows at 8192 tokens, others at 2048, both at
    # 12288 where there are more trees than compute units
    (8192, 40, 3, 70, torch.bfloat16, 0), (8200, 40, 3, 70, torch.bfloat16, 0), (8196, 40, 257, 3, torch.float32, 0),
    (8196, 40, 256, 3, torch.float32, 0), (2048, 33, 3, 20, torch.float32, 1), (2049, 33, 257, 2, torch.bfloat16, 1),
    (2050, 33, 256, 2, torch.float32, 3), (12288, 64, 257, 2, torch.bfloat16, 0), (12296, 64, 257, 2, torch.bfloat16, 0),
    (5001, 1100, 2, 300, torch.bfloat16, 1)])
def test_plain_rule_between_the_kernels(oracle_mod, lantern_gpu, V, k, B, M, dtype, offset, divergence):
    test_plain_rule(oracle_mod, lantern_gpu, V, k, B, M, dtype, offset, divergence)


@pytest.mark.parametrize("dtype,V,draw,limit", [(torch.float32, 1024, True, 1.2), (torch.bfloat16, 4096, True, 1.2),
                                                (torch.float32, 8192, False, 0.65), (torch.bfloat16, 16384, False, 0.4)])
def test_what_follows_the_decisions_costs_little(lantern_gpu, dtype, V, draw, limit):
    """A plain step of 64 trees less its decisions, against lantern_resample_selected of 64 candidates.  With every
    candidate rejected both draw from a row: the same time.  With every candidate accepted the walk remains, against
    finding that there is nothing to draw: 0.25 to 0.36 times (V = 8192) and 0.22 to 0.25 (16384).  With a walk that
    stages the tree in 1024 threads first it was 1.3 to 1.5 times with the draw, and 0.76 to 0.87 and 0.50 to 0.57 without."""
    B, M, k = 64, 60, 100
    parent = random_trees(np.random.default_rng(V), B, M, max_children=4)
    g = torch.Generator(device="cuda").manual_seed(V)
    target = torch.randn(B * M, V, generator=g, device="cuda").to(dtype)
    draft = (target.float() + 0.3 * torch.randn(B * M, V, generator=g, device="cuda")).to(dtype)
    tokens = (draft.float() - target.float()).argmax(dim=1).to(torch.int32)
    uniforms = torch.full((B * M, 2), 1 - 2.0 ** -24 if draw else 0.0, device="cuda")
    table = ((torch.arange(V, device="cuda")[:, None] + torch.arange(k, device="cuda")[None, :]) % V).to(torch.int32)
    par = torch.from_numpy(parent.reshape(-1)).cuda()
    lantern_gpu.prepare(dtype, V, k)
    select = torch.arange(0, B * M, M, dtype=torch.int32, device="cuda")
    step, decide, draws = replay_us(
        lambda: lantern_gpu.verify_trees(target, draft, None, par, M, tokens, table, 0.0, uniforms),
        lambda: lantern_gpu.decide_rows(target, draft, None, tokens, table, 0.0, uniforms),
        lambda: lantern_gpu.resample_selected(target, draft, None, tokens, table, 0.0, uniforms, select))
    accepted = lantern_gpu.decide_rows(target, draft, None, tokens, table, 0.0, uniforms)
    assert int((accepted == 1).sum()) == (0 if draw else B * M)
    assert step - decide < limit * draws, (step, decide, draws)
