"""Rejected rows through the one-pass fp64 evaluation, and the rows it hands to the general path: more tokens on the
list of undecided signs than it holds, logits too far from zero, filtered tokens on either side."""
import numpy as np
import pytest
import torch

from parity_utils import compare_verify, random_table

pytestmark = pytest.mark.gpu

N = 8


def _inputs(kind, V, dtype, seed):
    rng = np.random.default_rng(seed)
    target = torch.from_numpy((1.5 * rng.standard_normal((N, V))).astype(np.float32))
    if kind == "list":
        # the drafter's row is the target's with two tokens exchanged: the other probabilities agree, so the sign of
        # every residual but theirs is open in fp32
        target = target.to(dtype)
        draft = target.clone()
        lo, hi = target.float().argmin(dim=1), target.float().argmax(dim=1)
        rows = torch.arange(N)
        draft[rows, lo], draft[rows, hi] = target[rows, hi], target[rows, lo]
        tokens = lo.to(torch.int32)
    else:
        draft = target + torch.from_numpy(rng.standard_normal((N, V)).astype(np.float32))
        wide = 20.0 if dtype == torch.bfloat16 else 1.0      # bf16 has steps of 16 and 32 there
        if kind == "near":          # the reference logits just inside what the pass takes
            target, draft = wide * target + 3900.0, wide * draft - 3900.0
        if kind == "far":
            target, draft = wide * target + 5000.0, wide * draft - 5000.0
        if kind == "filtered":
            target[torch.from_numpy(rng.random((N, V)) < 0.3)] = -float("inf")
            draft[torch.from_numpy(rng.random((N, V)) < 0.3)] = -float("inf")
            draft[:, V // 3] = target[:, V // 2] = -float("inf")
            draft[:, V // 2] = 0.5
        target, draft = target.to(dtype), draft.to(dtype)
        tokens = draft.float().argmax(dim=1).to(torch.int32)
        if kind == "filtered":
            tokens[::2] = V // 2    # t(xt) = 0
    uniforms = torch.from_numpy(rng.random((N, 2)).astype(np.float32))
    uniforms[:, 0] = 1 - 2.0 ** -24
    uniforms[1, 0] = uniforms[2, 0] = uniforms[2, 1] = 0.0
    return target, draft, tokens, uniforms


@pytest.mark.parametrize("kind", ["list", "near", "far", "filtered"])
@pytest.mark.parametrize("dtype,V", [(torch.float32, 1024), (torch.float32, 8192), (torch.float32, 4004), (torch.float32, 12288),
                                     (torch.bfloat16, 2040), (torch.bfloat16, 16384), (torch.bfloat16, 24576),
                                     (torch.bfloat16, 33000)])
def test_kinds_of_rows(oracle_mod, lantern_gpu, dtype, V, kind):
    target, draft, tokens, uniforms = _inputs(kind, V, dtype, V)
    table = random_table(V, 40, seed=3) if V <= 4096 else \
        ((np.arange(V)[:, None] + np.concatenate([[0], 1 + np.random.default_rng(V).permutation(V - 1)[:39]])[None, :]) % V).astype(np.int32)
    for delta in (0.0, 0.02):
        acc, *_ = compare_verify(oracle_mod, lantern_gpu, target, draft, tokens, table, delta, uniforms,
                                 label=f"{kind} V={V} {dtype} delta={delta}")
        assert (acc == 0).any()


@pytest.mark.parametrize("below", [620.0, 668.0, 715.0])
@pytest.mark.parametrize("dtype,V", [(torch.float32, 1024), (torch.float32, 8192), (torch.bfloat16, 2040), (torch.bfloat16, 16384),
                                     (torch.bfloat16, 33000)])
def test_draw_of_exactly_zero(oracle_mod, lantern_gpu, dtype, V, below):
    """A draw of zero takes the first token that has any residual at all: here one that lies hundreds of nats below the
    row's maximum and is filtered on the drafter's side."""
    target, draft, tokens, uniforms = _inputs("plain", V, torch.float32, V + 1)
    first = 3
    target[:, first], draft[:, :first + 1] = target.max(dim=1).values - below, -float("inf")
    target[:, :first] = -float("inf")
    tokens = draft.to(dtype).float().argmax(dim=1).to(torch.int32)
    uniforms[:, 0], uniforms[:, 1] = 1 - 2.0 ** -24, 0.0
    table = np.arange(V, dtype=np.int32)[:, None]
    acc, res, *_ = compare_verify(oracle_mod, lantern_gpu, target.to(dtype), draft.to(dtype), tokens, table, 0.0, uniforms,
                                  label=f"V={V} {dtype} {below} below")
    assert (res[acc == 0] == first).all() and (acc == 0).any()
