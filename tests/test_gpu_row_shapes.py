"""Rows of any length at any address through the fp32 pass and the residual draw of lantern_verify (Section 4.3;
Algorithm 1, accept / resample branch): the edges of the 256, 512 and 1024 thread variants, one vector, partial
last vectors, rows that start between two vectors.  Decisions and tokens are compared exactly."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

EDGES = {torch.bfloat16: [8, 9, 15, 2048, 2055, 16383, 16384, 16385, 32768, 32771, 65535, 65536, 65537],
         torch.float32: [4, 5, 7, 1025, 8192, 8193, 16384, 16386, 32767, 32768, 32769]}


def _inputs(V, k, N, dtype, start, seed):
    rng = np.random.default_rng(seed)
    stride = V + start + int(rng.integers(0, 9))
    wide = torch.from_numpy(rng.standard_normal((2, N, stride)).astype(np.float32))
    target = (2.5 * wide[0]).to(dtype)
    draft = (2.5 * wide[0] + wide[1]).to(dtype)
    tokens = draft[:, start:start + V].float().argmax(dim=1).to(torch.int32)
    offsets = np.concatenate([[0], 1 + rng.permutation(V - 1)[:k - 1]])
    table = ((np.arange(V)[:, None] + offsets[None, :]) % V).astype(np.int32)
    uniforms = torch.from_numpy(rng.random((N, 2)).astype(np.float32))
    uniforms[::2, 0] = 1 - 2.0 ** -24
    return target, draft, tokens, torch.from_numpy(table), uniforms


@pytest.mark.parametrize("start", [0, 3])
@pytest.mark.parametrize("dtype,V", [(dt, V) for dt, sizes in EDGES.items() for V in sizes])
def test_edges(oracle_mod, lantern_gpu, dtype, V, start):
    N, k = 6, min(V, 50 + V % 3)
    target, draft, tokens, table, uniforms = _inputs(V, k, N, dtype, start, V + start)
    dev = [x.cuda() for x in (target, draft, tokens, table, uniforms)]
    t_dev, g_dev = dev[0][:, start:start + V], dev[1][:, start:start + V]
    for delta in (0.0, 0.05):
        acc, res, _ = oracle_mod.verify(target[:, start:start + V].contiguous(), draft[:, start:start + V].contiguous(),
                                        tokens, table.numpy(), k, delta, uniforms, threads=6)
        got_acc, got_res = lantern_gpu.verify(t_dev, g_dev, dev[2], dev[3], delta, dev[4])
        np.testing.assert_array_equal(got_acc.cpu().numpy(), acc)
        np.testing.assert_array_equal(got_res.cpu().numpy(), res)
        decided = lantern_gpu.decide_rows(t_dev, g_dev, None, dev[2], dev[3], delta, dev[4])
        np.testing.assert_array_equal(decided.cpu().numpy(), acc)


@pytest.mark.parametrize("dtype,V", [(torch.bfloat16, 5001), (torch.bfloat16, 40001), (torch.float32, 9002)])
def test_filtered_and_unusable_rows(oracle_mod, lantern_gpu, dtype, V):
    """-inf logits (filtered tokens), a NaN in the last, partial vector, and a token out of range."""
    start, N, k = 1, 6, 40
    target, draft, tokens, table, uniforms = _inputs(V, k, N, dtype, start, V)
    target[1, start + V // 2:start + V] = -float("inf")
    draft[1, start + V // 2:start + V] = -float("inf")
    tokens[1] = 0
    target[2, start + V - 1] = float("nan")
    draft[3, start + V - 1] = float("inf")
    tokens[4] = V
    dev = [x.cuda() for x in (target, draft, tokens, table, uniforms)]
    acc, res, _ = oracle_mod.verify(target[:, start:start + V].contiguous(), draft[:, start:start + V].contiguous(),
                                    tokens, table.numpy(), k, 0.02, uniforms, threads=6)
    got_acc, got_res = lantern_gpu.verify(dev[0][:, start:start + V], dev[1][:, start:start + V], dev[2], dev[3], 0.02,
                                          dev[4])
    np.testing.assert_array_equal(got_acc.cpu().numpy(), acc)
    np.testing.assert_array_equal(got_res.cpu().numpy(), res)
    assert list(acc[2:5]) == [-1, -1, -1]
