"""The tree step under the sequential rule decides the first child of every node beforehand and no other candidate:
parity with the oracle where the search for earlier siblings can go wrong (trees of 1 .. 200 nodes, siblings in
different steps of 64, rows for the fp32 pass and for the fp64 path), with decisions left over in the workspace that
would be accepted if they were read."""
import numpy as np
import pytest
import torch

from synth import workloads
from parity_utils import random_table, random_trees, tree_step

pytestmark = pytest.mark.gpu


def _far_siblings(B, M):
    """Node i and node i + M/2 are siblings: every later child lies half a tree behind its first one."""
    half = max(1, M // 2)
    parent = np.empty((B, M), dtype=np.int32)
    for i in range(M):
        parent[:, i] = (i % half) - 1
    return parent


@pytest.mark.parametrize("V,k", [(1024, 16), (1003, 16), (2048, 1100)])    # whole vectors, odd rows, beyond the scan
@pytest.mark.parametrize("M", [1, 64, 65, 129, 200])
def test_first_children(oracle_mod, lantern_gpu, V, k, M):
    cfg = workloads.Config("first", V, 8, "f32", True, k, 0.3, 64, 1, "f32", 1.5, 0.5, index=60)
    table = random_table(V, k, seed=M)
    B = 4
    later = 0
    for step, parent in enumerate((_far_siblings(B, M), random_trees(np.random.default_rng(M), B, M, max_children=5))):
        st, row_index, tokens, un = tree_step(cfg, parent, step=step, variant="peaked")
        n_o, path_o, next_o = oracle_mod.verify_trees_sequential(st.target_logits, st.draft_logits, row_index, parent, M,
                                                                 tokens, table, k, cfg.delta, un, threads=8)
        work = torch.ones(lantern_gpu.trees_sequential_workspace_bytes(B, M, V) // 4, dtype=torch.int32, device="cuda")
        n, path, nxt = lantern_gpu.verify_trees_sequential(
            st.target_logits.cuda(), st.draft_logits.cuda(), torch.from_numpy(np.ascontiguousarray(row_index)).cuda(),
            torch.from_numpy(parent).cuda().reshape(-1), M, torch.from_numpy(np.ascontiguousarray(tokens)).cuda(),
            torch.from_numpy(table).cuda(), cfg.delta, un.cuda(), workspace=work.view(torch.uint8))
        torch.cuda.synchronize()
        np.testing.assert_array_equal(n.cpu().numpy(), n_o)
        np.testing.assert_array_equal(path.cpu().numpy(), path_o)
        np.testing.assert_array_equal(nxt.cpu().numpy(), next_o)
        later += sum(int((parent[b, :path_o[b, j]] == parent[b, path_o[b, j]]).any())
                     for b in range(B) for j in range(n_o[b]))
    assert M < 100 or later > 0
