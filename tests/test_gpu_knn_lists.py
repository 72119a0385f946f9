"""Neighbour tables through candidate lists (Section 4.2; Algorithm 2, precompute part) where the lists are awkward: more
nearly equal keys than the selection holds at once, more hits in a tile than are staged at once, equal codes, codes
that are no numbers; and every form that the selection's exact keys take.  Whole tables, or a stretch of rows of the
larger ones, against the oracle's ranking."""
import numpy as np
import pytest
import torch

from parity_utils import replay_us

pytestmark = pytest.mark.gpu


def _table(lantern, cb, k, metric, max_exact_rows):
    got, exact = lantern.build_knn(cb.cuda(), k, metric=metric, return_stats=True)
    torch.cuda.synchronize()
    assert int(exact.item()) <= max_exact_rows
    return got.cpu().numpy()


def _clusters(V, d, size, spread, seed):
    """Clusters of `size` codes next to each other in the codebook."""
    rng = np.random.default_rng(seed)
    centre = rng.standard_normal((-(-V // size), d))
    return (np.repeat(centre, size, axis=0)[:V] + spread * rng.standard_normal((V, d))).astype(np.float32)


# most: rows that may be left to the all-pairs pass.  None where distances within a cluster are well above the error of the
# approximate keys, about 1e-6 of the codes' norms; any where they are not.
@pytest.mark.parametrize("V,d,k,size,spread,dtype,metric,most", [
    (8192, 8, 1000, 1400, 1e-3, torch.float32, "l2", 0),        # a cluster is one bucket of the list's range
    (8192, 8, 1000, 1150, 1e-3, torch.float32, "l2", 0),        # and holds more than the selection: it is divided again
    (8192, 8, 1000, 1150, 0.03, torch.bfloat16, "l2", 0),
    (8192, 8, 1000, 1400, 1e-3, torch.float32, "cosine", 8192),
    (9000, 16, 900, 1100, 0.02, torch.bfloat16, "l2", 0),
    (8192, 8, 100, 700, 1e-3, torch.float32, "l2", 8192),
    (8192, 8, 100, 700, 1e-2, torch.float32, "l2", 0),
    (12288, 16, 100, 300, 0.01, torch.float32, "l2", 0),        # codes of four vectors
    (6000, 24, 500, 800, 1e-3, torch.float32, "l2", 6000),      # lists with keys
    (6000, 24, 500, 800, 0.1, torch.float32, "l2", 0),
])
def test_clustered_codes(oracle_mod, lantern_gpu, V, d, k, size, spread, dtype, metric, most):
    cb = torch.from_numpy(_clusters(V, d, size, spread, V + d + k)).to(dtype)
    got = _table(lantern_gpu, cb, k, metric, most)
    want = oracle_mod.build_knn(cb.float().numpy(), k, metric=metric, threads=16)
    np.testing.assert_array_equal(got, want)


@pytest.mark.parametrize("V,d,k,dtype,scale", [(8192, 8, 1000, torch.float32, 2.0 ** -52), (8200, 8, 900, torch.bfloat16, 2.0 ** -54),
                                               (12288, 16, 600, torch.float32, 2.0 ** -54), (8192, 8, 1000, torch.float32, 2.0 ** 55)])
def test_small_and_large_codes(oracle_mod, lantern_gpu, V, d, k, dtype, scale):
    """Distances of 1e-30 and less, or 1e33, are as good as any other: no row is left to the all-pairs pass."""
    cb = (torch.randn(V, d, generator=torch.Generator().manual_seed(V + k)) * scale).to(dtype)
    got = _table(lantern_gpu, cb, k, "l2", 0)
    rows = (0, V) if V < 10000 else (V - 2500, V)
    want = oracle_mod.build_knn(cb.float().numpy(), k, rows=rows, threads=16)
    np.testing.assert_array_equal(got[rows[0]:rows[1]], want)


def _reach(cb, code, ranks):
    """Rows that have `code` within their first `ranks` tokens, themselves among them."""
    c = cb.double().cuda()
    closer = torch.cat([(((row[:, None, :] - c[None]) ** 2).sum(2) < ((row - c[code]) ** 2).sum(1)[:, None]).sum(1)
                        for row in c.split(256)])
    return int((closer < ranks).sum())


# A run of equal codes that does not fit leaves the rows whose table or list reaches it to the all-pairs pass: lists are about
# 300 tokens long for k = 70.
@pytest.mark.parametrize("k", [70, 1000])
def test_more_equal_codes_than_the_selection_holds(oracle_mod, lantern_gpu, k):
    rng = np.random.default_rng(k)
    cb = rng.standard_normal((8192, 8)).astype(np.float32)
    equal = rng.permutation(8192)[:1200]
    cb[equal] = cb[17]
    got = _table(lantern_gpu, torch.from_numpy(cb), k, "l2", _reach(torch.from_numpy(cb), equal[0], max(k, 512)))
    np.testing.assert_array_equal(got, oracle_mod.build_knn(cb, k, threads=16))


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_longer_lists_than_their_room(oracle_mod, lantern_gpu, dtype):
    """6000 equal codes in a row of the codebook: every pair of a tile is a hit, and lists end inside a run of them."""
    cb = torch.randn(8192, 8, generator=torch.Generator().manual_seed(9))
    cb[1000:7000] = cb[1000]
    cb = cb.to(dtype)
    got = _table(lantern_gpu, cb, 70, "l2", _reach(cb, 1000, 512))
    np.testing.assert_array_equal(got, oracle_mod.build_knn(cb.float().numpy(), 70, threads=16))


@pytest.mark.parametrize("V,d,size,k,dtype", [(8192, 8, 512, 100, torch.float32), (10304, 8, 400, 380, torch.bfloat16)])
def test_clusters_in_order_cost_no_more(lantern_gpu, V, d, size, k, dtype):
    """The same codes with those of a cluster next to each other, and in no order: 116 / 119 and 181 / 181 us (231 / 111
    and 276 / 175 where the tiles of a cluster were what the launch waited for)."""
    cb = torch.from_numpy(_clusters(V, d, size, 0.1, 3)).to(dtype).cuda()
    mixed = cb[torch.randperm(V, generator=torch.Generator().manual_seed(1)).cuda()].contiguous()
    work = torch.empty(lantern_gpu.binding.knn_workspace_bytes(1 if dtype == torch.bfloat16 else 0, V, d, k), dtype=torch.uint8, device="cuda")
    out = torch.empty((V, k), dtype=torch.int32, device="cuda")
    ordered_us, mixed_us = replay_us(*(lambda c=c: lantern_gpu.build_knn(c, k, workspace=work, out=out) for c in (cb, mixed)))
    assert ordered_us < 1.3 * mixed_us


@pytest.mark.parametrize("metric", ["l2", "cosine"])
@pytest.mark.parametrize("V,d,k", [(8192, 8, 300), (5000, 40, 120)])
def test_codes_that_are_no_numbers(oracle_mod, lantern_gpu, V, d, k, metric):
    rng = np.random.default_rng(V)
    cb = rng.standard_normal((V, d)).astype(np.float32)
    cb[5, 3], cb[700, 0], cb[V - 1, d - 1] = np.nan, np.inf, -np.inf
    cb[900] = 0.0
    got = _table(lantern_gpu, torch.from_numpy(cb), k, metric, 16)
    np.testing.assert_array_equal(got, oracle_mod.build_knn(cb, k, metric=metric, threads=16))


@pytest.mark.parametrize("metric", ["l2", "cosine"])
@pytest.mark.parametrize("V,d,k,dtype", [
    (8192, 4, 90, torch.float32), (8200, 8, 1000, torch.bfloat16), (4097, 8, 1000, torch.float32),   # one and two vectors
    (12300, 16, 300, torch.float32), (12288, 32, 200, torch.bfloat16),                               # four vectors
    (6001, 20, 150, torch.float32), (4500, 120, 700, torch.bfloat16), (8192, 16, 1000, torch.float32),   # lists with keys
    (2000, 12, 60, torch.float32), (1500, 88, 400, torch.bfloat16), (300, 1028, 50, torch.float32),      # whole rows
    (20000, 8, 100, torch.float32), (33000, 8, 230, torch.bfloat16),                                     # larger samples
    (1000, 9, 100, torch.float32), (4000, 8, 30, torch.float32), (4000, 16, 100, torch.bfloat16),        # whole rows by elements,
    (9000, 8, 30, torch.bfloat16), (20000, 8, 30, torch.float32), (34000, 8, 20, torch.bfloat16),        # of any length
    (2000, 16, 200, torch.float32), (2000, 24, 30, torch.bfloat16), (4000, 8, 300, torch.bfloat16),      # by vectors: 64 bytes and many cosine
    (4000, 16, 300, torch.float32), (9000, 32, 30, torch.bfloat16), (20000, 24, 40, torch.float32),      # keys, 48 bytes, more than 256 slots
])
def test_forms_of_the_exact_keys(oracle_mod, lantern_gpu, V, d, k, dtype, metric):
    g = torch.Generator().manual_seed(V + d)
    cb = torch.randn(V, d, generator=g)
    cb = (cb * (0.5 + torch.rand(V, 1, generator=g))).to(dtype)
    got = _table(lantern_gpu, cb, k, metric, 0)
    rows = (0, V) if V < 10000 else (V - 2500, V)
    want = oracle_mod.build_knn(cb.float().numpy(), k, metric=metric, rows=rows, threads=16)
    np.testing.assert_array_equal(got[rows[0]:rows[1]], want)
