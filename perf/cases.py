"""The work by which this library's speed is measured.

A serving loop calls the library once per step of the target model: it has the logits of the drafted
positions, the drafted tokens, two uniforms per candidate and the neighbour table of its codebook, and
wants the decisions, the walk and the resampled tokens.  The table itself is built once per codebook.
The cases below are those calls: single steps where latency counts, batches that fill the device, both
logit types, the three sibling rules of a draft tree, rows that are not aligned, vocabularies from a
thousand tokens to the whole text-and-image vocabulary of a unified model, and table builds.

Fields of a case
  op       rows: lantern.verify, one verification per row, then the walk of the drafted chains if `chain` > 0
           decide: lantern.decide_rows, the decisions of such rows without the resampled tokens
           trees / sequential / greedy: a step over draft trees under one of the three sibling rules
           table: lantern.build_knn
  dtype    of the logits (of the codebook for a table)
  N        verifications of a `rows` case;  B, M  trees and candidates per tree
  V, k     tokens and table width;  d  latent width of the codebook
  start    first column of the logits inside wider rows of `stride` elements (0 and V: the rows are V wide)
  mix      plain: nearly every candidate is accepted.  peaked: logits five times as wide, the bound cuts the
           neighbourhoods and about 45 % are rejected.  reject: acceptance draws just below one
  bound    of the neighbourhood: tvd or jsd, below `delta`
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2410_03355_amd as lantern
from synth import trees, workloads

DEVICE = "cuda"


def _rows(name, N, V, k, delta, dtype, mix, scale, noise, start=0, stride=0, chain=0, op="rows"):
    return {"name": name, "op": op, "N": N, "V": V, "k": k, "delta": delta, "dtype": dtype, "mix": mix,
            "scale": scale, "noise": noise, "start": start, "stride": stride or V, "chain": chain}


def _trees(name, op, B, M, V, k, delta, dtype, mix, scale, noise, bound="tvd"):
    return {"name": name, "op": op, "B": B, "M": M, "V": V, "k": k, "delta": delta, "dtype": dtype, "mix": mix,
            "scale": scale, "noise": noise, "bound": bound}


def _table(name, V, d, k, dtype, metric="l2", normalise=True):
    return {"name": name, "op": "table", "V": V, "d": d, "k": k, "dtype": dtype, "metric": metric,
            "normalise": normalise}


def listed():
    return [
        # the smallest call: 64 drafted positions over a small codebook, bound by launches and the host
        _rows("rows_tiny", 64, 1024, 16, 0.1, "f32", "plain", 3.0, 1.0),
        # one image being decoded: a single tree of 60 candidates per step, bound by latency
        _trees("step_one_image", "trees", 1, 60, 16384, 1000, 0.4, "bf16", "peaked", 1.2, 0.5),
        # 64 images decoded together
        _trees("step_batch", "trees", 64, 60, 16384, 1000, 0.4, "bf16", "peaked", 1.2, 0.5),
        # the same batch under the sibling rule that keeps the target's law
        _trees("step_sequential", "sequential", 64, 60, 16384, 1000, 0.4, "bf16", "peaked", 1.2, 0.5),
        # 16 images under greedy decoding, narrower table
        _trees("step_greedy", "greedy", 16, 60, 16384, 300, 0.2, "bf16", "plain", 1.2, 0.5),
        # the decisions of a full batch of rows of their own: bound by reading the logits
        _rows("rows_decided", 3840, 16384, 1000, 0.4, "bf16", "peaked", 1.2, 0.5, op="decide"),
        # the same with a resampled token for every second row
        _rows("rows_rejected", 3840, 16384, 1000, 0.4, "bf16", "peaked", 1.2, 0.5),
        # fp32 logits of a codebook with wide latents
        _rows("rows_f32", 3840, 8192, 100, 0.3, "f32", "peaked", 1.5, 0.5),
        # chains of 60; the image tokens are columns 4 .. 8195 of a unified vocabulary's logits, so no row is
        # 16-byte aligned
        _rows("chains_slice", 960, 8192, 300, 0.2, "bf16", "peaked", 1.2, 0.5, start=4, stride=65536, chain=60),
        # the unified vocabulary as a whole
        _rows("rows_large_vocab", 960, 65536, 1000, 0.4, "bf16", "peaked", 1.2, 0.5),
        # neighbour tables of the two codebook shapes
        _table("table_narrow", 16384, 8, 1000, "f32"),
        _table("table_wide", 8192, 256, 100, "bf16", normalise=False),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _vocab(rng, lo, hi):
    """Half of them whole multiples of 64 as codebooks mostly are, half of any size."""
    V = _log_int(rng, lo, hi)
    return max(lo, V // 64 * 64) if rng.random() < 0.5 else V


ROW_BYTES = 224 << 20     # most bytes of logits of a drawn case (the listed ones: up to 252e6)


def draw(rng):
    op = rng.choice(["rows", "rows", "rows", "decide", "trees", "trees", "sequential", "greedy", "table"])
    if op == "table":
        dtype = rng.choice(["f32", "bf16"])
        V = _vocab(rng, 1024, 12288)
        # latent widths are mostly whole vectors of the codebook's type; some are not
        d = _log_int(rng, 4, 160)
        d = max(8, d // 8 * 8) if rng.random() < 0.75 else d
        return {"op": op, "V": V, "d": d, "k": _log_int(rng, 16, 1000), "dtype": dtype,
                "metric": rng.choice(["l2", "l2", "cosine"]), "normalise": rng.random() < 0.5}
    dtype = rng.choice(["bf16", "bf16", "f32"])
    size = 2 if dtype == "bf16" else 4
    V = _vocab(rng, 1024, 65536)
    k = _log_int(rng, 16, min(1000, V))
    mix = rng.choice(["plain", "peaked", "peaked", "reject"])
    delta = 0.0 if rng.random() < 0.15 else round(rng.uniform(0.05, 0.5), 3)
    common = {"op": op, "V": V, "k": k, "delta": delta, "dtype": dtype, "mix": mix,
              "scale": round(rng.uniform(1.0, 3.0), 2), "noise": round(rng.uniform(0.3, 1.0), 2)}
    if op in ("rows", "decide"):
        start, stride = (0, V)
        if rng.random() < 0.25:
            start = rng.randrange(0, 9)
            stride = V + start + rng.randrange(0, 4096)
        N = min(_log_int(rng, 1, 3840), max(1, ROW_BYTES // (2 * stride * size)))
        if mix != "plain" or V % 8:      # rows that may be evaluated in fp64 throughout
            N = max(1, min(N, (3840 * 8192) // V))
        chain = rng.choice([0, 0, 1, 5, 60]) if op == "rows" else 0
        if chain:
            N = max(1, N // chain) * chain
            if 2 * N * stride * size > ROW_BYTES:
                chain = 0
                N = max(1, ROW_BYTES // (2 * stride * size))
        return {**common, "N": N, "start": start, "stride": stride, "chain": chain}
    M = _log_int(rng, 4, 64)
    sides = 1 if op == "greedy" else 2
    B = min(_log_int(rng, 1, 64), max(1, ROW_BYTES // (sides * (M + 1) * V * size)))
    if V % 8 or V > 16384:
        B = max(1, min(B, (960 * 16384) // (M * V)))
    return {**common, "B": B, "M": M, "bound": "jsd" if op != "greedy" and rng.random() < 0.2 else "tvd"}


def _config(case, seed, rows):
    """The input recipe's configuration for the case; the seed goes in through its index."""
    return workloads.Config("case", case["V"], case.get("d", 8), "f32", True, case["k"], case.get("delta", 0.0), rows, 1,
                            case["dtype"], case.get("scale", 1.0), case.get("noise", 1.0), index=100 + seed % 100000)


def _wide_rows(x, start, stride):
    """The same logits as columns start .. start + V - 1 of rows of `stride` elements."""
    N, V = x.shape
    if stride == V and start == 0:
        return x
    room = torch.zeros((N, stride), dtype=x.dtype, device=x.device)
    view = room[:, start:start + V]
    view.copy_(x)
    return view


def prepare(case, seed):
    V, k = case["V"], case["k"]
    if case["op"] == "table":
        g = torch.Generator(device=DEVICE).manual_seed(seed)
        cb = torch.randn(V, case["d"], generator=g, device=DEVICE)
        if case["normalise"]:
            cb = cb / cb.norm(dim=1, keepdim=True)
        cb = cb.to(workloads.torch_dtype(case["dtype"])).contiguous()
        return {"case": case, "codebook": cb}
    by_row = case["op"] in ("rows", "decide")
    rows = case["N"] if by_row else case["B"] * (case["M"] + 1)
    cfg = _config(case, seed, rows)
    knn = lantern.build_knn(workloads.make_codebook(cfg, device=DEVICE), k)
    lantern.prepare(workloads.torch_dtype(case["dtype"]), V, k)
    state = {"case": case, "knn": knn}
    if by_row:
        st = workloads.make_step(cfg, step=0, variant=case["mix"], device=DEVICE)
        state["target"] = _wide_rows(st.target_logits, case["start"], case["stride"])
        state["draft"] = _wide_rows(st.draft_logits, case["start"], case["stride"])
        state["tokens"], state["uniforms"] = st.draft_tokens, st.uniforms
        return state
    B, M = case["B"], case["M"]
    parent = trees.level_order(trees.random_trees(np.random.default_rng(seed), B, M))
    st, row_index, tokens, uniforms = trees.tree_step(cfg, parent, step=0, variant=case["mix"], device=DEVICE)
    state["target"], state["draft"], state["uniforms"] = st.target_logits, st.draft_logits, uniforms
    state["parent"] = torch.from_numpy(parent.reshape(-1)).to(DEVICE)
    state["row_index"] = torch.from_numpy(row_index).to(DEVICE)
    state["tokens"] = torch.from_numpy(tokens).to(DEVICE)
    if case["op"] == "sequential":
        need = lantern.trees_sequential_workspace_bytes(B, M, V)
        state["workspace"] = torch.empty(need, dtype=torch.uint8, device=DEVICE)
    return state


def run(state):
    case = state["case"]
    op = case["op"]
    if op == "table":
        return lantern.build_knn(state["codebook"], case["k"], metric=case["metric"])
    delta, knn, tokens = case["delta"], state["knn"], state["tokens"]
    if op == "rows":
        accept, resample = lantern.verify(state["target"], state["draft"], tokens, knn, delta, state["uniforms"])
        if not case["chain"]:
            return accept, resample
        kept, following = lantern.accept_chains(accept, resample, case["chain"])
        return accept, resample, kept, following
    if op == "decide":
        return lantern.decide_rows(state["target"], state["draft"], None, tokens, knn, delta, state["uniforms"])
    if op == "greedy":
        return lantern.verify_trees_greedy(state["target"], state["row_index"], state["parent"], case["M"], tokens, knn,
                                           delta)
    if op == "sequential":
        return lantern.verify_trees_sequential(state["target"], state["draft"], state["row_index"], state["parent"],
                                               case["M"], tokens, knn, delta, state["uniforms"],
                                               divergence=case["bound"], workspace=state["workspace"])
    return lantern.verify_trees(state["target"], state["draft"], state["row_index"], state["parent"], case["M"], tokens,
                                knn, delta, state["uniforms"], divergence=case["bound"])


def work(case):
    V, k = case["V"], case["k"]
    if case["op"] == "table":
        size = 4 if case["dtype"] == "f32" else 2
        return {"bytes": V * case["d"] * size + 4 * V * k, "flops": 2.0 * V * V * case["d"]}
    row = V * (2 if case["dtype"] == "bf16" else 4)
    sides = 1 if case["op"] == "greedy" else 2
    # a softmax takes a subtraction, an exponential and an addition per logit
    if case["op"] in ("rows", "decide"):
        N = case["N"]
        return {"bytes": N * (2 * row + 4 * k + 20), "flops": 6.0 * N * V}
    N = case["B"] * case["M"]
    if case["op"] == "sequential":
        # decisions along the walk only: at least the rows of the prefix, and the children tried there
        contexts, tried = case["B"], case["B"]
    else:
        # every candidate is decided; about half the nodes of such a tree have children, and a pair of
        # rows per node with children and one for the prefix are read
        contexts, tried = case["B"] + N // 2, N
    return {"bytes": contexts * sides * row + tried * (4 * k + 24), "flops": 3.0 * sides * contexts * V}


def tolerance(case):
    # tokens, decisions and table entries are whole numbers, defined by fp64 evaluation of the rule
    return "exact"
