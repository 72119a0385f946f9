"""The step calls' host half in native code against the same functions through ctypes: the same results for ordinary
calls, and nothing taken that the Python checks would treat otherwise (they then raise what they raise)."""
import numpy as np
import pytest
import torch

from paper_2410_03355_amd import binding
from synth import workloads
from parity_utils import random_table, random_trees, tree_step

pytestmark = pytest.mark.gpu


class _Tensor(torch.Tensor):
    pass


class _Declines:
    def __getattr__(self, name):
        return lambda *args: None


def _inputs(dtype, V=1000, k=20, B=3, M=7):
    cfg = workloads.Config("marshal", V, 8, "f32", True, k, 0.3, 64, 1, dtype, 1.5, 0.5, index=70)
    parent = random_trees(np.random.default_rng(5), B, M, max_children=3)
    st, row_index, tokens, un = tree_step(cfg, parent, step=0, variant="peaked")
    own = workloads.make_step(cfg, step=1, rows=B * M, variant="peaked", device="cuda")
    return {"t": st.target_logits.cuda(), "g": st.draft_logits.cuda(), "ri": torch.from_numpy(row_index).cuda(),
            "par": torch.from_numpy(parent.reshape(-1).copy()).cuda(), "M": M, "tok": torch.from_numpy(tokens).cuda(),
            "un": un.cuda(), "knn": torch.from_numpy(random_table(V, k, seed=3)).cuda(), "own": own}


def _calls(x):
    o, knn = x["own"], x["knn"]
    tree = (x["ri"], x["par"], x["M"], x["tok"], knn, 0.3)
    acc, res = binding.verify(o.target_logits, o.draft_logits, o.draft_tokens, knn, 0.3, o.uniforms)
    return {
        "verify": (o.target_logits, o.draft_logits, o.draft_tokens, knn, 0.3, o.uniforms),
        "verify_rows": (x["t"], x["g"], x["ri"], x["tok"], knn, 0.3, x["un"], "jsd"),
        "decide_rows": (x["t"], x["g"], x["ri"], x["tok"], knn, 0, x["un"], "tvd"),
        "verify_greedy": (o.target_logits, o.draft_tokens, knn, 0.3),
        "verify_greedy_rows": (x["t"], x["ri"], x["tok"], knn, 0.3),
        "verify_trees": (x["t"], x["g"], *tree, x["un"], "tvd"),
        "verify_trees_sequential": (x["t"], x["g"], *tree, x["un"], "jsd", None),
        "verify_trees_greedy": (x["t"], *tree),
        "accept_chains": (acc, res, x["M"]),
        "accept_trees": (acc, res, x["par"], x["M"]),
    }


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_same_results(lantern_gpu, monkeypatch, dtype):
    calls = _calls(_inputs(dtype))
    for name, args in calls.items():
        native = getattr(binding._marshal, name)(*args)
        assert native is not None and native.__class__ is not int, name
        public = getattr(binding, name)(*args)
        with monkeypatch.context() as m:
            m.setattr(binding, "_marshal", _Declines())
            general = getattr(binding, name)(*args)
        for got in (native, public):
            got, want = (v if isinstance(v, tuple) else (v,) for v in (got, general))
            assert len(got) == len(want), name
            for a, b in zip(got, want):
                assert a.dtype == b.dtype and a.shape == b.shape and a.device == b.device and torch.equal(a, b), name


def test_declined(lantern_gpu):
    calls = _calls(_inputs("bf16"))
    for name, args in calls.items():
        fast = getattr(binding._marshal, name)
        for i, arg in enumerate(args):
            if isinstance(arg, torch.Tensor):
                wrong = [arg.cpu(), arg.double(), arg.as_subclass(_Tensor), arg[:0],
                         arg.repeat_interleave(2, -1)[..., ::2]]            # the last one strided
            elif isinstance(arg, str):
                wrong = ["other", None]
            elif isinstance(arg, int) and arg == 7:                         # nodes of a tree or chain; 21 in all
                wrong = [0, -1, 4, 2 ** 40, 7.0]
            elif arg is None:
                wrong = [torch.empty(1 << 20, dtype=torch.uint8)]           # a workspace in host memory
            else:
                wrong = [np.float64(0.3), "0.3", None]
            for w in wrong:
                assert fast(*args[:i], w, *args[i + 1:]) is None, (name, i, type(w))
        assert fast(*args[:-1]) is None and fast(*args, None) is None
        with torch.device("cpu"):                                           # a mode of the interpreter
            assert fast(*args) is None
    o = calls["verify"]
    for bad in ((o[0].float(), *o[1:]), (*o[:2], o[2].long(), *o[3:]), (*o[:5], o[5][:4])):
        with pytest.raises((TypeError, ValueError)):
            binding.verify(*bad)
    with pytest.raises(binding.LanternError) as e:
        binding.verify(*o[:4], -1.0, o[5])
    assert e.value.status == binding.E_DELTA


def test_other_stream_and_outputs(lantern_gpu):
    """A stream or outputs of the caller's: the general way, on the stream that is named or current."""
    args = _calls(_inputs("f32"))["verify"]
    want = binding.verify(*args)
    out = torch.empty_like(want[0]), torch.empty_like(want[1])
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    named = binding.verify(*args, out_accept=out[0], out_resample=out[1], stream=side)
    assert named[0] is out[0] and named[1] is out[1]
    with torch.cuda.stream(side):
        current = binding.verify(*args)
    side.synchronize()
    for got in (named, current):
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
