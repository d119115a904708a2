"""The call sequence of a layer on the CPU, with stand-ins for the library's calls: what is passed on, and what a call that fails leaves."""
import pytest
import torch

from paper_2404_01847_amd import ffn as layer

CALLS = [n for n in dir(layer.s24) if n.startswith(("spmm_", "dense_", "act_", "glu_", "swiglu_", "bias_grad", "compress_batch"))]


@pytest.fixture
def calls(monkeypatch):
    """(name, arguments) of each call; those in `calls.fail` raise instead."""
    class Calls(list):
        fail = ()
    seen = Calls()
    def stand_in(name):
        def call(*args, **kw):
            if name in seen.fail:
                raise layer.s24.S24Error(-1, name)
            seen.append((name, [list(a) if isinstance(a, list) else a for a in args]))
        return call
    for name in CALLS:
        monkeypatch.setattr(layer.s24, name, stand_in(name))
    monkeypatch.setattr(layer.s24, "strerror", lambda status: "refused")
    return seen


def make(act, biases=(), **kw):
    p, d, f = 8, 64, 128
    new = lambda *shape: torch.zeros(shape, dtype=torch.bfloat16)
    gated = act in ("swiglu", "geglu")
    weights = {"Wg": new(f, d), "Wu": new(f, d), "Wd": new(d, f)} if gated else {"W1": new(f, d), "W2": new(d, f)}
    rows = {"Wgu": 2 * f, "W1": f, "Wd": d, "W2": d}
    return layer.SparseFFN(weights, p, act, 1e-3, biases={n: new(rows[n]) for n in biases}, **kw), new(p, d), new(p, d)


def submitted(calls):
    """The gradients that the calls since the last look were to compute."""
    got = [pr[2] for name, args in calls for pr in (args[-1] if name in ("spmm_bwd_dx_dw", "dense_dw_batch") else ())]
    calls.clear()
    return got


@pytest.mark.parametrize("act, kw, failing", [
    ("gelu", {}, "spmm_bwd_dx_dw"), ("swiglu", dict(concat_gate_up=True), "spmm_bwd_dx_dw"),
    ("gelu", dict(biases=("W1",)), "bias_grad"),          # between the two gradients
    ("swiglu", {}, "dense_dw_batch"), ("swiglu", {}, "swiglu_bwd")])
def test_a_backward_pass_that_fails_leaves_nothing_to_the_next(calls, act, kw, failing):
    ffn, X, dY = make(act, **kw)
    calls.fail = (failing,)
    with pytest.raises(layer.s24.S24Error):
        ffn.backward(X, dY)
    calls.fail = ()
    calls.clear()
    ffn.backward(X, dY)
    got = submitted(calls)
    assert len(got) == len(ffn.w) and {id(g) for g in got} == {id(w.grad) for w in ffn.w.values()}


def test_a_bias_taken_away_has_no_gradient(calls):
    ffn, X, dY = make("gelu", biases=("W1", "W2"))
    ffn.bias["W1"] = None
    ffn.backward(X, dY)
    assert [args[1] is ffn.bias_grad["W2"] for name, args in calls if name == "bias_grad"] == [True]
