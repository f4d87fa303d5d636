"""VerifyLayer.step makes its library calls itself: weights that do not fit the
layer are refused before the first of them, with the errors route() and
moe_forward() raise.  No GPU: the library is a recorder and the tensors are host
tensors that say they are on the device."""
import numpy as np
import pytest
import torch

from paper_2608_02989_amd import _lib as L
from paper_2608_02989_amd import ops

E, H, I, K, T = 6, 32, 64, 2, 5


class Recorder:
    def __init__(self):
        self.calls = []

    def __getattr__(self, name):
        def call(*args):
            self.calls.append(name)
            return L.OK
        return call


class Dev(torch.Tensor):
    """A host tensor that the binding takes for a device tensor."""
    is_cuda = property(lambda self: True)


def zeros(*shape, dtype=torch.float32):
    return torch.zeros(*shape, dtype=dtype).as_subclass(Dev)


@pytest.fixture
def recorder(monkeypatch):
    rec = Recorder()
    monkeypatch.setattr(ops, "lib", lambda: rec)
    monkeypatch.setattr(ops, "_stream_ptr", lambda stream=None: None)
    return rec


def layer(dtype=torch.float32):
    ly = ops.VerifyLayer.__new__(ops.VerifyLayer)
    ly.router = ops.PackedRouter(zeros(1, dtype=torch.int16), E, H)
    ly.E, ly.I, ly.H, ly.k, ly.dtype = E, I, H, K, dtype
    ly.beta, ly.mode, ly.budget, ly.removal_cap = 0.5, L.MODE_SELF_SIZING, 0, -1
    ly.wgu = ops.PackedGateUp(zeros(E * 2 * I * H, dtype=dtype), E, I, H)
    ly.wd = zeros(E, H, I, dtype=dtype)
    ly.max_tokens, ly.max_trees = T, 1
    ly.logits, ly.out = zeros(T, E), zeros(T, H)
    ly.sel_ws = ly.fwd_ws = zeros(256, dtype=torch.uint8)
    ly.sel_out = {"eligible": zeros(1, E, dtype=torch.uint8), "idx": zeros(T, K, dtype=torch.int32),
                  "gate": zeros(T, K), "stats": zeros(1, L.NUM_STATS, dtype=torch.int32)}
    return ly


def block(dtype=torch.float32):
    return zeros(T, H, dtype=dtype), None, zeros(T, dtype=torch.int32), zeros(T)


def test_step_calls_the_three_steps(recorder):
    logits, outs, out = layer().step(*block())
    assert recorder.calls == ["acceptmoe_route", "acceptmoe_select", "acceptmoe_moe_forward"]
    assert logits.shape == (T, E) and out.shape == (T, H) and outs["idx"].shape == (T, K)


def set_router(e, h):
    return lambda ly: setattr(ly, "router", ops.PackedRouter(ly.router.data, e, h))


def set_gate_up(e, i, h, dtype=torch.float32):
    return lambda ly: setattr(ly, "wgu", ops.PackedGateUp(zeros(e * 2 * i * h, dtype=dtype), e, i, h))


def set_down(t):
    return lambda ly: setattr(ly, "wd", t)


@pytest.mark.parametrize("change,error", [
    (set_router(E, 2 * H), ValueError),                    # the planes of another hidden size
    (set_router(E - 1, H), ValueError),                    # of fewer experts than the layer routes to
    (set_router(E + 1, H), ValueError),                    # of more experts than the logits hold
    (lambda ly: setattr(ly, "router", ly.router.data), TypeError),
    (set_gate_up(E, I, 2 * H), ValueError),
    (set_gate_up(E, 2 * I, H), ValueError),                # another I than the down stack's
    (set_gate_up(E, I, H, torch.bfloat16), TypeError),
    (lambda ly: setattr(ly, "wgu", ly.wgu.data), TypeError),
    (set_down(zeros(E, I, H)), ValueError),          # the stack of w_down not transposed
    (set_down(zeros(E - 1, H, I)), ValueError),
    (set_down(zeros(E, H, I // 2)), ValueError),
    (set_down(zeros(E, H, I, dtype=torch.bfloat16)), TypeError),
    (set_down(zeros(E, I, H).transpose(1, 2)), ValueError),  # not contiguous
    (set_down(zeros(E * H, I)), ValueError)])
def test_step_refuses_weights_that_do_not_fit(recorder, change, error):
    ly = layer()
    change(ly)
    with pytest.raises(error):
        ly.step(*block())
    assert recorder.calls == []


# the returned tensors are views: what a caller does to their shape or their
# autograd state stays with the caller, at the layer's full size too
def test_step_returns_views_of_the_buffers(recorder):
    ly = layer()
    logits, outs, out = ly.step(*block())
    out.unsqueeze_(0)
    out.requires_grad_()
    logits.t_()
    outs["idx"].squeeze_().unsqueeze_(2)
    del outs["gate"]
    logits2, outs2, out2 = ly.step(*block())
    assert out2.shape == (T, H) and not out2.requires_grad and logits2.shape == (T, E)
    assert outs2["idx"].shape == (T, K) and set(outs2) == {"eligible", "idx", "gate", "stats"}
    assert out2.data_ptr() == out.data_ptr() == ly.out.data_ptr()


@pytest.mark.parametrize("offsets", [[[0], [T]], [[0, T]], np.zeros((2, 2), np.int64), [[]]])
def test_two_dimensional_tree_offsets_are_refused(recorder, offsets):
    hidden, parent, depth, prob = block()
    with pytest.raises(TypeError):
        layer().step(hidden, parent, depth, prob, offsets)
    for fn in (ops.select, ops.select_noalloc):
        with pytest.raises(TypeError):
            fn(zeros(T, E), parent, depth, prob, offsets, K)
    assert recorder.calls == []
