"""Which steps a whole pass of an operator calls (CPU only: the library's functions are replaced by ones that note their name)."""
import pytest
import torch

from paper_2407_02327_amd import qsync as Q
from paper_2407_02327_amd.operator import QConv3x3, QLinear


@pytest.fixture
def called(monkeypatch):
    names = []
    for name in Q.SIGNATURES:
        if not (name.endswith("_bytes") or name.startswith("qsync_debug")) and hasattr(Q, name):
            monkeypatch.setattr(Q, name, lambda *a, _n=name, **k: names.append(_n))
    return names


def _linear(cls, tag):
    op = cls(tag, 64, 32, 48, device="cpu")
    return op, (torch.zeros(64, 48), torch.zeros(32, 48)), torch.zeros(64, 32)


def _conv(cls, tag):
    op = cls(tag, 2, 4, 4, 16, 32, device="cpu")
    return op, (torch.zeros(2, 4, 4, 16), torch.zeros(32, 9 * 16)), torch.zeros(32, 32)


OPERATORS = [(QLinear, _linear, t) for t in (Q.INT8, Q.FP16, Q.FP32)] + [(QConv3x3, _conv, t) for t in (Q.INT8, Q.FP16)]
STEPS = {QLinear: ("convert_x", "convert_w", "gemm_fwd", "convert_dy", "gemm_bwd"),
         QConv3x3: ("convert_x", "convert_w", "conv_fwd", "convert_dy", "conv_dgrad", "conv_wgrad")}
each_operator = pytest.mark.parametrize("cls, make, tag", OPERATORS, ids=lambda v: v.__name__ if isinstance(v, type) else str(v))


@each_operator
@pytest.mark.parametrize("place", ["subclass", "object", "class"])
def test_a_step_of_the_callers_own_is_called(cls, make, tag, place, called, monkeypatch):
    """A step replaced in a subclass, on the object or on the class -- weights that are kept, a wrapper that times -- runs once in
    every whole pass, and so do the other steps of that direction."""
    for step in STEPS[cls]:
        mine, own = [], getattr(cls, step)

        def replacement(self, *args, **kw):
            mine.append(step)
            return own(self, *args, **kw)

        with monkeypatch.context() as m:
            if place == "class":
                m.setattr(cls, step, replacement)
            op, inputs, dy = make(type("Mine", (cls,), {step: replacement}) if place == "subclass" else cls, tag)
            if place == "object":
                setattr(op, step, lambda *args, **kw: replacement(op, *args, **kw))
            for passes in (1, 2):
                del called[:]
                op.forward(*inputs)
                op.backward(dy)
                assert mine == [step] * passes
                assert ("qsync_convert_operands" in called) == (step not in ("convert_x", "convert_w"))


@each_operator
def test_the_operators_own_steps_go_together(cls, make, tag, called):
    op, inputs, dy = make(cls, tag)
    op.forward(*inputs)
    assert called[0] == "qsync_convert_operands" and len(called) == 2
    del called[:]
    op.backward(dy)
    if cls is QLinear and tag != Q.INT8:
        assert called == ["qsync_qlinear_backward"]


def test_weights_that_are_kept_stay(called):
    class Frozen(QLinear):
        def convert_w(self, w, stream=None):
            if not hasattr(self, "frozen"):
                self.frozen = True
                super().convert_w(w, stream)

    op, (x, w), _ = _linear(Frozen, Q.INT8)
    for _ in range(3):
        op.forward(x, w)
    assert called.count("qsync_prepare_weights") == 1 and called.count("qsync_absmax_quantize") == 3
