"""The binding's own state, without a device: the workspace sizes a handle keeps,
and the kinds of tensors it makes."""
from types import SimpleNamespace

import torch

from paper_2609_01864_amd import autograd as A
from paper_2609_01864_amd import credit as C


class Stub:
    """A handle whose library is a few Python functions."""

    def __init__(self, monkeypatch):
        self.option, self.during = 0, lambda: None
        lib = SimpleNamespace(credit_set_option=self.set_option)
        monkeypatch.setattr(C, "lib", lambda: lib)
        self.h = h = object.__new__(C.Handle)
        h.ptr, h._ws, h._sizes, h._generation = None, {}, {}, 0
        h.workspace_size = self.size
        h.workspace = lambda n, stream: n

    def set_option(self, ptr, opt, value):
        self.during()
        self.option = value
        return C.OK

    def size(self, *args):
        n = 100 + self.option
        self.during()
        return n


def test_sizes_follow_the_options(monkeypatch):
    s = Stub(monkeypatch)
    call = lambda: s.h._call_ws(C.SOFTMAX, C.FWD, C.F32, 4, 8, None, 0)
    assert call() == 100
    s.h.set_option(C.OPT_ROWS, 2)
    assert call() == 102


def test_size_kept_by_a_call_while_an_option_changes(monkeypatch):
    # another thread's call between the start of set_option and the change
    s = Stub(monkeypatch)
    call = lambda: s.h._call_ws(C.SOFTMAX, C.FWD, C.F32, 4, 8, None, 0)
    s.during = lambda: (setattr(s, "during", lambda: None), call())
    s.h.set_option(C.OPT_ROWS, 2)
    assert call() == 102


def test_size_worked_out_before_an_option_changed(monkeypatch):
    # a call that sized its workspace before another thread's set_option and
    # keeps the size after it
    s = Stub(monkeypatch)
    call = lambda: s.h._call_ws(C.SOFTMAX, C.FWD, C.F32, 4, 8, None, 0)
    s.during = lambda: (setattr(s, "during", lambda: None), s.h.set_option(C.OPT_ROWS, 2))
    call()
    assert call() == 102


class Kind(torch.Tensor):
    pass


def test_results_of_tensor_subclasses():
    # the operators make plain tensors; the autograd functions return the kind
    # of their input, as they do for one of more than two dimensions
    C.io_dtype(torch.empty(0))  # (the binding's torch)
    for x in (torch.ones(2, 3), torch.nn.Parameter(torch.ones(2, 3)), torch.ones(2, 3).as_subclass(Kind)):
        y = C._empty_like_out(x)
        assert type(y) is torch.Tensor and y.shape == (2, 3) and y.dtype == x.dtype and y.is_contiguous()
        want = Kind if type(x) is Kind else torch.Tensor
        assert type(A._out(y, x)) is want and type(A._out(y, x.view(1, 2, 3))) is want
    t = torch.ones(3, 2).t()
    assert C._empty_like_out(t).is_contiguous()
