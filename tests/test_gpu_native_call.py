"""The two ways a linear call reaches the library: native marshalling for plain arguments and the
Python checks for everything else, compared on the forms that decide between them."""
import os

import pytest
import torch

import paper_2105_14500_amd as tess
from paper_2105_14500_amd import binding as B
from gpu_util import share_desc, workspace

pytestmark = pytest.mark.gpu


class _Subclass(torch.Tensor):
    pass


class _Native:
    """Counts what the native code took."""

    def __init__(self):
        self.real, self.status = B._native(), []

    def __getattr__(self, name):
        def call(*args):
            self.status.append(getattr(self.real, name)(*args))
            return self.status[-1]
        return call


@pytest.mark.parametrize("form,native", [("list", True), ("tuple", True), ("view", True), ("parameter", True), ("subclass", False), ("stream", False)])
@pytest.mark.parametrize("m,kb,n", [(1, 8, 16), (64, 1, 3), (72, 40, 56)])
def test_every_form_gives_the_same_result(monkeypatch, form, native, m, kb, n):
    q = 2
    gen = torch.Generator().manual_seed(m + kb + n)
    new = lambda *s: torch.randint(-2, 3, s, generator=gen).float().cuda()  # noqa: E731
    x, w, dy, bias = new(q, m, kb), new(q, kb, n), new(q, m, n), new(n)
    desc = share_desc(q, 1, m, kb, n, "f32", "f32")
    if form == "view":
        wide = torch.zeros((q, m, kb + 5), device="cuda:0")
        wide[:, :, :kb] = x
        x_in = [t[:, :kb] for t in wide]
    elif form == "subclass":
        x_in = [t.as_subclass(_Subclass) for t in x]
    elif form == "parameter":
        x_in = [torch.nn.Parameter(t, requires_grad=False) for t in x]
    else:
        x_in = tuple(x) if form == "tuple" else list(x)
    stream = torch.cuda.current_stream() if form == "stream" else None
    y, z, dw, db = torch.empty((m, n), device="cuda:0"), torch.empty((m, n), device="cuda:0"), \
        torch.empty((kb, n), device="cuda:0"), torch.empty((n,), device="cuda:0")
    spy = _Native()
    monkeypatch.setattr(B, "_native", lambda: spy)
    tess.linear_fwd(desc, x_in, list(w), bias, B.ACT_GELU_ERF, y, preact_out=z, workspace=workspace(desc, B.OP_FWD), stream=stream)
    tess.linear_bwd_dw_bias(desc, x_in, list(dy), dw, db, stream=stream)
    assert spy.status == ([0, 0] if native else [-1, -1])
    want = sum(x[t].double() @ w[t].double() for t in range(q)) + bias
    assert torch.equal(z.double(), want)
    assert torch.allclose(y.double(), torch.nn.functional.gelu(want), rtol=1e-6, atol=1e-6)
    assert torch.equal(dw.double(), sum(x[t].double().t() @ dy[t].double() for t in range(q)))
    assert torch.equal(db.double(), dy.double().sum((0, 1)))


def test_what_is_refused_stays_refused():
    desc = share_desc(2, 1, 16, 8, 8, "f32", "f32")
    t = lambda *s, **k: torch.zeros(s, device="cuda:0", **k)  # noqa: E731
    x, w, y = list(t(2, 16, 8)), list(t(2, 8, 8)), t(16, 8)
    for bad in (dict(x=x[:1] + [t(16, 9)]), dict(x=x[:1] + [t(8, 16).t()]), dict(x=x[:1] + [t(16, 8, dtype=torch.bfloat16)]),
                dict(x=x[:1] + [t(16, 10)[:, :8]]), dict(x=x[:1] + [torch.zeros(16, 8)]), dict(y=t(16, 16)[:, ::2]),
                dict(bias=t(9)), dict(z=t(16, 9)[:, :8])):
        with pytest.raises(ValueError):
            tess.linear_fwd(desc, bad.get("x", x), w, bad.get("bias"), B.ACT_NONE, bad.get("y", y), preact_out=bad.get("z"))
    with pytest.raises(tess.TessError):
        tess.linear_fwd(desc, x, w, None, 7, y)


def test_a_call_with_a_stream_is_turned_down_at_once():
    """What the Python code will serve is not looked over twice: the activation code is asked for its value
    once, by the Python call."""

    class Act:
        asked = 0

        def __index__(self):
            self.asked += 1
            return B.ACT_NONE

    desc = share_desc(1, 1, 16, 8, 8, "f32", "f32")
    x, w, y = torch.ones((16, 8), device="cuda:0"), torch.ones((8, 8), device="cuda:0"), torch.zeros((16, 8), device="cuda:0")
    act = Act()
    tess.linear_fwd(desc, [x], [w], None, act, y, stream=torch.cuda.current_stream())
    assert act.asked == 1 and torch.equal(y, torch.full_like(y, 8.0))


def test_a_forked_child_is_refused():
    """The runtime does not survive a fork: PyTorch refuses to name a stream in the child, and with the
    stream left to the call so does every linear call, before any device call is made."""
    desc = share_desc(1, 1, 16, 8, 8, "f32", "f32")
    x, w, y = (torch.zeros(s, device="cuda:0") for s in ((16, 8), (8, 8), (16, 8)))
    torch.cuda.synchronize()
    child = os.fork()
    if child == 0:
        code = 1
        try:
            tess.linear_fwd(desc, [x], [w], None, B.ACT_NONE, y)
        except RuntimeError as e:
            code = 0 if "fork" in str(e) else 2
        finally:
            os._exit(code)
    assert os.waitstatus_to_exitcode(os.waitpid(child, 0)[1]) == 0
