"""The natively marshalled fused calls take exactly the plain valid case: the
same results as the binding's own path, the caller's outputs handed back, and
everything else (errors, other argument types, a stream, validation) left to
that path, with its exceptions."""
import numpy as np
import pytest
import torch

import paper_2207_05808_amd as mdn
from paper_2207_05808_amd import binding
from paper_2207_05808_amd import workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture
def call():
    p = W.make("classifier_tiny", N=77)
    dev = lambda x: torch.from_numpy(np.ascontiguousarray(x)).to(DEV)
    lut, scale, offset = mdn.build_lut(dev(p.P), dev(p.B))
    tab = mdn.build_lut_f32(dev(p.P), dev(p.B))
    return dict(A=dev(p.A), split=dev(p.split), thr=dev(p.thr), lut=lut, scale=scale, offset=offset, tab=tab,
                bias=torch.randn(10, device=DEV))


def both(monkeypatch, f):
    """f() through the native path (which must take it) and through the binding's own."""
    seen = []
    native = binding._native
    monkeypatch.setattr(binding, "_native", lambda *a: seen.append(native(*a)) or seen[-1])
    fast = f()
    assert seen and seen[-1] is not None
    monkeypatch.setattr(binding, "_native", lambda *a: None)
    slow = f()
    monkeypatch.setattr(binding, "_native", native)
    return fast, slow


def same(a, b):
    if isinstance(a, tuple):
        return len(a) == len(b) and all(same(x, y) for x, y in zip(a, b))
    return a is None and b is None or (a.dtype == b.dtype and a.shape == b.shape and bool((a == b).all()))


@pytest.mark.parametrize("act", ["none", "bias", "relu", "softmax", 2])
def test_same_results(call, monkeypatch, act):
    k = call
    t = (k["A"], k["split"], k["thr"])
    q = (k["lut"], k["scale"], k["offset"])
    for f in (lambda: mdn.matmul(*t, *q), lambda: mdn.matmul(*t, *q, want_acc=True, want_idx=True),
              lambda: mdn.matmul(t[0][:1], *t[1:], *q), lambda: mdn.matmul(t[0][::2], *t[1:], *q),
              lambda: mdn.matmul_f32(*t, k["tab"], want_idx=True),
              lambda: mdn.matmul_act(*t, *q, col_bias=k["bias"], act=act), lambda: mdn.matmul_act(*t, *q, act=act),
              lambda: mdn.matmul_act_f32(*t, k["tab"], col_bias=k["bias"], act=act)):
        fast, slow = both(monkeypatch, f)
        assert same(fast, slow)


def test_callers_outputs(call):
    k = call
    y = torch.empty(77, 10, device=DEV)
    acc = torch.empty(77, 10, dtype=torch.int32, device=DEV)
    idx = torch.empty(77, 4, dtype=torch.uint8, device=DEV)
    r = mdn.matmul(k["A"], k["split"], k["thr"], k["lut"], k["scale"], k["offset"], y_out=y, acc_out=acc, idx_out=idx)
    assert r[0] is y and r[1] is acc and r[2] is idx
    assert mdn.matmul_act(k["A"], k["split"], k["thr"], k["lut"], k["scale"], k["offset"], y_out=y) is y


@pytest.mark.parametrize("change,error", [
    (dict(A=lambda t: t.double()), TypeError), (dict(A=lambda t: t.cpu()), ValueError),
    (dict(A=lambda t: t.t()), ValueError), (dict(split=lambda t: t.long()), TypeError),
    (dict(thr=lambda t: t[:, :14].contiguous()), ValueError), (dict(lut=lambda t: t[:3].contiguous()), ValueError),
    (dict(lut=lambda t: t.transpose(1, 2)), ValueError), (dict(scale=lambda t: t[:2]), ValueError),
    (dict(offset=lambda t: None), TypeError), (dict(A=lambda t: 3), TypeError)])
def test_errors_as_before(call, change, error):
    k = {n: change[n](t) if n in change else t for n, t in call.items()}
    with pytest.raises(error):
        mdn.matmul(k["A"], k["split"], k["thr"], k["lut"], k["scale"], k["offset"])


@pytest.mark.parametrize("act,error", [(-1, mdn.MaddnessError), (4, mdn.MaddnessError), ("gelu", ValueError),
                                       (None, TypeError)])
def test_act_errors_as_before(call, act, error):
    k = call
    with pytest.raises(error):
        mdn.matmul_act(k["A"], k["split"], k["thr"], k["lut"], k["scale"], k["offset"], act=act)


def test_other_callers(call):
    """Parameters, empty inputs, a side stream and the current-stream context."""
    k = call
    ref = mdn.matmul(k["A"], k["split"], k["thr"], k["lut"], k["scale"], k["offset"])[0]
    q = (k["split"], k["thr"], k["lut"], k["scale"], k["offset"])
    assert same(mdn.matmul(torch.nn.Parameter(k["A"]), *q)[0], ref)
    assert mdn.matmul(k["A"][:0], *q)[0].shape == (0, 10)
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    y1 = mdn.matmul(k["A"], *q, stream=s)[0]
    with torch.cuda.stream(s):
        y2 = mdn.matmul(k["A"], *q)[0]
    torch.cuda.synchronize()
    assert same(y1, ref) and same(y2, ref)


@pytest.mark.parametrize("yes,no", [(1, 0), (np.True_, np.False_), ("acc", None)])
def test_truth_values(call, yes, no):
    """want_acc and want_idx go by truth, whatever their type."""
    k = call
    t = (k["A"], k["split"], k["thr"])
    q = (k["lut"], k["scale"], k["offset"])
    ref = mdn.matmul(*t, *q, want_acc=True, want_idx=True)
    assert same(mdn.matmul(*t, *q, want_acc=yes, want_idx=yes), ref)
    assert same(mdn.matmul(*t, *q, want_acc=yes, want_idx=no), (ref[0], ref[1], None))
    assert same(mdn.matmul(*t, *q, want_acc=no, want_idx=yes), (ref[0], None, ref[2]))
    assert same(mdn.matmul_f32(*t, k["tab"], want_idx=yes)[1], ref[2])
    assert mdn.matmul_f32(*t, k["tab"], want_idx=no)[1] is None


def test_without_native_marshalling(call, monkeypatch, tmp_path):
    """The binding serves every call itself where _calls.so is missing."""
    from paper_2207_05808_amd import _lib
    k = call
    f = lambda: (mdn.matmul(k["A"], k["split"], k["thr"], k["lut"], k["scale"], k["offset"], want_acc=True, want_idx=True)
                 + mdn.matmul_f32(k["A"], k["split"], k["thr"], k["tab"], want_idx=True))
    ref = f()
    monkeypatch.setattr(_lib, "CALLS_PATH", str(tmp_path / "none.so"))
    monkeypatch.setattr(_lib, "_calls", None)
    monkeypatch.setattr(binding, "_fused", None)
    with pytest.warns(UserWarning, match="is not used"):
        assert same(f(), ref)
    assert same(f(), ref)
