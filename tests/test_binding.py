"""Host-only checks of the Python binding: what it refuses before it calls the library."""
import os
import shutil
import warnings

import pytest
import torch

import paper_2510_21956_amd as la
from paper_2510_21956_amd import binding


class DeviceTensor:
    """Stands for a device tensor: the shape, strides and type of a host tensor, on device 0."""
    is_cuda = True

    def __init__(self, t):
        self.t, self.shape, self.dtype = t, t.shape, t.dtype

    def get_device(self):
        return 0

    def __getattr__(self, name):  # dim, is_contiguous, numel, element_size, data_ptr
        return getattr(self.t, name)


def _calls(q):
    """Every entry point that takes tensors, with q as its first tensor and packed others."""
    B, H, N, D = 2, 3, 8, 16
    x = lambda: DeviceTensor(torch.zeros(B, H, N, D))
    G = DeviceTensor(torch.zeros(B, H, N))
    ws = DeviceTensor(torch.zeros(1 << 16, dtype=torch.uint8))
    st = DeviceTensor(torch.zeros(1 << 12))
    fwd = (q, x(), x(), x(), G, 1.0, 0.5, True)
    bwd = (q, x(), x(), x(), G, x(), x(), x(), x(), 1.0, 0.5, True, ws)
    return [lambda: la.la_forward(*fwd, ws), lambda: la.la_forward_traced(*fwd, ws),
            lambda: la.la_forward_static(*fwd), lambda: la.la_forward_save(*fwd, ws, None),
            lambda: la.la_forward_qknorm(*fwd, ws), lambda: la.la_forward_qknorm_save(*fwd, ws, None),
            lambda: la.la_backward(*bwd), lambda: la.la_backward_traced(*bwd),
            lambda: la.la_backward_saved(*bwd, None), lambda: la.la_backward_qknorm(*bwd),
            lambda: la.la_backward_qknorm_saved(*bwd, None),
            lambda: la.la_backward_ab(q, x(), x(), x(), G, x(), st, 1.0, 0.5, True, ws),
            lambda: la.la_decode_step(q, x(), x(), x(), G, st, 1.0, 0.5),
            lambda: la.la_decode_prefill(q, x(), st, 0, ws)]


@pytest.mark.parametrize("form", ["transposed", "expanded", "strided", "host"])
def test_first_tensor_is_checked_like_the_others(monkeypatch, form):
    """A first tensor whose elements do not lie one after another is refused, not read as if they
    did (an expanded one is smaller than what the kernels would read)."""
    def reached():
        raise AssertionError("the library was reached")
    monkeypatch.setattr(binding, "load_library", reached)
    q = {"transposed": torch.zeros(2, 8, 3, 16).transpose(1, 2),
         "expanded": torch.zeros(1, 1, 8, 16).expand(2, 3, 8, 16),
         "strided": torch.zeros(2, 3, 8, 32)[..., ::2],
         "host": torch.zeros(2, 3, 8, 16)}[form]
    q = q if form == "host" else DeviceTensor(q)
    for call in _calls(q):
        with pytest.raises(ValueError):
            call()


def test_packed_first_tensor_reaches_the_library(monkeypatch):
    class Reached(Exception):
        pass

    def reached():
        raise Reached
    monkeypatch.setattr(binding, "load_library", reached)
    for call in _calls(DeviceTensor(torch.zeros(2, 3, 8, 16))):
        with pytest.raises(Reached):
            call()


@pytest.mark.parametrize("form", ["fits", "absent", "not a library", "a header alone", "another torch"])
def test_marshalling_that_does_not_load_is_left_out(monkeypatch, tmp_path, form):
    """The library loads at the first call and at every later one, on the Python functions if need be, with one
    warning where a file is there and not used."""
    path = tmp_path / "_marshal.so"
    la.load_library()
    if not os.path.exists(binding._MARSHAL_PATH):
        pytest.skip("_marshal.so is not built")
    if form in ("fits", "another torch"):
        shutil.copy(binding._MARSHAL_PATH, path)
    elif form == "a header alone":
        path.write_bytes(open(binding._MARSHAL_PATH, "rb").read()[:64])
    elif form == "not a library":
        path.write_text("text")
    if form == "another torch":
        monkeypatch.setattr(torch, "__version__", "1.0.0")
    for name, value in (("_MARSHAL_PATH", str(path)), ("_lib", None), ("_native", None)):
        monkeypatch.setattr(binding, name, value)
    with warnings.catch_warnings(record=True) as seen:
        warnings.simplefilter("always")
        lib = la.load_library()
        assert la.load_library() is lib and la.la_version() >= 100
    assert (binding._native is not None) == (form == "fits")
    assert [w.category for w in seen] == ([] if form in ("fits", "absent") else [RuntimeWarning])


@pytest.mark.parametrize("compiler", ["/nonexistent/c++", "false"])
def test_build_goes_on_without_the_marshalling(monkeypatch, tmp_path, compiler):
    """No host compiler, or one that fails (torch's headers missing): a warning, and no stale file."""
    from paper_2510_21956_amd import build
    stale = tmp_path / "_marshal.so"
    stale.write_text("of an older library")
    monkeypatch.setattr(build, "CXX", compiler, raising=False)
    real = build.subprocess.run
    monkeypatch.setattr(build.subprocess, "run", lambda cmd, **k: real([compiler] + cmd[1:], **k))
    with pytest.warns(RuntimeWarning, match="not built"):
        assert build.build_marshal(out=str(stale)) is None
    assert not stale.exists()
