"""The C extension that launches for the binding, on the CPU: argument kinds,
error status and the workspace retry, with calls that launch nothing."""
import ctypes
import os
import sysconfig

import numpy as np
import pytest
import torch

import paper_1911_08076_amd as P
from paper_1911_08076_amd import _ffi

X = torch.zeros(64, dtype=torch.uint8)
THR = torch.zeros(64, 4, dtype=torch.int32)


def conv(n=0):
    return P.conv_desc(n, 28, 28, 64, 64, 3, 1, 1, 2, 2, 3, 3)


def test_calls_that_launch_nothing_succeed():
    P.ifq_conv_forward(conv(), X, X, THR, X, stream=0)
    P.ifq_conv_forward(conv(), None, None, THR, None, stream=0)
    P.ifq_maxpool_codes(P.pool_desc(0, 8, 8, 64, 2, 2, 0, 2, 1), X, np.zeros(4, np.uint8),
                        stream=0)
    P.ifq_convert_codes(0, 4, 4, 64, 0, 3, X, X, stream=0)


def test_status_and_text_reach_the_caller():
    with pytest.raises(P.IfqError, match="thresholds required") as e:
        P.ifq_conv_forward(conv(), X, X, None, X, stream=0)
    assert e.value.status == _ffi.IFQ_ERR_INVALID_ARGUMENT
    with pytest.raises(P.IfqError, match="layouts"):
        P.ifq_convert_codes(1, 4, 4, 64, 0, 0, X, X, stream=0)
    with pytest.raises(P.IfqError, match="need n"):
        P.ifq_convert_codes(-1, 4, 4, 64, 0, 3, X, X, stream=0)


@pytest.mark.parametrize("call,error", [
    (lambda: P.ifq_maxpool_codes(conv(), X, X, stream=0), ctypes.ArgumentError),
    (lambda: P.ifq_conv_forward(P.pool_desc(0, 8, 8, 64, 2, 2, 0), X, X, THR, X, stream=0),
     ctypes.ArgumentError),
    (lambda: P.ifq_conv_forward(conv(), 4096, X, THR, X, stream=0), AttributeError),
    (lambda: P.ifq_conv_forward(conv(), X, X, THR, X, join=X, stream=0), ctypes.ArgumentError),
    (lambda: P.ifq_convert_codes(1, 4, 4, 64, 0.5, 3, X, X, stream=0), TypeError),
    (lambda: P.ifq_convert_codes(1, 4, 4, 64, 0.5, 3, X, X, stream=0), ctypes.ArgumentError),
    (lambda: P.ifq_convert_codes(0, 4, 4, 64, None, 3, X, X, stream=0), ctypes.ArgumentError),
    (lambda: P.ifq_convert_codes(0, 4, 4, 64, 0, None, X, X, stream=0), ctypes.ArgumentError),
    (lambda: P.ifq_convert_codes(0, 4, 4, 64, "0", 3, X, X, stream=0), ctypes.ArgumentError),
    (lambda: _ffi.call.maxpool_codes(0, X, X), TypeError),
])
def test_wrong_kinds_are_refused(call, error):
    with pytest.raises(error):
        call()


@pytest.mark.parametrize("kind", [np.int32, np.int64, np.uint8, ctypes.c_int32])
def test_integers_of_other_types_are_taken(kind):
    P.ifq_convert_codes(0, 4, 4, 64, kind(0), kind(3), X, X, stream=0)
    with pytest.raises(P.IfqError, match="layouts"):
        P.ifq_convert_codes(0, 4, 4, 64, kind(2), kind(3), X, X, stream=0)


def test_extension_is_built_for_this_interpreter(monkeypatch):
    suffix = sysconfig.get_config_var("EXT_SUFFIX")
    assert os.path.basename(_ffi.call.__file__) == "_ifqcall" + suffix
    # one that any interpreter would import must not be beside it
    assert not os.path.exists(os.path.join(_ffi.HERE, "_ifqcall.so"))
    monkeypatch.setattr(_ffi, "_lib", None)
    monkeypatch.setattr(_ffi, "CALL_PATH", os.path.join(_ffi.HERE, "missing" + suffix))
    with pytest.raises(ImportError, match="missing.*is not built"):
        _ffi.load()


class FakeCall:
    """conv_forward that asks for a workspace of `need` bytes as the library does."""
    def __init__(self, need):
        self.need, self.seen = need, []

    def conv_forward(self, d, x, w, thr, join, y, dump, ws, ws_bytes, stream):
        self.seen.append((ws, ws_bytes, stream, dump))
        return 0 if ws_bytes >= self.need else _ffi.IFQ_ERR_INSUFFICIENT_BUFFER


def test_a_layer_that_needs_a_workspace_gets_one(monkeypatch):
    from paper_1911_08076_amd import api
    fake = FakeCall(4096)
    monkeypatch.setattr(_ffi, "call", fake)
    monkeypatch.setattr(api, "ifq_conv_workspace_bytes", lambda desc: 4096)
    P.ifq_conv_forward(conv(1), X, X, THR, X, acc_dump=THR, stream=7)
    (ws0, n0, s0, _), (ws1, n1, s1, dump) = fake.seen
    assert ws0 is None and n0 == 0 and s0 == s1 == 7 and dump is THR
    assert n1 == ws1.numel() == 4096 and ws1.device == X.device and not ws1.any()
    # a workspace of the caller's that is too small is the caller's error, not retried
    fake.seen.clear()
    with pytest.raises(P.IfqError):
        P.ifq_conv_forward(conv(1), X, X, THR, X, ws=torch.zeros(64, dtype=torch.uint8), stream=7)
    assert len(fake.seen) == 1
    # and one that is large enough is passed on
    ws = torch.zeros(1024, dtype=torch.int32)
    fake.seen.clear()
    P.ifq_conv_forward(conv(1), X, X, THR, X, ws=ws, stream=7)
    assert [(a is ws, b) for a, b, _, _ in fake.seen] == [(True, 4096)]
