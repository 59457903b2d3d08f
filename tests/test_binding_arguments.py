"""What the binding takes and refuses before it touches the device.  No call here launches anything: the arguments are
host tensors, and every one of them is refused (or, where it is accepted, the call stops at the missing device)."""
import os

import numpy as np
import pytest
import torch

import paper_2103_14949_amd as hago


@pytest.fixture(scope="module", autouse=True)
def built():
    if not os.path.exists(hago.library_path()):
        from paper_2103_14949_amd import build
        build.build()


I8 = hago.QType(hago.I8)
MULT, SHIFT = torch.full((4,), 2 ** 30, dtype=torch.int32), torch.zeros(4, dtype=torch.int32)
ACC = torch.zeros(1, 4, 2, dtype=torch.int32)


@pytest.mark.parametrize("mult,shift", [
    (MULT.numpy(), SHIFT), (MULT.tolist(), SHIFT), (2 ** 30, SHIFT), (np.int32(2 ** 30), SHIFT),
    (MULT, SHIFT.numpy()), (None, [0, 0, 0, 0]), (MULT.numpy(), SHIFT.numpy())])
def test_requant_parameters_that_are_not_tensors_are_refused(mult, shift):
    """Only multiplier None selects the shift-only form; anything else that is no tensor is an error."""
    rq = hago.Requant(mult, shift, I8, per_channel=1)
    a, w = torch.zeros(2, 16, dtype=torch.int8), torch.zeros(4, 16, dtype=torch.int8)
    for call in (lambda: hago.requantize(ACC, rq),
                 lambda: hago.qdense(a, I8, w, I8, None, hago.I32, rq),
                 lambda: hago.qdense(a, I8, w, I8, None, hago.I32, rq, prepare=True),
                 lambda: hago.qconv2d(a.view(1, 2, 4, 4), I8, w.view(4, 2, 2, 4), I8, rq=rq)):
        with pytest.raises(TypeError):
            call()


@pytest.mark.parametrize("lo,hi,per_channel", [
    (-128.0, 127.0, None), (np.float32(-128), np.int64(127), np.bool_(True)), (torch.tensor(-128), torch.tensor(127.0), 1.0),
    (-128, 127, np.bool_(False)), (True, 5.9, False)])
def test_clip_limits_and_per_channel_are_converted_with_int(lo, hi, per_channel):
    """The operators take whatever int() takes; without a device such a call gets as far as its output's allocation."""
    x = torch.zeros(1, 4, 2)
    scale, zp = torch.ones(4), torch.zeros(4, dtype=torch.int32)
    I8 = hago.QType(hago.I8)
    I8.is_signed = np.bool_(True)
    for call in (lambda: hago.simquant(x, scale, zp, I8, lo, hi, per_channel),
                 lambda: hago.simquant_wrap(x, scale, zp, I8, lo, hi, per_channel),
                 lambda: hago.quantize(x, scale, zp, I8, lo, hi, per_channel),
                 lambda: hago.simquant_codes(x, scale, zp, I8, lo, hi, per_channel),
                 lambda: hago.dequantize(x.to(torch.int8), I8, scale, zp, per_channel)):
        with pytest.raises(RuntimeError) as e:   # no TypeError: the arguments were taken
            call()
        assert not isinstance(e.value, hago.HagoError)


@pytest.mark.parametrize("lo", ["x", [1], 1j, float("nan"), float("inf")])
def test_clip_limits_that_int_refuses_are_refused(lo):
    x, scale, zp = torch.zeros(1, 4, 2), torch.ones(4), torch.zeros(4, dtype=torch.int32)
    for call in (lambda: hago.simquant(x, scale, zp, I8, lo), lambda: hago.quantize(x, scale, zp, I8, None, lo)):
        with pytest.raises((TypeError, ValueError, OverflowError)):
            call()


def _dense(a=torch.zeros(2, 16, dtype=torch.int8), w=torch.zeros(4, 16, dtype=torch.int8), **k):
    return hago.qdense(a, k.pop("a_t", I8), w, I8, **k)


def _conv(a=torch.zeros(1, 2, 4, 4, dtype=torch.int8), w=torch.zeros(4, 2, 2, 4, dtype=torch.int8), **k):
    return hago.qconv2d(a, I8, w, I8, **k)


@pytest.mark.parametrize("call,error", [
    (lambda: _dense(a=np.zeros((2, 16), np.int8)), TypeError),
    (lambda: _dense(a=None), TypeError),
    (lambda: _dense(w=torch.zeros(4, 15, dtype=torch.int8)), AssertionError),
    (lambda: _dense(a=torch.zeros(2, 4, 4, dtype=torch.int8)), AssertionError),
    (lambda: _dense(a=torch.zeros(16, 2, dtype=torch.int8).T), AssertionError),
    (lambda: _dense(bias=[0, 0, 0, 0]), TypeError),
    (lambda: _dense(out=np.zeros((2, 4), np.int32)), TypeError),
    (lambda: _dense(acc_dtype="int32"), TypeError),
    (lambda: _dense(acc_dtype=77), KeyError),
    (lambda: _dense(a_t=None), AttributeError),
    (lambda: _dense(flags=1.0), TypeError),
    (lambda: _dense(rq=object()), AttributeError),
    (lambda: _conv(a=torch.zeros(2, 4, 4, dtype=torch.int8)), AssertionError),
    (lambda: _conv(a=torch.zeros(1, 4, 4, 2, dtype=torch.int8).permute(0, 3, 1, 2)), AssertionError),
    (lambda: _conv(stride=(0, 1)), ZeroDivisionError),
    (lambda: _conv(stride=(1,)), IndexError),
    (lambda: _conv(stride=2), TypeError),
    (lambda: _conv(pad=(0.5, 0)), TypeError),
    (lambda: _conv(groups=None), TypeError),
    (lambda: hago.simquant(torch.zeros(4, 2), torch.ones(4), torch.zeros(4), I8), AssertionError),
    (lambda: hago.simquant(torch.zeros(1, 4, 2), [1.0], torch.zeros(4), I8), TypeError),
    (lambda: hago.simquant(torch.zeros(1, 4, 2), torch.ones(4), torch.zeros(4), hago.QType(hago.I8, 99)), hago.HagoError),
    (lambda: hago.quantize(torch.zeros(2, 4, 2).permute(1, 0, 2), torch.ones(4), torch.zeros(4), I8), AssertionError),
    (lambda: hago.simquant_batched(torch.zeros(1, 4, 2), torch.ones(2, 4), torch.zeros(2, 4), I8, [-1, -1], [1]), AssertionError),
    (lambda: hago.simquant_batched(torch.zeros(1, 4, 2), torch.ones(2, 4), torch.zeros(2, 4), I8, -1, 1), TypeError),
    (lambda: hago.absmax(torch.zeros(4, 2)), AssertionError),
    (lambda: hago.absmax(torch.zeros(1, 4, 2), out=[0.0] * 4), TypeError),
    (lambda: hago.requantize(torch.zeros(4, 2, dtype=torch.int32), hago.Requant(MULT, SHIFT, I8)), AssertionError),
])
def test_refusals(call, error):
    with pytest.raises(error):
        call()
