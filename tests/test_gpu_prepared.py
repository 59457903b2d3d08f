"""The call objects that prepare=True returns: their attribute, what they refuse and what they keep alive."""
import gc

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

from gpu_util import *  # noqa: E402,F401,F403


def _layer(rng):
    a, w = rng.integers(-128, 128, (5, 40)).astype(np.int8), rng.integers(-127, 128, (24, 40)).astype(np.int8)
    mult, shift = rng.integers(2 ** 30, 2 ** 31, 24).astype(np.int32), np.full(24, 9, np.int32)
    return a, w, mult, shift


def test_out_can_be_set_and_the_launch_keeps_its_buffer():
    a, w, mult, shift = _layer(np.random.default_rng(1))
    want = ref.qdense(a, 0, w, None, ref.I32, ref_requant(mult, shift))
    call = hago.qdense(dev(a), hago.QType(hago.I8), dev(w), hago.QType(hago.I8), None, hago.I32, gpu_requant(mult, shift), prepare=True)
    written = call.out.data_ptr()
    call.out = "elsewhere"
    gc.collect()
    taken = [torch.full((5, 24), 77, dtype=torch.int8, device=DEV) for _ in range(64)]   # would reuse a freed buffer
    assert call() == "elsewhere" and call.out == "elsewhere"
    torch.cuda.synchronize()
    assert all(t.data_ptr() != written and bool((t == 77).all()) for t in taken)
    with pytest.raises(AttributeError):
        del call.out
    again = hago.qdense(dev(a), hago.QType(hago.I8), dev(w), hago.QType(hago.I8), None, hago.I32, gpu_requant(mult, shift), prepare=True)
    mine = again.out
    assert again() is mine
    assert_same(host(mine), want)


def test_calls_take_no_arguments():
    call = hago.absmax(dev(np.ones((1, 4, 8), np.float32)), prepare=True)
    for bad in (lambda: call(1), lambda: call(out=None)):
        with pytest.raises(TypeError):
            bad()
    assert_same(host(call()), np.ones(4, np.float32))


@pytest.mark.parametrize("kind", ["dense", "conv", "requantize"])
def test_requant_tensors_outlive_their_attributes(kind):
    """Parameters that a search sets anew do not pull the tensors from under a call that was marshalled before."""
    a, w, mult, shift = _layer(np.random.default_rng(2))
    rq, i8 = gpu_requant(mult, shift), hago.QType(hago.I8)
    rr = ref_requant(mult, shift)
    if kind == "dense":
        call, want = hago.qdense(dev(a), i8, dev(w), i8, rq=rq, prepare=True), ref.qdense(a, 0, w, None, ref.I32, rr)
    elif kind == "conv":
        a4, w4 = a.reshape(5, 10, 2, 2), w.reshape(24, 10, 2, 2)
        call = hago.qconv2d(dev(a4), i8, dev(w4), i8, rq=rq, prepare=True)
        want = ref.qconv2d(a4, 0, w4, None, ref.NCHW, (1, 1), (0, 0), 1, ref.I32, rr)
    else:
        acc = np.random.default_rng(3).integers(-2 ** 17, 2 ** 17, (1, 24, 16)).astype(np.int32)
        call, want = hago.requantize(dev(acc), rq, prepare=True), ref.requantize(acc, rr)
    addresses = {rq.multiplier.data_ptr(), rq.shift.data_ptr()}
    rq.multiplier = rq.shift = None
    gc.collect()
    taken = [torch.zeros(24, dtype=torch.int32, device=DEV) for _ in range(64)]   # would reuse freed tensors
    assert_same(host(call()), want, kind)
    assert not addresses & {t.data_ptr() for t in taken}
