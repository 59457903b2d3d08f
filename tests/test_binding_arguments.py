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
