"""Which kernel serves a convolution, on the CPU: the layers that the GPU tests of the streamed channel-last convolution run at reach
it, with each of its tiles."""
import pytest

import test_gpu_conv_forms as forms
import test_gpu_conv_stream as stream


@pytest.mark.parametrize("shape,tile", [(0, "2,2,1,1,4,2,2,false"), (1, "1,4,2,1,4,2,2,false")])
def test_streamed_convolution(routes, shape, tile):
    layers = stream.CASES + [x for x in forms.CASES if x[1] % 16 == 0]
    assert len(layers) > len(stream.CASES)
    calls = [f"conv {act} 1 {B} {C} {H} {W} {O} {KH} {KW} {sh} {sw} {ph} {pw} {raw} 5 {shape}"
             for B, C, H, W, O, KH, KW, (sh, sw), (ph, pw) in layers for act in ("u8", "i8") for raw in (0, 1)]
    for call, kernels in zip(calls, routes(calls)):
        assert len(kernels) == 1 and kernels[0].startswith(f"qgemm_dma_kernel<{tile},"), (call, kernels)
