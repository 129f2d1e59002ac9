"""The binding enqueues on torch's current stream, whichever that is: a call between two operations of a stream reads what the one before it
wrote and is read by the one behind it, while the default stream is idle."""
import pytest
import torch

import paper_1801_04380_amd as sn
from paper_1801_04380_amd import workloads as wl

pytestmark = pytest.mark.gpu
N, C, H, W, K = 2, 16, 16, 16, 16


def _pass(x, w, y, dx, act, sh):
    sn.sn_conv2d_fwd(x, w, y, sh)
    sn.sn_relu_fwd(y, act)
    sn.sn_conv2d_bwd_data(act, w, dx, sh)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_calls_run_on_the_current_stream(dtype):
    t, code = (torch.bfloat16, sn.SN_BF16) if dtype == "bf16" else (torch.float32, sn.SN_F32)
    sh = sn.conv_shape(N, C, H, W, K, 3, 3, (1, 1), (1, 1), code, code)
    x, w = (wl.activation(s, dtype, i).cuda() for s, i in (((N, C, H, W), 3), ((K, C, 3, 3), 4)))
    bufs = [[torch.zeros((N, C, H, W), dtype=t, device="cuda") for _ in range(3)] for _ in range(3)]
    _pass(x, w, *bufs[0], sh)
    torch.cuda.synchronize()
    late = [torch.zeros_like(x) for _ in range(2)]
    streams = [torch.cuda.Stream() for _ in range(2)]
    for s in streams:
        s.wait_stream(torch.cuda.current_stream())
    for s, xl, b in zip(streams, late, bufs[1:]):
        with torch.cuda.stream(s):
            torch.cuda._sleep(20_000_000)   # some milliseconds: on another stream the calls would be done before x is there
            xl.copy_(x)
            _pass(xl, w, *b, sh)
            b[2].add_(1)
    torch.cuda.synchronize()
    for y, dx, act in bufs[1:]:
        assert torch.equal(y, bufs[0][0]) and torch.equal(dx, bufs[0][1]) and torch.equal(act, bufs[0][2] + 1)
