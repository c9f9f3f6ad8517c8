"""gp_encode_with that ends in an error: nothing of it may still run when it returns, for
the caller's scratch is then free for other use.

The error is forced from the host: the runtime reports an earlier call's failure
(a device number that does not exist) at the next check, which the encoder makes
after its first launches.  The stream is kept busy, so that a return without
waiting is seen.  Every kernel runs to its end on valid buffers.
"""
import ctypes
import re

import pytest
import torch

from paper_2603_20611_amd import synth

pytestmark = pytest.mark.gpu


def _hip():
    """The HIP runtime that this process already uses."""
    with open("/proc/self/maps") as f:
        path = re.search(r"\S*/libamdhip64\.so\S*", f.read()).group(0)
    return ctypes.CDLL(path)


def test_no_kernel_is_left_behind(gp):
    from paper_2603_20611_amd import binding as B
    lib = B.load()
    n = 4096
    p = torch.from_numpy(synth.gaussians_uniform(n, (64.0, 48.0, 32.0), 0.2, 0.3, seed=3)).cuda()
    codes = torch.zeros(11, n, dtype=torch.int16, device="cuda")
    header = torch.zeros(9, device="cuda")
    need = lib.gp_encode_scratch(n)
    scratch = torch.zeros(need, dtype=torch.uint8, device="cuda")
    P = lambda t: ctypes.c_void_p(t.data_ptr())
    a = torch.rand(4096, 4096, device="cuda")
    out = torch.empty_like(a)
    stream = torch.cuda.current_stream()
    torch.mm(a, a, out=out)
    torch.cuda.synchronize()
    print("[encode error]", flush=True)
    hip = _hip()
    for _ in range(20):
        torch.mm(a, a, out=out)
    assert hip.hipSetDevice(9999) != 0
    st = lib.gp_encode_with(P(p), n, n, P(codes), n, None, P(header), P(scratch), need,
                            ctypes.c_void_p(stream.cuda_stream))
    idle = stream.query()
    torch.cuda.synchronize()
    hip.hipGetLastError()
    assert st == B.GP_EHIP
    assert idle
    # and the next call works
    B.check(lib.gp_encode_with(P(p), n, n, P(codes), n, None, P(header), P(scratch), need,
                               ctypes.c_void_p(stream.cuda_stream)))
