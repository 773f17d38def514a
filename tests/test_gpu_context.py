"""Work that a context enqueues while it is created."""
import ctypes as C

import pytest
import torch

pytestmark = pytest.mark.gpu


def test_context_buffers_are_cleared_when_creation_returns():
    """The reduction tickets are cleared on the stream bound at creation (the null stream) and used
    on whatever stream is bound later: creation waits for the clearing, behind the work that the
    null stream holds already."""
    from paper_0910_0992_amd import _lib as L
    lib = L.load()
    a = torch.randn(8192, 8192, device="cuda")
    b = torch.empty_like(a)
    torch.mm(a, a, out=b)
    torch.cuda.synchronize()
    done = torch.cuda.Event()
    with torch.cuda.stream(torch.cuda.default_stream()):
        for _ in range(40):  # about 0.3 s
            torch.mm(a, a, out=b)
        done.record()
    assert not done.query()
    ctx = C.c_void_p()
    L.check(lib.tp_ctx_create((C.c_int32 * 4)(4, 4, 4, 8), -1, 0, C.byref(ctx)))
    finished = done.query()
    L.check(lib.tp_ctx_destroy(ctx))
    assert finished
