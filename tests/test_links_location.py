"""Where the links may lie: on the host, on the operator's device, or elsewhere (another device,
pinned host memory handed over as a device pointer), from where they are copied to the operator's
device before a kernel reads them."""
import ctypes as C

import pytest
import torch

import synth

DIMS = (4, 2, 2, 4)


class _Lib:
    """A library that accepts every call and keeps the arguments of tp_gauge_create."""

    def __getattr__(self, name):
        def call(*args):
            if name == "tp_gauge_create":
                self.links, self.where = args[1].value, args[2]
            return 0

        return call


class _CudaLinks:
    """Links on CUDA device `index`; a copy has another address."""

    def __init__(self, index, addr=0x1000):
        self.device, self.addr, self.is_cuda, self.dtype = torch.device("cuda", index), addr, True, torch.complex128
        self.shape = (4,) + DIMS[::-1] + (3, 3)

    def dim(self):
        return 7

    def to(self, device):
        return self if torch.device(device) == self.device else _CudaLinks(torch.device(device).index, self.addr + 0x1000)

    def contiguous(self):
        return self

    def data_ptr(self):
        return self.addr


@pytest.mark.parametrize("index,device,moved", [(0, 0, False), (1, 0, True), (0, 1, True), (1, 1, False)])
def test_cuda_links_reach_the_operators_device(monkeypatch, index, device, moved):
    from paper_0910_0992_amd import Operator, api
    lib = _Lib()
    monkeypatch.setattr(api.L, "load", lambda: lib)
    monkeypatch.setattr(api, "_stream_ptr", lambda d: C.c_void_p(0))
    op = Operator(_CudaLinks(index), 0.05, 3.0, device=device, allocator="hip")
    assert lib.links == (0x2000 if moved else 0x1000) and lib.where == api.L.TP_DEVICE
    op.close()


@pytest.mark.gpu
def test_links_outside_the_device_are_staged():
    """Device links are read where they lie (two allocations of their size: the planes of both
    layouts), pinned host memory handed over as a device pointer through a third one, with the
    same result."""
    from paper_0910_0992_amd import _lib as L
    lib = L.load()
    links = torch.from_numpy(synth.make_links(DIMS, 0.35, 0.2, 1100))
    nbytes = links.numel() * 16
    results = []
    for t, copies in ((links.cuda(), 2), (links.pin_memory(), 3)):
        print(f"[case] pinned={t.is_pinned()}", flush=True)
        kept, sizes = {}, []

        def alloc(n, stream, user):
            b = torch.empty(n, dtype=torch.uint8, device="cuda")
            kept[b.data_ptr()] = b
            sizes.append(n)
            return b.data_ptr()

        def free(ptr, n, stream, user):
            del kept[ptr]

        cb = L.ALLOC_FN(alloc), L.FREE_FN(free)
        ctx, gauge, ps, pt = C.c_void_p(), C.c_void_p(), C.c_double(), C.c_double()
        torch.cuda.synchronize()
        L.check(lib.tp_ctx_create((C.c_int32 * 4)(*DIMS), -1, 0, C.byref(ctx)))
        L.check(lib.tp_ctx_set_allocator(ctx, cb[0], cb[1], None))
        L.check(lib.tp_gauge_create(ctx, C.c_void_p(t.data_ptr()), L.TP_DEVICE, C.byref(gauge)))
        assert sizes.count(nbytes) == copies
        L.check(lib.tp_gauge_plaquette(gauge, C.byref(ps), C.byref(pt)))
        results.append((ps.value, pt.value))
        L.check(lib.tp_gauge_destroy(gauge))
        L.check(lib.tp_ctx_destroy(ctx))
        assert not kept
    assert results[0] == results[1]
