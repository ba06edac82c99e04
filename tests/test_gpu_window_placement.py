"""Small one-kernel windows play on one XCD on streams that have every compute unit, and on no others: a stream's mask may leave that
XCD too few of them."""
import ctypes
from types import SimpleNamespace

import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,d,B,one_xcd", [(2, 1000, 8, True), (16, 1000, 8, True), (17, 1000, 8, False), (2, 1000, 32, True), (8, 1000, 32, True), (9, 1000, 32, False),
                                         (30, 4, 4, True), (31, 4, 4, False), (48, 8, 8, True), (49, 8, 8, False), (64, 16, 8, True), (48, 3, 8, True), (49, 3, 8, False)])
def test_windows_on_masked_streams_are_spread(n, d, B, one_xcd):
    import torch
    import paper_2306_00256_amd as P
    from paper_2306_00256_amd import binding as Bn
    assert torch.cuda.is_available()
    P.lib()
    hip = ctypes.CDLL("libamdhip64.so.7")
    # 32 units, and all but four of the 256
    masks = [(ctypes.c_uint32 * 8)(0xFFFFFFFF), (ctypes.c_uint32 * 8)(0xFFFFFFF0, *[0xFFFFFFFF] * 7)]
    streams = []
    try:
        for bits in masks:
            streams.append(ctypes.c_void_p())
            assert hip.hipExtStreamCreateWithCUMask(ctypes.byref(streams[-1]), ctypes.c_uint32(8), bits) == 0
        gen = torch.Generator(device="cuda").manual_seed(n + B)
        N, iters, lr = B + 3, 9, 0.001
        A = torch.randn((n, N, d), generator=gen, device="cuda")
        t = torch.randn((n, N), generator=gen, device="cuda")
        idx = torch.randint(0, N, (iters, n, B), dtype=torch.int32, device="cuda", generator=gen)
        S = 0.1 * torch.randn((2 * n, d), generator=gen, device="cuda")
        loss = Bn.make_minibatch_loss(Bn.LOSS_LSQ, A, t, N, B)
        ws = torch.empty(P.dsgd_ceca_run_workspace_bytes(n, d, loss), dtype=torch.uint8, device="cuda")
        ref = torch.empty_like(S)
        P.dsgd_ceca_run(S, ref, n, d, loss, idx, lr, 0, iters, 2, workspace=ws)
        assert P.ceca_last_form() == Bn.FORM_RUN_WINDOW and Bn.ceca_last_window_on_one_xcd() == one_xcd
        for stream, units in zip(streams, (32, 252)):
            out = torch.full_like(S, float("nan"))
            torch.cuda.synchronize()
            P.dsgd_ceca_run(S, out, n, d, loss, idx, lr, 0, iters, 2, workspace=ws, stream=SimpleNamespace(cuda_stream=stream.value))
            torch.cuda.synchronize()
            if P.ceca_last_form() == Bn.FORM_RUN_WINDOW:
                assert not Bn.ceca_last_window_on_one_xcd(), units
            else:
                assert n > 2 and units == 32                     # more than an eighth of the 32 units' places
            assert torch.equal(out, ref), units
    finally:
        for stream in streams:
            assert hip.hipStreamDestroy(stream) == 0
