"""GPU parity: dsgd_ceca_run (several minibatch iterations per call; each iteration after the first finishes
the iteration before inside its gradient kernel: one kernel per iteration where the one-pass gradient
applies, two where the gradient takes two passes) against single dsgd_ceca_step calls (bit for bit) and
against the fp64 oracle (1e-4 over the run)."""
import numpy as np
import pytest

import workloads as WL
from oracle import ceca as OC
from oracle import losses as OL
from oracle import schedule as OS
from gpu_util import make_state, rel_err, split_state

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    import torch
    import paper_2306_00256_amd as P
    assert torch.cuda.is_available()
    P.lib()
    return torch, P


def _aligned(torch, nbytes):
    buf = torch.empty(nbytes + 256, dtype=torch.uint8, device="cuda")
    return buf[(-buf.data_ptr()) % 256:][:nbytes]


def _problem(torch, Bn, kind, n, N, d, B, iters, seed, noise=0.0):
    if kind == "lsq":
        A, t, _ = WL.lsq_data(n, N, d, seed=seed)
    else:
        A, t, _ = WL.logistic_data_sparse(n, N, d, seed=seed, density=0.5)
    idx = WL.batch_indices(n, N, B, iters, seed=seed)
    Ad, td, idxd = torch.from_numpy(A).cuda(), torch.from_numpy(t).cuda(), torch.from_numpy(idx).cuda()
    code = Bn.LOSS_LSQ if kind == "lsq" else Bn.LOSS_LOGISTIC
    return A, t, idx, Ad, td, idxd, code


@pytest.mark.parametrize("kind", ["lsq", "logistic"])
@pytest.mark.parametrize("n,port,d,B,ld", [(130, 2, 4096, 16, None), (128, 1, 2052, 5, 2056), (129, 2, 8192, 9, None),
                                           (130, 1, 16384, 3, None), (131, 2, 1100, 40, None),
                                           (6, 1, 1000, 8, None), (5, 2, 4100, 7, None), (130, 2, 515, 4, None),
                                           (258, 1, 10, 50, None), (12, 2, 63, 9, None), (9, 2, 255, 20, 258),
                                           (6, 1, 1023, 12, None), (6, 2, 1027, 5, None), (4, 2, 1000, 40, None),
                                           (6, 2, 10000, 32, None), (30, 1, 8192, 16, 8192 + 64), (7, 2, 2000, 33, 2064),
                                           (6, 1, 1500, 6, 1501)])
def test_run_equals_single_steps_and_oracle(env, kind, n, port, d, B, ld):
    torch, P = env
    from paper_2306_00256_amd import binding as Bn
    N, iters, k0, lr, noise = 10, 7, 4, 0.002, 0.05
    A, t, idx, Ad, td, idxd, code = _problem(torch, Bn, kind, n, N, d, B, iters, seed=n + d)
    tau = OS.num_rounds(n)
    x0 = 0.05 * WL.initial_state(n, d, seed=n + 1)
    y0 = 0.05 * WL.initial_state(n, d, seed=n + 2)
    mk = lambda k: Bn.make_minibatch_loss(code, Ad, td, N, B, noise_std=noise, seed=9, k=k)
    # reference: one dsgd_ceca_step per iteration
    ws1 = _aligned(torch, P.dsgd_ceca_workspace_bytes(n, d, mk(0)))
    S = make_state(torch, x0, y0=y0, ld=ld)
    T = S if port == 1 else make_state(torch, np.zeros_like(x0), ld=ld)
    mid = None
    for t_ in range(iters):
        if t_ == iters - 1:
            mid = S.clone()                                  # the state after iters - 1 iterations
        P.dsgd_ceca_step(S, T, n, d, mk(k0 + t_), idxd[t_], lr, (k0 + t_) % tau, port, workspace=ws1)
        if T is not S:
            S, T = T, S
    rx, ry = split_state(S, n, d)
    ws = _aligned(torch, P.dsgd_ceca_run_workspace_bytes(n, d, mk(0)))
    # fused iterations keep the state in half-step form between them (default) or as full states with two
    # message buffers; shapes on the two-pass gradient are not affected by the switch
    for half in (1, 0):
        P.ceca_set_option(Bn.OPT_HALF_STEP_RUN, half)
        for inplace in (False, True):
            for count in (iters, iters - 1):                 # odd and even: the closing combine always reads the copy
                A_ = make_state(torch, x0, y0=y0, ld=ld)
                B_ = A_ if inplace else make_state(torch, np.zeros_like(x0), ld=ld)
                P.dsgd_ceca_run(A_, B_, n, d, mk(k0), idxd, lr, k0 % tau, count, port, workspace=ws)
                if count == iters:
                    gx, gy = split_state(B_, n, d)
                    assert np.array_equal(gx, rx) and np.array_equal(gy, ry), (half, inplace)
                else:
                    assert torch.equal(B_[:, :d], mid[:, :d]), (half, inplace, "one iteration fewer")
                if not inplace:
                    ax, ay = split_state(A_, n, d)
                    assert np.array_equal(ax, x0.astype(np.float64)) and np.array_equal(ay, y0.astype(np.float64))
                if ld is not None:
                    assert bool((B_[:, d:] == 12345.0).all())
    P.ceca_reset_options()
    grad = OL.make_minibatch_grad(kind, A, t, idx, k0=k0, noise_std=noise, seed=9)
    x, y = OC.run(x0, port, lr, grad, iters, store32=True, y0=y0, k0=k0)
    assert max(rel_err(rx, x)) <= 1e-4 and max(rel_err(ry, y)) <= 1e-4


def test_single_iteration_and_argument_errors(env):
    torch, P = env
    from paper_2306_00256_amd import binding as Bn
    n, d, N, B = 130, 4096, 6, 4
    A, t, idx, Ad, td, idxd, code = _problem(torch, Bn, "lsq", n, N, d, B, 2, seed=1)
    loss = Bn.make_minibatch_loss(code, Ad, td, N, B)
    x0 = 0.05 * WL.initial_state(n, d, seed=2)
    ws = _aligned(torch, P.dsgd_ceca_run_workspace_bytes(n, d, loss))
    S1, T1 = make_state(torch, x0), make_state(torch, np.zeros_like(x0))
    P.dsgd_ceca_step(S1, T1, n, d, loss, idxd[0], 0.01, 0, 2, workspace=_aligned(torch, P.dsgd_ceca_workspace_bytes(n, d, loss)))
    S2, T2 = make_state(torch, x0), make_state(torch, np.zeros_like(x0))
    P.dsgd_ceca_run(S2, T2, n, d, loss, idxd, 0.01, 0, 1, 2, workspace=ws)
    assert torch.equal(T1, T2)
    for kwargs, code_ in [(dict(iters=0), Bn.CECA_EINVAL), (dict(ws=ws[:1024]), Bn.CECA_EWORKSPACE), (dict(ws=None), Bn.CECA_EWORKSPACE)]:
        with pytest.raises(P.CecaError) as e:
            P.dsgd_ceca_run(S2, T2, n, d, loss, idxd, 0.01, 0, kwargs.get("iters", 2), 2, workspace=kwargs.get("ws", ws))
        assert e.value.code == code_
    c = torch.zeros((n, d), dtype=torch.float32, device="cuda")
    with pytest.raises(P.CecaError) as e:
        P.dsgd_ceca_run(S2, T2, n, d, Bn.make_quad_center_loss(c, 0.0, 0, 0), idxd, 0.01, 0, 2, 2, workspace=ws)
    assert e.value.code == Bn.CECA_EINVAL


@pytest.mark.parametrize("iters", [2, 3, 4, 5])
@pytest.mark.parametrize("n,port,d,B", [(8, 2, 20000, 32), (6, 1, 2051, 9)])
def test_two_pass_shapes_for_every_parity_of_the_iteration_count(env, iters, n, port, d, B):
    """Shapes on the two-pass gradient alternate the state between S_out and a copy in the workspace: the
    result must land in S_out for odd and even iteration counts, in place and out of place."""
    torch, P = env
    from paper_2306_00256_amd import binding as Bn
    N, lr = 12, 0.003
    A, t, idx, Ad, td, idxd, code = _problem(torch, Bn, "logistic", n, N, d, B, iters, seed=iters)
    tau = OS.num_rounds(n)
    x0 = 0.05 * WL.initial_state(n, d, seed=3)
    loss = Bn.make_minibatch_loss(code, Ad, td, N, B)
    ws1 = _aligned(torch, P.dsgd_ceca_workspace_bytes(n, d, loss))
    S = make_state(torch, x0)
    for t_ in range(iters):
        P.dsgd_ceca_step(S, S, n, d, loss, idxd[t_], lr, (1 + t_) % tau, port, workspace=ws1)
    ws = _aligned(torch, P.dsgd_ceca_run_workspace_bytes(n, d, loss))
    for inplace in (False, True):
        A_ = make_state(torch, x0)
        B_ = A_ if inplace else torch.full_like(A_, float("nan"))
        P.dsgd_ceca_run(A_, B_, n, d, loss, idxd, lr, 1 % tau, iters, port, workspace=ws)
        assert P.ceca_last_form() == Bn.FORM_RUN_TWO_PASS
        assert torch.equal(B_, S), (iters, inplace)


@pytest.mark.parametrize("n,port,d,B,window", [
    (2, 1, 4, 1, True), (3, 2, 1024, 8, True), (8, 1, 1020, 9, True), (96, 2, 1024, 16, True), (97, 2, 1024, 16, False), (64, 1, 512, 17, True),
    (5, 2, 600, 32, True), (4, 1, 1024, 33, True), (32, 2, 1000, 64, True), (7, 2, 1028, 8, True), (32, 1, 4096, 16, True), (33, 2, 4096, 9, False),
    (5, 2, 4096, 17, True), (8, 1, 4100, 9, True), (6, 2, 9984, 32, False), (2, 2, 9000, 64, True), (384, 1, 64, 16, True), (385, 2, 64, 16, False),
    (512, 1, 63, 16, True), (512, 2, 64, 64, False), (512, 2, 63, 17, True), (513, 2, 63, 17, False), (2, 2, 1, 64, True), (9, 2, 65, 16, True),
    (512, 1, 256, 8, True), (257, 2, 252, 9, True), (256, 2, 256, 32, True), (128, 1, 64, 33, True), (129, 2, 256, 64, False), (9, 2, 260, 40, True),
    (128, 2, 255, 17, True), (10, 1, 257, 33, True), (32, 2, 1023, 64, True), (4, 1, 1999, 4, True), (2, 2, 1025, 9, True), (3, 2, 2049, 8, False)])
def test_long_windows_at_the_edges_of_the_shapes(env, n, port, d, B, window):
    """Windows of many iterations (every message slot is used again and again), at the edges of workgroup sizes, batch
    tiles, chunk counts, resident agents and the words that fit the workspace: the bits of the form with one or two
    kernels per iteration, twice on the same workspace, and two windows on two streams at once; the one-kernel form
    inside those edges and another one outside."""
    torch, P = env
    from paper_2306_00256_amd import binding as Bn
    N, iters, lr = max(B // 2, 3), 61, 0.02 / (d * B) ** 0.5
    gen = torch.Generator(device="cuda").manual_seed(n * d + B)
    A = torch.randn((n, N, d), generator=gen, device="cuda")
    t = torch.randn((n, N), generator=gen, device="cuda").sign()
    idx = torch.randint(0, N, (iters, n, B), dtype=torch.int32, device="cuda", generator=gen)
    S = torch.randn((2 * n, d), generator=gen, device="cuda")
    loss = Bn.make_minibatch_loss(Bn.LOSS_LOGISTIC, A, t, N, B, noise_std=0.01, seed=5)
    nbytes = P.dsgd_ceca_run_workspace_bytes(n, d, loss)
    ws = [torch.full((nbytes + 256,), 255, dtype=torch.uint8, device="cuda") for _ in range(2)]
    ws = [w[(-w.data_ptr()) % 256:][:nbytes] for w in ws]
    ref, got = torch.empty_like(S), [torch.full_like(S, float("nan")) for _ in range(2)]
    P.ceca_set_option(Bn.OPT_HALF_STEP_RUN, 0)
    P.dsgd_ceca_run(S, ref, n, d, loss, idx, lr, 1 % OS.num_rounds(n), iters, port, workspace=ws[0])
    P.ceca_reset_options()
    assert bool(torch.isfinite(ref).all()) and P.ceca_last_form() != Bn.FORM_RUN_WINDOW
    for _ in range(2):
        P.dsgd_ceca_run(S, got[0], n, d, loss, idx, lr, 1 % OS.num_rounds(n), iters, port, workspace=ws[0])
        assert (P.ceca_last_form() == Bn.FORM_RUN_WINDOW) == window
        assert torch.equal(got[0], ref)
    torch.cuda.synchronize()
    got[0].fill_(float("nan"))
    streams = [torch.cuda.Stream() for _ in range(2)]
    torch.cuda.synchronize()
    for s, w, g in zip(streams, ws, got):
        P.dsgd_ceca_run(S, g, n, d, loss, idx, lr, 1 % OS.num_rounds(n), iters, port, workspace=w, stream=s)
    torch.cuda.synchronize()
    assert torch.equal(got[0], ref) and torch.equal(got[1], ref)


@pytest.mark.parametrize("kind", ["lsq", "logistic"])
@pytest.mark.parametrize("n,port,d,B", [(2, 1, 4, 1), (3, 2, 1024, 8), (6, 1, 1020, 9), (70, 2, 1024, 16), (5, 2, 256, 17), (63, 2, 1024, 32),
                                        (64, 1, 1024, 32), (65, 2, 1024, 32), (258, 1, 10, 50), (2, 2, 1, 64), (9, 2, 64, 16), (9, 2, 65, 17),
                                        (4, 1, 255, 16), (7, 2, 253, 64), (6, 2, 1024, 33), (5, 2, 257, 8), (9, 2, 256, 8), (9, 2, 252, 32), (9, 2, 260, 9)])
def test_single_launch_step_equals_the_two_kernel_form(env, kind, n, port, d, B):
    """One out-of-place step whose workgroups also evaluate their peer's message, at the edges of its workgroup sizes,
    batch tiles and size limit (and just past them), every round of a cycle: the bits of gradient kernel + combine."""
    torch, P = env
    from paper_2306_00256_amd import binding as Bn
    N, lr = max(B // 2, 3), 0.02 / (d * B) ** 0.5
    gen = torch.Generator(device="cuda").manual_seed(n * d + B)
    A = torch.randn((n, N, d), generator=gen, device="cuda")
    t = torch.randn((n, N), generator=gen, device="cuda").sign()
    idx = torch.randint(-1, N + 1, (n, B), dtype=torch.int32, device="cuda", generator=gen)      # out-of-range numbers are clamped
    S = torch.randn((2 * n, d), generator=gen, device="cuda")
    for r in range(OS.num_rounds(n)):
        loss = Bn.make_minibatch_loss(Bn.LOSS_LSQ if kind == "lsq" else Bn.LOSS_LOGISTIC, A, t, N, B, noise_std=0.01, seed=5, k=r)
        ws = _aligned(torch, P.dsgd_ceca_workspace_bytes(n, d, loss))
        one, two, inplace = torch.full_like(S, float("nan")), torch.full_like(S, float("nan")), S.clone()
        P.dsgd_ceca_step(S, one, n, d, loss, idx, lr, r, port, workspace=ws)
        assert (P.ceca_last_form() == Bn.FORM_STEP_SINGLE) == (B <= (64 if d % 4 else 32) and d <= (256 if d % 4 else 1024) and n * B * d <= 2 << 20)
        P.dsgd_ceca_step(inplace, inplace, n, d, loss, idx, lr, r, port, workspace=ws)
        P.ceca_set_option(Bn.OPT_HALF_STEP_RUN, 0)
        P.dsgd_ceca_step(S, two, n, d, loss, idx, lr, r, port, workspace=ws)
        P.ceca_reset_options()
        assert P.ceca_last_form() in (Bn.FORM_STEP_ONE_PASS, Bn.FORM_STEP_TWO_PASS)
        assert bool(torch.isfinite(two).all())
        assert torch.equal(one, two) and torch.equal(inplace, two), r


@pytest.mark.parametrize("missing,iters", [(1, 2), (1, 40), (3, 9), (1 << 20, 9)])
@pytest.mark.parametrize("n,port,d,B,noise", [(5, 2, 1000, 8, 0.0), (6, 1, 250, 64, 0.01), (40, 1, 24, 50, 0.01), (6, 2, 10000, 32, 0.0), (2, 2, 9000, 64, 0.01),
                                              (12, 2, 4096, 16, 0.0), (9, 2, 255, 20, 0.01), (12, 1, 63, 9, 0.0), (3, 2, 1000, 40, 0.0), (4, 1, 1999, 4, 0.01)])
def test_window_whose_workgroups_are_not_all_there(env, n, port, d, B, noise, missing, iters):
    """Workgroups that never reach the device: the others give the window up (none of them stores anything) and one does
    it alone -- the bits of the whole window, in place and out of place; the next call runs normally."""
    torch, P = env
    from paper_2306_00256_amd import binding as Bn
    N, lr, tau = max(B // 2, 3), 0.02 / (d * B) ** 0.5, OS.num_rounds(n)
    gen = torch.Generator(device="cuda").manual_seed(n * d + B)
    A = torch.randn((n, N, d), generator=gen, device="cuda")
    t = torch.randn((n, N), generator=gen, device="cuda").sign()
    idx = torch.randint(-1, N + 1, (iters, n, B), dtype=torch.int32, device="cuda", generator=gen)
    S = torch.randn((2 * n, d), generator=gen, device="cuda")
    loss = Bn.make_minibatch_loss(Bn.LOSS_LOGISTIC if port == 2 else Bn.LOSS_LSQ, A, t, N, B, noise_std=noise, seed=5, k=3)
    ws = _aligned(torch, P.dsgd_ceca_run_workspace_bytes(n, d, loss))
    ref, got, inplace = torch.empty_like(S), torch.full_like(S, float("nan")), S.clone()
    P.ceca_set_option(Bn.OPT_HALF_STEP_RUN, 0)
    P.dsgd_ceca_run(S, ref, n, d, loss, idx, lr, 1 % tau, iters, port, workspace=ws)
    P.ceca_reset_options()
    P.ceca_set_option(Bn.OPT_WINDOW_MISSING, missing)
    for out in (got, inplace):
        P.dsgd_ceca_run(inplace if out is inplace else S, out, n, d, loss, idx, lr, 1 % tau, iters, port, workspace=ws)
        assert P.ceca_last_form() == Bn.FORM_RUN_WINDOW
        torch.cuda.synchronize()
    P.ceca_reset_options()
    assert bool(torch.isfinite(ref).all()) and torch.equal(got, ref) and torch.equal(inplace, ref)
    P.dsgd_ceca_run(S, got.fill_(float("nan")), n, d, loss, idx, lr, 1 % tau, iters, port, workspace=ws)
    assert torch.equal(got, ref)


def test_workspace_without_room_for_the_roll(env):
    """The size that dsgd_ceca_run took before the window kept a roll is still taken; where the window's words fill it, with
    another form and the same bits."""
    torch, P = env
    from paper_2306_00256_amd import binding as Bn
    for n, d, B, fits in [(2, 18240, 4, False), (6, 10000, 32, True)]:
        N, iters = 5, 4
        A, t, idx, Ad, td, idxd, code = _problem(torch, Bn, "logistic", n, N, d, B, iters, seed=n)
        loss = Bn.make_minibatch_loss(code, Ad, td, N, B)
        ws = _aligned(torch, P.dsgd_ceca_run_workspace_bytes(n, d, loss))
        S = make_state(torch, 0.05 * WL.initial_state(n, d, seed=3))
        outs = []
        for w, form in ((ws, True), (ws[:-256], fits)):
            outs.append(torch.full_like(S, float("nan")))
            P.dsgd_ceca_run(S, outs[-1], n, d, loss, idxd, 0.003, 0, iters, 2, workspace=w)
            assert (P.ceca_last_form() == Bn.FORM_RUN_WINDOW) == form
        assert torch.equal(*outs)
        with pytest.raises(P.CecaError):
            P.dsgd_ceca_run(S, outs[0], n, d, loss, idxd, 0.003, 0, iters, 2, workspace=ws[:-257])


def test_window_on_streams_of_every_kind(env):
    """The one-kernel window on the null stream, the per-thread default stream and streams restricted to 32 compute
    units, where a window of 16 workgroups of 256 threads (an eighth of 32 x 4) still runs as one kernel and 17 do not."""
    import ctypes
    from types import SimpleNamespace
    torch, P = env
    from paper_2306_00256_amd import binding as Bn
    hip = ctypes.CDLL("libamdhip64.so.7")
    masked = ctypes.c_void_p()
    bits = (ctypes.c_uint32 * 8)(0xFFFFFFFF)
    assert hip.hipExtStreamCreateWithCUMask(ctypes.byref(masked), ctypes.c_uint32(8), bits) == 0
    try:
        for n in (16, 17):
            d, B, N, iters, lr = 1000, 8, 20, 9, 0.001
            A, t, idx, Ad, td, idxd, code = _problem(torch, Bn, "lsq", n, N, d, B, iters, seed=n)
            loss = Bn.make_minibatch_loss(code, Ad, td, N, B, noise_std=0.1, seed=2)
            ws = _aligned(torch, P.dsgd_ceca_run_workspace_bytes(n, d, loss))
            S = make_state(torch, 0.05 * WL.initial_state(n, d, seed=3))
            ref = torch.full_like(S, float("nan"))
            P.ceca_set_option(Bn.OPT_HALF_STEP_RUN, 0)
            P.dsgd_ceca_run(S, ref, n, d, loss, idxd, lr, 0, iters, 2, workspace=ws)
            P.ceca_reset_options()
            for handle, window in ((0, True), (2, True), (masked.value, n == 16)):          # 2: hipStreamPerThread
                out = torch.full_like(S, float("nan"))
                torch.cuda.synchronize()
                P.dsgd_ceca_run(S, out, n, d, loss, idxd, lr, 0, iters, 2, workspace=ws, stream=SimpleNamespace(cuda_stream=handle))
                torch.cuda.synchronize()
                assert (P.ceca_last_form() == Bn.FORM_RUN_WINDOW) == window, (n, handle)
                assert torch.equal(out, ref), (n, handle)
    finally:
        assert hip.hipStreamDestroy(masked) == 0
