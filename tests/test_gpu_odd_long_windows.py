"""Windows of small batches on a few agents with long rows of odd length: one kernel in chunks of 1024 columns, also where the last
chunk is a single short group, with the bits of two kernels per iteration, and when the window is given up."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["lsq", "logistic"])
@pytest.mark.parametrize("n,d,B,offset,window", [(2, 2049, 1, 1, True), (8, 2265, 2, 0, True), (9, 2277, 1, 3, True), (5, 2895, 3, 0, True), (4, 3073, 7, 2, True), (3, 4097, 6, 0, True),
                                                 (6, 4098, 4, 1, True), (2, 5702, 2, 0, True), (4, 9219, 5, 0, True), (3, 2051, 8, 0, False), (32, 4099, 4, 0, False), (25, 5121, 1, 0, False)])
def test_windows_of_small_batches_on_long_odd_rows(kind, n, d, B, offset, window):
    import torch
    import paper_2306_00256_amd as P
    from paper_2306_00256_amd import binding as Bn
    assert torch.cuda.is_available()
    P.lib()
    gen = torch.Generator(device="cuda").manual_seed(n * d + B)
    N, iters, lr, tau, port = B + 2, 9, 0.02 / (d * B) ** 0.5, P.ceca_tau(n), 2
    A = torch.empty(offset + n * N * d, device="cuda")[offset:].view(n, N, d).normal_(generator=gen)
    t = torch.randn((n, N), generator=gen, device="cuda").sign()
    idx = torch.randint(-1, N + 1, (iters, n, B), dtype=torch.int32, device="cuda", generator=gen)
    S = 0.1 * torch.empty(offset + 2 * n * d, device="cuda").normal_(generator=gen)
    S = S[offset:].view(2 * n, d)
    code = Bn.LOSS_LSQ if kind == "lsq" else Bn.LOSS_LOGISTIC
    loss = Bn.make_minibatch_loss(code, A, t, N, B, noise_std=0.02, seed=4, k=2)
    ws = torch.empty(P.dsgd_ceca_run_workspace_bytes(n, d, loss), dtype=torch.uint8, device="cuda")
    ref = torch.empty_like(S)
    P.ceca_set_option(Bn.OPT_HALF_STEP_RUN, 0)
    P.dsgd_ceca_run(S, ref, n, d, loss, idx, lr, 1 % tau, iters, port, workspace=ws)
    P.ceca_reset_options()
    assert P.ceca_last_form() != Bn.FORM_RUN_WINDOW and bool(torch.isfinite(ref).all())
    for missing in (0, 1) if window else (0,):
        out, inplace = torch.full_like(S, float("nan")), S.clone()
        for src, dst in ((S, out), (inplace, inplace)):
            P.ceca_set_option(Bn.OPT_WINDOW_MISSING, missing)
            P.dsgd_ceca_run(src, dst, n, d, loss, idx, lr, 1 % tau, iters, port, workspace=ws)
            P.ceca_reset_options()
            assert (P.ceca_last_form() == Bn.FORM_RUN_WINDOW) == window
            assert torch.equal(dst, ref), missing
    step = S.clone()
    for k in range(iters):
        one = Bn.make_minibatch_loss(code, A, t, N, B, noise_std=0.02, seed=4, k=2 + k)
        P.dsgd_ceca_step(step, step, n, d, one, idx[k], lr, (1 + k) % tau, port, workspace=ws)
    assert torch.equal(step, ref)
