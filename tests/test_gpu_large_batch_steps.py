"""Which gradient kernel a single step takes: batches over 32 on rows of up to 1024 columns (two passes on few agents, one on many) and
small batches on rows of odd length (the chunked kernel), at the edges of the rules, with the bits of the other kernels and of a run."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,d,B,two", [(2, 4, 64, True), (8, 256, 49, True), (95, 252, 64, True), (96, 252, 64, False), (8, 256, 48, False), (4, 260, 33, True), (127, 400, 48, True),
                                       (128, 400, 48, False), (128, 400, 49, True), (255, 260, 64, True), (256, 260, 64, False), (4, 1021, 40, True), (9, 387, 64, True),
                                       (130, 387, 40, False), (4, 1024, 32, False), (9, 253, 64, False)])
def test_steps_with_large_batches(n, d, B, two):
    import torch
    import paper_2306_00256_amd as P
    from paper_2306_00256_amd import binding as Bn
    assert torch.cuda.is_available()
    P.lib()
    gen = torch.Generator(device="cuda").manual_seed(n * d + B)
    N, iters, lr, tau = B // 2 + 3, 3, 0.02 / (d * B) ** 0.5, P.ceca_tau(n)
    A = torch.randn((n, N, d), generator=gen, device="cuda")
    t = torch.randn((n, N), generator=gen, device="cuda").sign()
    idx = torch.randint(-1, N + 1, (iters, n, B), dtype=torch.int32, device="cuda", generator=gen)
    S = 0.1 * torch.randn((2 * n, d), generator=gen, device="cuda")

    def loss(k):
        return Bn.make_minibatch_loss(Bn.LOSS_LOGISTIC, A, t, N, B, noise_std=0.02, seed=4, k=k)

    ws = torch.empty(P.dsgd_ceca_run_workspace_bytes(n, d, loss(0)), dtype=torch.uint8, device="cuda")
    got, want = S.clone(), S.clone()
    for k in range(iters):
        P.dsgd_ceca_step(got, got, n, d, loss(k), idx[k], lr, k % tau, 2, workspace=ws)
        assert P.ceca_last_form() == (Bn.FORM_STEP_TWO_PASS if two else Bn.FORM_STEP_ONE_PASS)
        P.ceca_set_option(Bn.OPT_ONEPASS, 0)
        P.dsgd_ceca_step(want, want, n, d, loss(k), idx[k], lr, k % tau, 2, workspace=ws)
        P.ceca_reset_options()
        assert P.ceca_last_form() == Bn.FORM_STEP_TWO_PASS
        assert torch.equal(got, want), k
    for half in (1, 0):
        P.ceca_set_option(Bn.OPT_HALF_STEP_RUN, half)
        run = torch.empty_like(S)
        P.dsgd_ceca_run(S, run, n, d, loss(0), idx, lr, 0, iters, 2, workspace=ws)
        P.ceca_reset_options()
        assert torch.equal(run, got), half


@pytest.mark.parametrize("n,d,B", [(4, 257, 8), (9, 1021, 1), (40, 262, 5), (33, 8193, 4), (64, 9001, 1), (95, 16383, 3), (33, 8190, 4), (40, 258, 9)])
def test_small_batches_on_odd_lengths(n, d, B):
    import torch
    import paper_2306_00256_amd as P
    from paper_2306_00256_amd import binding as Bn
    assert torch.cuda.is_available()
    P.lib()
    gen = torch.Generator(device="cuda").manual_seed(n * d + B)
    N, lr = B + 3, 0.02 / (d * B) ** 0.5
    A = torch.randn((n, N, d), generator=gen, device="cuda")
    t = torch.randn((n, N), generator=gen, device="cuda").sign()
    idx = torch.randint(-1, N + 1, (n, B), dtype=torch.int32, device="cuda", generator=gen)
    S = 0.1 * torch.randn((2 * n, d), generator=gen, device="cuda")
    loss = Bn.make_minibatch_loss(Bn.LOSS_LOGISTIC, A, t, N, B, noise_std=0.02, seed=4, k=3)
    ws = torch.empty(P.dsgd_ceca_workspace_bytes(n, d, loss), dtype=torch.uint8, device="cuda")
    got, want = torch.empty_like(S), torch.empty_like(S)
    P.dsgd_ceca_step(S, got, n, d, loss, idx, lr, 1, 2, workspace=ws)
    assert P.ceca_last_form() == Bn.FORM_STEP_ONE_PASS
    P.ceca_set_option(Bn.OPT_CHUNKED_GRADIENT, 0)              # the looping kernel
    P.dsgd_ceca_step(S, want, n, d, loss, idx, lr, 1, 2, workspace=ws)
    P.ceca_reset_options()
    assert torch.equal(got, want) and bool(torch.isfinite(got).all())
