"""Minibatch losses on rows of up to 256 columns that lie off 16-byte boundaries: one-kernel windows and single-launch steps up to
the agents and batches that single columns hold, runs with the bits of their steps, and the results of aligned rows."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    torch = pytest.importorskip("torch")
    import paper_2306_00256_amd as P
    assert torch.cuda.is_available()
    P.lib()
    return torch, P


def _rows(torch, shape, d, extra, offset):
    count = 1
    for s in shape:
        count *= s
    flat = torch.full((offset + count * (d + extra) + 64,), 7.0, device="cuda")
    return flat[offset:offset + count * (d + extra)].view(*shape, d + extra)


# edges of the columns a wavefront holds, of the batches of the register tiles and of the resident agents
@pytest.mark.parametrize("n,d,B,window", [(166, 4, 60, True), (391, 56, 40, True), (448, 12, 13, True), (512, 64, 64, True), (513, 64, 17, False), (132, 44, 48, True),
                                          (9, 68, 33, True), (128, 256, 33, True), (129, 256, 33, False), (256, 68, 32, True), (12, 8, 56, True), (2, 4, 1, True), (40, 252, 64, True)])
def test_unaligned_short_rows(env, n, d, B, window):
    torch, P = env
    from paper_2306_00256_amd import binding as Bn
    gen = torch.Generator(device="cuda").manual_seed(n * d + B)
    N, iters, lr, tau, port = B + 3, 7, 0.02 / (d * B) ** 0.5, P.ceca_tau(n), 2
    A = torch.randn((n, N, d), generator=gen, device="cuda")
    t = torch.randn((n, N), generator=gen, device="cuda").sign()
    idx = torch.randint(-1, N + 1, (iters, n, B), dtype=torch.int32, device="cuda", generator=gen)
    x0 = 0.1 * torch.randn((2 * n, d), generator=gen, device="cuda")
    ref = None
    # (extra columns, offsets of S_in, S_out and A); the first is aligned, in the last two only one of S_in and S_out is
    for extra, off_in, off_out, off_a in ((-d % 4, 0, 0, 0), (1, 0, 0, 0), (0, 1, 3, 0), (0, 0, 0, 2), (0, 0, 1, 0), (0, 2, 0, 0)):
        a = _rows(torch, (n, N), d, extra, off_a)
        a[..., :d] = A
        loss = Bn.make_minibatch_loss(Bn.LOSS_LOGISTIC, a, t, N, B, noise_std=0.02, seed=4, k=2)
        src, dst, want = _rows(torch, (2 * n,), d, extra, off_in), _rows(torch, (2 * n,), d, extra, off_out), _rows(torch, (2 * n,), d, extra, off_out)
        src[:, :d] = x0
        ws = torch.empty(P.dsgd_ceca_run_workspace_bytes(n, d, loss), dtype=torch.uint8, device="cuda")
        P.dsgd_ceca_run(src, dst, n, d, loss, idx, lr, 1 % tau, iters, port, workspace=ws)
        aligned, mixed = extra == 0 and not (off_in or off_out or off_a), (off_in == 0) != (off_out == 0) and not (d > 64 and B <= 32)
        if not aligned:
            assert (P.ceca_last_form() == Bn.FORM_RUN_WINDOW) == (window and not mixed), (extra, off_in, off_out, off_a)
        for k in range(iters):
            one = Bn.make_minibatch_loss(Bn.LOSS_LOGISTIC, a, t, N, B, noise_std=0.02, seed=4, k=2 + k)
            P.dsgd_ceca_step(src if k == 0 else want, want, n, d, one, idx[k], lr, (1 + k) % tau, port, workspace=ws)
            if k == 0 and not aligned and (off_in or extra or off_a) and n * B * d <= 2 << 20:
                assert P.ceca_last_form() == Bn.FORM_STEP_SINGLE
        assert torch.equal(dst[:, :d], want[:, :d]), (extra, off_in, off_out, off_a)
        assert bool((dst[:, d:] == 7.0).all()) and bool(torch.isfinite(dst).all())
        ref = dst[:, :d].clone() if ref is None else ref
        # the same sums of up to 256 columns and 64 samples in another order: a few units in the last place of numbers below 1
        assert float((dst[:, :d] - ref).abs().max()) <= 2e-6
