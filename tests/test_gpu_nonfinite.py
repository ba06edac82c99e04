"""An infinite feature in a sampled row of the logistic loss: the margin of that sample is infinite, its coefficient finite, so
only the feature's own column of the message is lost.  On rows of a length that is no multiple of four the kernels read the row's
last four columns for a short last group, and every column of the row has to keep this, in every form of the calls."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def env():
    torch = pytest.importorskip("torch")
    import paper_2306_00256_amd as P
    assert torch.cuda.is_available()
    P.lib()
    return torch, P


def _oracle_step(schedule, A, t, idx, S, n, lr):
    """One step in fp64; columns that an infinite feature reached are not finite."""
    rd, peer = schedule
    z = S[n:] if rd.exchange_y else S[:n]
    with np.errstate(all="ignore"):
        v = np.empty_like(z)
        for i in range(n):
            a, lab = A[i][idx[i]], t[i][idx[i]]
            m = (a * z[i]).sum(axis=1)
            coef = -lab / (1.0 + np.exp(lab * m)) / len(idx[i])
            v[i] = z[i] - lr * (coef[:, None] * a).sum(axis=0)
        dz = v - z
        x, y = S[:n] + dz, S[n:] + dz
        a_, b_ = rd.a_num / rd.a_den, rd.b_num / rd.b_den
        return np.concatenate([a_ * x + (1 - a_) * v[peer], b_ * y + (1 - b_) * v[peer]])


# odd lengths over 256 columns in every form: one pass with 256 and 1024 threads, chunks of the batch, two passes; one-kernel
# windows of one workgroup and of several per agent, one and two kernels per iteration
@pytest.mark.parametrize("n,d,B,form", [
    (12, 257, 8, "WINDOW"), (12, 258, 32, "WINDOW"), (12, 1027, 16, "WINDOW"), (11, 1031, 9, "WINDOW"), (4, 1030, 40, "WINDOW"), (4, 2047, 20, "WINDOW"),
    (6, 2051, 9, "TWO_PASS"), (12, 8195, 20, "TWO_PASS"), (40, 4094, 16, "HALF_STEPS"), (34, 9001, 4, "HALF_STEPS"), (34, 5002, 8, "HALF_STEPS"),
    (130, 1001, 33, "HALF_STEPS"), (130, 4098, 20, "HALF_STEPS"), (100, 9003, 20, "HALF_STEPS"), (400, 257, 20, "HALF_STEPS")])
def test_infinite_feature_is_lost_alone(env, n, d, B, form):
    torch, P = env
    from paper_2306_00256_amd import binding as Bn
    rng = np.random.default_rng(n + d)
    N, iters, lr, port, tau = B + 1, 3, 0.05, 2, P.ceca_tau(n)
    A = rng.standard_normal((n, N, d)).astype(np.float32) * 0.3
    t = np.where(rng.standard_normal((n, N)) > 0, 1.0, -1.0).astype(np.float32)
    first = [0, 1, 2, 3, 4, d // 2, d - 8, d - 7, d - 6, d - 5, d - 4, d - 3, d - 2, d - 1]
    bad = np.array([first[(i * 5 + 3 * n) % len(first)] for i in range(n)])
    idx = rng.integers(0, N - 1, (iters, n, B)).astype(np.int32)
    idx[-1, :, B // 2] = N - 1                                   # the last sample is taken in the last iteration alone
    S0 = (0.1 * rng.standard_normal((2 * n, d))).astype(np.float32)
    td, idxd, S = torch.from_numpy(t).cuda(), torch.from_numpy(idx).cuda(), torch.from_numpy(S0).cuda()

    for turn in range(3):
        A[np.arange(n), N - 1] = 0.3
        A[np.arange(n), N - 1, bad] = np.inf
        Ad = torch.from_numpy(A).cuda()
        loss = Bn.make_minibatch_loss(Bn.LOSS_LOGISTIC, Ad, td, N, B)
        ws = torch.empty(max(P.dsgd_ceca_run_workspace_bytes(n, d, loss), P.dsgd_ceca_workspace_bytes(n, d, loss)), dtype=torch.uint8, device="cuda")
        before = torch.empty_like(S)                             # the state that the last iteration starts from
        P.dsgd_ceca_run(S, before, n, d, loss, idxd, lr, 0, iters - 1, port, workspace=ws)
        assert bool(torch.isfinite(before).all())
        rd, peer = P.ceca_schedule(n, (iters - 1) % tau, port)
        want = _oracle_step((rd, np.array(peer)), A.astype(np.float64), t.astype(np.float64), idx[-1], before.cpu().numpy().astype(np.float64), n, lr)
        lost = np.zeros((n, d), dtype=bool)
        lost[np.arange(n), bad] = True
        lost |= lost[np.array(peer)]
        lost = np.concatenate([lost, lost])

        def check(got, what):
            got = got.cpu().numpy()
            assert np.isfinite(got[~lost]).all(), (what, turn, sorted(set(np.argwhere(~np.isfinite(got) & ~lost)[:, 0].tolist()))[:8])
            # sums of up to 64 products of numbers below 2, and of B such coefficients: far within this
            assert np.abs(got[~lost] - want[~lost]).max() <= 1e-5, what

        for missing in (0, 1) if form == "WINDOW" else (0,):
            out = torch.zeros_like(S)
            P.ceca_set_option(Bn.OPT_WINDOW_MISSING, missing)
            P.dsgd_ceca_run(S, out, n, d, loss, idxd, lr, 0, iters, port, workspace=ws)
            P.ceca_reset_options()
            assert P.ceca_last_form() == getattr(Bn, "FORM_RUN_" + form)
            check(out, ("run", missing))
        for half in (0, 1):
            out = torch.zeros_like(S)
            P.ceca_set_option(Bn.OPT_HALF_STEP_RUN, half)
            P.dsgd_ceca_step(before, out, n, d, loss, idxd[-1], lr, (iters - 1) % tau, port, workspace=ws)
            inplace = before.clone()
            P.dsgd_ceca_step(inplace, inplace, n, d, loss, idxd[-1], lr, (iters - 1) % tau, port, workspace=ws)
            P.ceca_reset_options()
            check(out, ("step", half))
            check(inplace, ("step in place", half))
        out = torch.zeros_like(S)                                # two passes whatever the shape
        P.ceca_set_option(Bn.OPT_ONEPASS, 0)
        P.dsgd_ceca_run(S, out, n, d, loss, idxd, lr, 0, iters, port, workspace=ws)
        P.ceca_reset_options()
        check(out, "two passes")
        bad = np.array([first[(first.index(b) + 5) % len(first)] for b in bad])
