"""Rows of any base, pitch and length: the kernels load and store 16-byte groups whatever their alignment, and the last
group of a row may be short.  Every call on an unaligned layout has the bits of the same call on an aligned one (columns
are independent, and every column's operations are the same wherever it lies) and leaves everything beyond the rows as
it was; the consensus observables (fp64 sums in another order) agree to 1e-12."""
import numpy as np
import pytest


pytestmark = pytest.mark.gpu

PAD = 12345.0
# (columns, floats between rows beyond them, floats the base is off a 16-byte boundary); 4 is the shortest vector row
LAYOUTS = [(4, 0, 0), (5, 0, 1), (6, 1, 2), (7, 2, 3), (131, 0, 0), (1026, 3, 1), (1029, 4, 0), (1031, 1, 2), (4099, 0, 3)]


@pytest.fixture(scope="module")
def env():
    torch = pytest.importorskip("torch")
    import paper_2306_00256_amd as P
    assert torch.cuda.is_available()
    P.lib()
    return torch, P


def _guarded(torch, rows, d, ld, offset, seed):
    """rows x ld floats at an offset, PAD in and around the padding; the flat buffer and the view of the rows."""
    flat = torch.full((offset + rows * ld + 64,), PAD, dtype=torch.float32, device="cuda")
    view = flat[offset:offset + rows * ld].view(rows, ld)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    view[:, :d] = torch.empty((rows, d), device="cuda").normal_(generator=gen)
    return flat, view


def _compare(torch, call, rows, d, extra, offset, in_place):
    """`call(src, dst, ld)` on the layout (d + extra, offset) against 16-byte aligned rows."""
    ld, ref_ld = d + extra, -(-d // 64) * 64
    flat, src = _guarded(torch, rows, d, ld, offset, 7)
    ref_src = torch.zeros((rows, ref_ld), dtype=torch.float32, device="cuda")
    ref_src[:, :d] = src[:, :d]
    ref_dst = torch.zeros_like(ref_src)
    out_flat, dst = (flat, src) if in_place else _guarded(torch, rows, d, ld, (offset + 1) % 4, 8)
    call(ref_src, ref_dst, ref_ld)
    call(src, dst, ld)
    torch.cuda.synchronize()
    assert torch.equal(dst[:, :d], ref_dst[:, :d])
    assert bool((dst[:, d:] == PAD).all()), "padding written"
    start = (dst.data_ptr() - out_flat.data_ptr()) // 4
    assert bool((out_flat[:start] == PAD).all()) and bool((out_flat[start + rows * ld:] == PAD).all()), "written beyond the rows"


@pytest.mark.parametrize("in_place", [False, True])
@pytest.mark.parametrize("d,extra,offset", LAYOUTS)
@pytest.mark.parametrize("n", [3, 64, 130, 600, 1026])
def test_register_tile_kernels(env, n, d, extra, offset, in_place):
    torch, P = env
    import workloads as WL
    from paper_2306_00256_amd import binding as B
    tau = P.ceca_tau(n)

    def rounds(src, dst, ld):
        P.ceca_gossip_rounds(src, dst, n, d, tau + 1, 2, ld=ld)

    def average(src, dst, ld):
        P.ceca_average(src, dst, n, d, 2, ld=ld)

    def mix(kind):
        specs = [P.ceca_topology_round(kind, n, k) for k in range(tau)]
        return lambda src, dst, ld: P.ceca_mix_rounds(src, dst, n, d, specs[:1] if kind != B.TOPO_ONE_PEER_EXP else specs, tau, ld=ld)

    tables = [torch.from_numpy(t[None].copy()).cuda() for t in WL.graph_table(n, WL.edges_of("ring", n, n))]

    def graph(src, dst, ld):
        P.ceca_graph_rounds(src, dst, n, d, *tables, tau, ld=ld)

    _compare(torch, rounds, 2 * n, d, extra, offset, in_place)
    for call in (average, mix(B.TOPO_RING), mix(B.TOPO_STATIC_EXP), mix(B.TOPO_ONE_PEER_EXP), graph):
        _compare(torch, call, n, d, extra, offset, in_place)


@pytest.mark.parametrize("in_place", [False, True])
@pytest.mark.parametrize("d,extra,offset", LAYOUTS + [(1, 0, 1), (3, 1, 0)])
@pytest.mark.parametrize("n,port", [(3, 2), (64, 1), (130, 2)])
def test_steps_with_noise(env, n, port, d, extra, offset, in_place):
    """Fused and single iterations with the elementwise losses: noise is keyed by the column, so a short group has to keep
    its place."""
    torch, P = env
    from paper_2306_00256_amd import binding as B
    cref = torch.zeros((n, -(-d // 4) * 4), dtype=torch.float32, device="cuda")
    _, codd = _guarded(torch, n, d, d + 1, 1, 9)
    cref[:, :d] = codd[:, :d]

    def pick(ld):
        return codd if ld == d + extra and (ld % 4 or offset) else cref

    def fused(src, dst, ld):
        P.dsgd_ceca_steps(src, dst, n, d, B.make_quad_center_loss(pick(ld), 0.3, 5), 0.1, 0, 9, port, ld=ld)

    def single(src, dst, ld):
        P.dsgd_ceca_step(src, dst, n, d, B.make_quad_center_loss(pick(ld), 0.3, 5, 4), None, 0.1, P.ceca_tau(n) - 1, port, ld=ld)

    def gradient(src, dst, ld):
        P.dsgd_ceca_step(src, dst, n, d, B.make_gradient_loss(pick(ld)), None, 0.1, 0, port, ld=ld)

    def gossip(src, dst, ld):
        P.ceca_gossip_round(src, dst, n, d, 1, port, ld=ld)

    for call in (fused, single, gradient, gossip):
        _compare(torch, call, 2 * n, d, extra, offset, in_place)


@pytest.mark.parametrize("d,extra,offset", LAYOUTS + [(1, 0, 1), (3, 1, 0), (70001, 0, 1)])
@pytest.mark.parametrize("n", [2, 31, 100, 113, 300, 1026])
def test_consensus(env, n, d, extra, offset):
    torch, P = env
    ld = d + extra
    _, X = _guarded(torch, n, d, ld, offset, 3)
    X[:, :d] += 2.0
    ws = torch.empty(P.consensus_error_workspace_bytes(n, d), dtype=torch.uint8, device="cuda")
    out = torch.zeros(5, dtype=torch.float64, device="cuda")
    xbar = torch.full((d + 8,), PAD, dtype=torch.float32, device="cuda")
    P.consensus_error(X, n, d, out, xbar=xbar, workspace=ws, ld=ld)
    x = X[:, :d].double().cpu().numpy()
    m = x.mean(axis=0)
    dev = np.sqrt(((x - m) ** 2).sum(axis=1))
    want = np.array([(dev ** 2).sum(), dev.sum(), dev.max(), np.sqrt((m ** 2).sum()), n])
    assert np.allclose(out.cpu().numpy(), want, rtol=1e-12, atol=0)
    got = xbar.cpu().numpy()
    assert np.allclose(got[:d], m.astype(np.float32), rtol=2e-7, atol=1e-7) and (got[d:] == PAD).all()


@pytest.mark.parametrize("kind", ["lsq", "logistic"])
@pytest.mark.parametrize("n,d,B", [(3, 5, 3), (6, 63, 64), (6, 65, 9), (4, 66, 64), (40, 67, 17), (5, 255, 33), (6, 257, 8), (7, 1001, 40), (130, 1001, 33),
                                   (5, 1027, 16), (4, 1030, 40), (6, 2051, 9), (130, 2051, 9), (130, 4099, 16), (3, 5000, 40), (130, 9001, 5)])
def test_minibatch_losses(env, kind, n, d, B):
    """Steps and windows (full batches that come again, and random ones), in place and out of place, on rows of the state
    and of the samples at odd bases and pitches: the bits of 16-byte aligned rows."""
    torch, P = env
    from paper_2306_00256_amd import binding as Bn
    gen = torch.Generator(device="cuda").manual_seed(n * d + B)
    N, iters, lr, tau = B, 6, 0.02 / (d * B) ** 0.5, P.ceca_tau(n)
    A = torch.randn((n, N, d), generator=gen, device="cuda")
    t = torch.randn((n, N), generator=gen, device="cuda").sign()
    full = torch.arange(N, dtype=torch.int32, device="cuda").expand(iters, n, -1).contiguous()
    some = torch.randint(-1, N + 1, (iters, n, B), dtype=torch.int32, device="cuda", generator=gen)
    x0 = 0.1 * torch.randn((2 * n, d), generator=gen, device="cuda")

    def rows(shape, extra, offset):
        flat = torch.full((offset + int(np.prod(shape)) * (d + extra) + 64,), float("inf"), device="cuda")
        return flat, flat[offset:offset + int(np.prod(shape)) * (d + extra)].view(*shape, d + extra)

    def outputs(extra, offset, idx):
        _, a = rows((n, N), extra, offset)
        a[..., :d] = A
        loss = Bn.make_minibatch_loss(Bn.LOSS_LSQ if kind == "lsq" else Bn.LOSS_LOGISTIC, a, t, N, B, noise_std=0.02, seed=4, k=2)
        out = []
        for call in ("step", "run"):
            size = P.dsgd_ceca_workspace_bytes if call == "step" else P.dsgd_ceca_run_workspace_bytes
            ws = torch.empty(size(n, d, loss), dtype=torch.uint8, device="cuda")
            for in_place in (False, True):
                src_flat, src = rows((2 * n,), extra, offset)
                src[:, :d] = x0
                flat, dst = (src_flat, src) if in_place else rows((2 * n,), extra, (offset + 1) % 4 if offset else 0)
                for two_kernels in (0, 1):
                    src[:, :d] = x0
                    Bn.ceca_set_option(Bn.OPT_HALF_STEP_RUN, 1 - two_kernels)
                    if call == "step":
                        P.dsgd_ceca_step(src, dst, n, d, loss, idx[0], lr, 1 % tau, 2, workspace=ws)
                    else:
                        P.dsgd_ceca_run(src, dst, n, d, loss, idx, lr, 1 % tau, iters, 2, workspace=ws)
                    out.append(dst[:, :d].clone())
                Bn.ceca_reset_options()
                assert bool(torch.isinf(dst[:, d:]).all()) and bool(torch.isinf(flat[:dst.storage_offset()]).all())
                assert bool(torch.isinf(flat[dst.storage_offset() + 2 * n * (d + extra):]).all())
        return out

    for idx in (full, some):
        ref = outputs(-d % 4, 0, idx)
        assert all(bool(torch.isfinite(r).all()) for r in ref)
        assert all(torch.equal(a, ref[0]) for a in ref[:4]) and all(torch.equal(a, ref[4]) for a in ref[4:])
        for extra, offset in ((0, 0), (1, 3), (3, 1)):
            for got, want in zip(outputs(extra, offset, idx), ref):
                assert torch.equal(got, want), (extra, offset)
