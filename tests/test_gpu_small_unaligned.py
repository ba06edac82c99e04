"""The register-tile kernels on both sides of the line between single columns and 16-byte groups, 2^20 elements (fused iterations 2^19)
on rows off 16-byte boundaries, and the streaming kernel on both sides of its own, 2^17: the bits of aligned rows.  The consensus
observables (2^19): fp64 sums in another order, 1e-12."""
import pytest

from test_gpu_large_layouts import _calls
from test_gpu_layouts import _compare, env  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [3, 64, 65, 97, 531, 2200, 3073])
@pytest.mark.parametrize("over", [-1, 0])
@pytest.mark.parametrize("extra,offset", [(1, 0), (0, 3)])
def test_both_sides_of_the_line(env, n, over, extra, offset):  # noqa: F811
    torch, P = env
    d = -(-(1 << 20) // n) + over
    extra = extra or -d % 4                                     # (0, 3): the base alone is off a boundary
    for halves, call in _calls(torch, P, n, d).values():
        _compare(torch, call, halves * n, d, extra, offset, False)


@pytest.mark.parametrize("n", [3, 64, 130, 531, 2200])
@pytest.mark.parametrize("over", [-1, 0])
def test_fused_iterations_on_both_sides_of_the_line(env, n, over):  # noqa: F811
    torch, P = env
    from paper_2306_00256_amd import binding as B
    d = -(-(1 << 19) // n) + over
    c = torch.randn((n, d + 1 + (d + 1) % 2), device="cuda")[:, :d]

    def fused(src, dst, ld):
        P.dsgd_ceca_steps(src, dst, n, d, B.make_quad_center_loss(c, 0.3, 5), 0.1, 0, 9, 2, ld=ld)

    _compare(torch, fused, 2 * n, d, 1, 3, False)


@pytest.mark.parametrize("in_place", [False, True])
@pytest.mark.parametrize("n,port", [(2, 1), (3, 2), (130, 1), (417, 2), (2500, 2)])
@pytest.mark.parametrize("over", [0, 1])
def test_single_rounds_and_steps_on_both_sides_of_the_line(env, n, port, over, in_place):  # noqa: F811
    torch, P = env
    from paper_2306_00256_amd import binding as B
    d = (1 << 17) // n + over
    c = torch.randn((n, d + 1 + (d + 1) % 2), device="cuda")[:, :d]
    last = P.ceca_tau(n) - 1
    assert P.ceca_describe_step_launch(n, d, d + 1 + d % 2, last, port, 0, in_place)["vec"] == (4 if over else 1)
    cycles = in_place and port == 2 and d % 4 != 0 and not over  # walks of odd rows that share lines
    assert P.ceca_describe_step_launch(n, d, -(-d // 4) * 4, last, port, 0, in_place)["vec"] == (1 if cycles else 4)

    for r in (0, last):
        _compare(torch, lambda src, dst, ld: P.ceca_gossip_round(src, dst, n, d, r, port, ld=ld), 2 * n, d, 1 + d % 2, 3, in_place)
        _compare(torch, lambda src, dst, ld: P.dsgd_ceca_step(src, dst, n, d, B.make_quad_center_loss(c, 0.3, 5, r), None, 0.1, r, port, ld=ld), 2 * n, d, 1 + d % 2, 3, in_place)
        _compare(torch, lambda src, dst, ld: P.dsgd_ceca_step(src, dst, n, d, B.make_gradient_loss(c), None, 0.1, r, port, ld=ld), 2 * n, d, 1 + d % 2, 3, in_place)


@pytest.mark.parametrize("n", [5, 64, 108, 130, 531, 1532, 2900, 3090])
@pytest.mark.parametrize("over", [0, 1])
@pytest.mark.parametrize("extra,offset", [(0, 1), (1, 0)])
def test_consensus_on_both_sides_of_the_line(env, n, over, extra, offset):  # noqa: F811
    torch, P = env
    d = (1 << 19) // n + over
    ld = d + extra
    flat = torch.full((offset + n * ld + 64,), 1e30, device="cuda")
    X = flat[offset:offset + n * ld].view(n, ld)
    X[:, :d] = torch.randn((n, d), device="cuda") + 2.0
    ws = torch.empty(P.consensus_error_workspace_bytes(n, d), dtype=torch.uint8, device="cuda")
    x = X[:, :d].double()
    m = x.mean(dim=0)
    dev = ((x - m) ** 2).sum(dim=1)
    want = torch.stack([dev.sum(), dev.sqrt().sum(), dev.sqrt().max(), (m * m).sum().sqrt()])
    for noalloc in (False, True):
        out = torch.zeros(5, dtype=torch.float64, device="cuda")
        xbar = torch.full((d + 8,), 7.0, device="cuda")
        if noalloc:
            P.consensus_error_noalloc(X, n, d, out, xbar=xbar, ld=ld)
        else:
            P.consensus_error(X, n, d, out, xbar=xbar, workspace=ws, ld=ld)
        assert torch.allclose(out[:4], want, rtol=1e-12, atol=0) and float(out[4]) == n
        assert torch.allclose(xbar[:d].double(), m, rtol=2e-7, atol=1e-7) and bool((xbar[d:] == 7.0).all())
