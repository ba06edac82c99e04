"""Large problems on rows of any base, pitch and length: at least 1024 tiles, no multiple of 128, so that the grid is rounded up to whole
runs per XCD, rows go through the caches and the last group is short, all at once; and rows of one to three columns on many
agents, which tiles of single columns take.  The bits of 16-byte aligned rows; nothing beyond the rows is written."""
import pytest

from test_gpu_layouts import _compare, _guarded, env  # noqa: F401

pytestmark = pytest.mark.gpu


def _calls(torch, P, n, d):
    import workloads as WL
    from paper_2306_00256_amd import binding as B
    tau = P.ceca_tau(n)
    tables = [torch.from_numpy(t[None].copy()).cuda() for t in WL.graph_table(n, WL.edges_of("ring", n, n))]

    def mix(kind):
        specs = [P.ceca_topology_round(kind, n, k) for k in range(tau if kind == B.TOPO_ONE_PEER_EXP else 1)]
        return lambda src, dst, ld: P.ceca_mix_rounds(src, dst, n, d, specs, 3, ld=ld)

    return {"rounds": (2, lambda src, dst, ld: P.ceca_gossip_rounds(src, dst, n, d, tau + 1, 2, ld=ld)),
            "average": (1, lambda src, dst, ld: P.ceca_average(src, dst, n, d, 2, ld=ld)),
            "ring": (1, mix(B.TOPO_RING)), "static": (1, mix(B.TOPO_STATIC_EXP)), "one-peer": (1, mix(B.TOPO_ONE_PEER_EXP)),
            "graph": (1, lambda src, dst, ld: P.ceca_graph_rounds(src, dst, n, d, *tables, 3, ld=ld))}


@pytest.mark.parametrize("in_place", [False, True])
@pytest.mark.parametrize("n,d,extra,offset", [(3, 1050003, 0, 1), (20, 560001, 3, 2), (130, 70001, 0, 1), (600, 40010, 1, 0), (1026, 70003, 0, 3), (2200, 16423, 0, 1)])
def test_tiles_in_runs_with_a_short_last_group(env, n, d, extra, offset, in_place):  # noqa: F811
    torch, P = env
    for halves, call in _calls(torch, P, n, d).values():
        _compare(torch, call, halves * n, d, extra, offset, in_place)


@pytest.mark.parametrize("n,port,d,extra,offset", [(3, 2, 1050003, 0, 1), (20, 1, 560001, 3, 2), (130, 2, 70001, 0, 1), (600, 2, 40010, 1, 0), (1026, 1, 20003, 0, 3)])
def test_fused_iterations_in_runs(env, n, port, d, extra, offset):  # noqa: F811
    torch, P = env
    from paper_2306_00256_amd import binding as B
    _, codd = _guarded(torch, n, d, d + 1, 1, 9)
    cref = torch.zeros((n, -(-d // 64) * 64), dtype=torch.float32, device="cuda")
    cref[:, :d] = codd[:, :d]

    def fused(src, dst, ld):
        c = codd if ld == d + extra else cref
        P.dsgd_ceca_steps(src, dst, n, d, B.make_quad_center_loss(c, 0.3, 5), 0.1, 0, 9, port, ld=ld)

    _compare(torch, fused, 2 * n, d, extra, offset, False)


@pytest.mark.parametrize("d,extra,offset", [(1, 0, 1), (2, 1, 0), (3, 0, 0)])
@pytest.mark.parametrize("n", [2, 64, 130, 600, 1026, 3000, 4096])
def test_rows_of_one_to_three_columns(env, n, d, extra, offset):  # noqa: F811
    """Against rows of four columns, which 16-byte groups take, with the same first columns."""
    torch, P = env
    from paper_2306_00256_amd import binding as B
    four = _calls(torch, P, n, 4)
    for name, (halves, call) in _calls(torch, P, n, d).items():
        flat, src = _guarded(torch, halves * n, d, d + extra, offset, 7)
        out_flat, dst = _guarded(torch, halves * n, d, d + extra, (offset + 1) % 4, 8)
        wide = torch.zeros((halves * n, 4), device="cuda")
        wide[:, :d] = src[:, :d]
        want = torch.empty_like(wide)
        call(src, dst, d + extra)
        four[name][1](wide, want, 4)
        assert torch.equal(dst[:, :d], want[:, :d]), name
        assert bool((dst[:, d:] == 12345.0).all()), name
    c = torch.randn((n, 4), device="cuda")
    short = c[:, :d].contiguous()
    x, y = torch.randn((2 * n, 4), device="cuda"), torch.empty((2 * n, 4), device="cuda")
    xs = x[:, :d].contiguous()
    ys = torch.empty_like(xs)
    for std in (0.0, 0.3):
        P.dsgd_ceca_steps(x, y, n, 4, B.make_quad_center_loss(c, std, 5), 0.1, 0, 15, 2)
        P.dsgd_ceca_steps(xs, ys, n, d, B.make_quad_center_loss(short, std, 5), 0.1, 0, 15, 2)
        assert torch.equal(ys, y[:, :d]), std
