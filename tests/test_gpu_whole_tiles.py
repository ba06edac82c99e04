"""Rows of whole 16-byte groups on whole 128-byte lines are streamed by kernel instances of their own: same bits as the same columns at a pitch
that is no whole line (through the caches) and as a length with a short last group (whose first columns they share)."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [32, 1056, 4128])
@pytest.mark.parametrize("n", [3, 4, 9, 17, 33, 64, 100, 130, 258, 520])
def test_whole_lines_against_other_pitches(n, d):
    import torch
    import paper_2306_00256_amd as P
    import workloads as WL
    from paper_2306_00256_amd import binding as B
    assert torch.cuda.is_available()
    P.lib()
    tau = P.ceca_tau(n)
    gen = torch.Generator(device="cuda").manual_seed(n + d)
    x = torch.randn((2 * n, d), generator=gen, device="cuda")
    c = torch.randn((n, d), generator=gen, device="cuda")
    ring = [P.ceca_topology_round(B.TOPO_RING, n)]
    peers = [P.ceca_topology_round(B.TOPO_ONE_PEER_EXP, n, k) for k in range(tau)]
    host = WL.graph_table(n, WL.edges_of("ring", n, 0))
    table = [torch.from_numpy(a).cuda() for a in host]
    nbr, w, ws = [torch.stack([a, a]) for a in table]         # the same round twice: read anew in every round

    def calls(cols, ld):
        """Outputs of every register-tile call on the first `cols` columns at pitch ld."""
        def rows(src, k):
            out = torch.zeros((k, ld), device="cuda")
            out[:, :cols] = src[:k, :cols]
            return out
        S, X, centres = rows(x, 2 * n), rows(x, n), rows(c, n)
        out = []
        for run, src in [
            (lambda a, b: P.ceca_gossip_rounds(a, b, n, cols, tau + 1, 2), S),
            (lambda a, b: P.ceca_average(a, b, n, cols, 2), X),
            (lambda a, b: P.ceca_mix_rounds(a, b, n, cols, ring, 3), X),
            (lambda a, b: P.ceca_mix_rounds(a, b, n, cols, peers, tau), X),
            (lambda a, b: P.dsgd_ceca_steps(a, b, n, cols, B.make_quad_center_loss(centres, 0.01, 3, 0), 0.1, 0, 5, 2), S),
            (lambda a, b: P.dsgd_ceca_steps(a, b, n, cols, B.make_quad_center_loss(centres, 0.0, 3, 0), 0.1, 1, 5, 2), S),
            (lambda a, b: P.ceca_graph_rounds(a, b, n, cols, nbr[:1], w[:1], ws[:1], 3), X),
            (lambda a, b: P.ceca_graph_rounds(a, b, n, cols, nbr, w, ws, 3), X),
        ]:
            for in_place in (False, True):
                a = src.clone()
                b = a if in_place else torch.zeros_like(a)
                run(a, b)
                assert not bool(b[:, cols:].any()), "written beyond the columns"
                out.append(b[:, :cols].clone())
        return out

    whole = calls(d, d)
    for k, (a, b) in enumerate(zip(whole, calls(d, d + 4))):
        assert torch.equal(a, b), k
    for k, (a, b) in enumerate(zip(whole, calls(d - 3, d))):
        assert torch.equal(a[:, :d - 3], b), k
