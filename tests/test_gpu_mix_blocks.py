"""GPU parity of mixing rounds with four or more peers per round in their form with blocks of consecutive rows: at the edges
of its tiles, with peers of any order, distance and number, against an fp64 evaluation and against the general form, which
has to agree bit for bit."""
import numpy as np
import pytest

import workloads as WL

pytestmark = pytest.mark.gpu

# a few agents, in one row of lanes, and first and last agent counts of every tile of the form, those where the rows per thread change, and counts beside them
NS = [9, 12, 16, 31, 96, 97, 104, 105, 119, 130, 192, 193, 217, 256, 257, 278, 279, 512, 513, 671, 672, 888, 889, 1026, 1142, 1143, 1152, 1153,
      1274, 1275, 1280, 1281, 1784, 1785, 2294, 2295]


@pytest.fixture(scope="module")
def env():
    import torch
    import paper_2306_00256_amd as P
    assert torch.cuda.is_available()
    P.lib()
    return torch, P


def _spec(Bn, shifts, ws):
    m = Bn.Mix()
    m.m, m.w_self = len(shifts), ws
    for j, s in enumerate(shifts):
        m.shift[j], m.w[j] = s, (1.0 - ws) * (j + 1) / (len(shifts) * (len(shifts) + 1) / 2)
    return m


def _sequences(P, Bn, n):
    st = P.ceca_topology_round(Bn.TOPO_STATIC_EXP, n)
    return {
        "static": [st],
        # all peers far; own row, repeated peers and the row behind among them; runs of 1, 2, 4, 8 cut short or out of order
        "mixed": [_spec(Bn, [n // 2, n - 1, 17, n - 9, 3], 0.25), _spec(Bn, [1, 2, 4, 8, 16, 0, 1, n - 8], 0.125), _spec(Bn, [1], 0.5),
                  _spec(Bn, [], 1.0), _spec(Bn, [1, 2, 5, n - 1], 0.5), _spec(Bn, [2, 1, 4, 8], 0.25), _spec(Bn, [1, 2, 4], 0.25), st],
    }


def _oracle(x, seq, rounds):
    for t in range(rounds):
        s = seq[t % len(seq)]
        if s.m:
            x = np.float64(s.w_self) * x + sum(np.float64(s.w[j]) * np.roll(x, s.shift[j], axis=0) for j in range(s.m))
    return x


@pytest.mark.parametrize("n,kind", [(n, kind) for n in NS for kind in ("static", "mixed") if n > 16 or kind == "static"])
def test_blocks(env, n, kind):
    torch, P = env
    from paper_2306_00256_amd import binding as Bn
    d, ld = [(131, 133), (68, 128), (5, 5), (4, 8)][n % 4]
    seq = _sequences(P, Bn, n)[kind]
    rounds = len(seq) + 2
    x0 = WL.initial_state(n, d, seed=n)
    X = torch.full((n, ld), 7.0, dtype=torch.float32, device="cuda")
    X[:, :d] = torch.from_numpy(x0).cuda()
    Y = torch.full_like(X, 7.0)
    print(n, d, ld, kind, flush=True)
    P.ceca_mix_rounds(X, Y, n, d, seq, rounds)
    assert torch.all(Y[:, d:] == 7.0)
    # every round is a mean of fp32 values with weights of sum 1: m + 1 roundings of at most half an ulp of the largest value
    want = _oracle(x0.astype(np.float64), seq, rounds)
    bound = sum(seq[t % len(seq)].m + 1 for t in range(rounds)) * 2.0 ** -24 * np.abs(x0).max()
    assert np.abs(Y[:, :d].cpu().numpy() - want).max() <= bound
    Z = torch.full_like(X, 7.0)
    try:                                                      # a tile shape that has no such form
        P.ceca_set_option(Bn.OPT_TILE_THREADS, 1024 if n <= 1280 else 256)
        P.ceca_set_option(Bn.OPT_ROWS, 13 if n <= 1280 else 16)
        P.ceca_mix_rounds(X, Z, n, d, seq, rounds)
    finally:
        P.ceca_set_option(Bn.OPT_TILE_THREADS, 0)
        P.ceca_set_option(Bn.OPT_ROWS, 0)
    assert torch.equal(Y, Z)
    P.ceca_mix_rounds(X, X, n, d, seq, rounds)                # in place
    assert torch.equal(X, Y)


@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
def test_one_bad_value_spreads_along_the_peers_alone(env, bad):
    torch, P = env
    from paper_2306_00256_amd import binding as Bn
    n, d = 1026, 64
    st = P.ceca_topology_round(Bn.TOPO_STATIC_EXP, n)
    X = torch.from_numpy(WL.initial_state(n, d, seed=3)).cuda()
    X[n - 1, 5] = bad
    Y = torch.empty_like(X)
    P.ceca_mix_rounds(X, Y, n, d, [st], 1)
    hit = {(n - 1, 5)} | {((n - 1 + st.shift[j]) % n, 5) for j in range(st.m)}
    assert {tuple(v) for v in (~torch.isfinite(Y)).nonzero().tolist()} == hit
