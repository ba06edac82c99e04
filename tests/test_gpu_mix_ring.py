"""GPU parity of ring gossip in the kernel that exchanges the first and last rows of its blocks alone: at the edges of its tiles,
against an fp64 evaluation and, bit for bit, the general form."""
import numpy as np
import pytest

import workloads as WL

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [64, 65, 80, 81, 130, 256, 257, 272, 273, 288, 289, 448, 449, 512, 513, 960, 961, 1026, 1152, 1153, 1792, 1793, 2048, 2049, 4095, 4096])
def test_ring(n):
    import torch
    import paper_2306_00256_amd as P
    from paper_2306_00256_amd import binding as Bn
    d, ld = [(131, 133), (68, 128), (5, 5), (4, 8)][n % 4]
    seq = []
    for w_self, w_back in [(0.5, 0.375), (0.25, 0.125)]:      # rounds of different weights, and the two peers' weights differ
        m = P.ceca_topology_round(Bn.TOPO_RING, n)
        m.w_self, m.w[0], m.w[1] = w_self, w_back, 1.0 - w_self - w_back
        seq.append(m)
    x0 = WL.initial_state(n, d, seed=n)
    X = torch.full((n, ld), 7.0, dtype=torch.float32, device="cuda")
    X[:, :d] = torch.from_numpy(x0).cuda()
    Y, Z = torch.full_like(X, 7.0), torch.full_like(X, 7.0)
    rounds, k0 = 7, 1
    print(n, d, ld, flush=True)
    P.ceca_mix_rounds(X, Y, n, d, seq, rounds, k0=k0)
    assert torch.all(Y[:, d:] == 7.0)
    want = x0.astype(np.float64)
    for t in range(rounds):
        s = seq[(k0 + t) % 2]
        want = np.float64(s.w_self) * want + np.float64(s.w[0]) * np.roll(want, 1, axis=0) + np.float64(s.w[1]) * np.roll(want, -1, axis=0)
    # every round is a mean of fp32 values with weights of sum 1: three roundings of at most half an ulp of the largest value
    assert np.abs(Y[:, :d].cpu().numpy() - want).max() <= 3 * rounds * 2.0 ** -24 * np.abs(x0).max()
    try:                                                      # a tile shape that is asked for takes the general form
        P.ceca_set_option(Bn.OPT_TILE_THREADS, 1024)
        P.ceca_mix_rounds(X, Z, n, d, seq, rounds, k0=k0)
    finally:
        P.ceca_set_option(Bn.OPT_TILE_THREADS, 0)
    assert torch.equal(Y, Z)
    P.ceca_mix_rounds(X, X, n, d, seq, rounds, k0=k0)         # in place
    assert torch.equal(X, Y)
