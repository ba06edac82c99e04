"""Measured cases: what a user of the library has it do, through the public entry points, on one GPU.

Every case is one of a few kinds of call (see `draw` for the range of each kind); the listed ones are the
repository's own configurations.  All data is fp32, drawn on the GPU from the case's seed."""
import math

import torch

import paper_2306_00256_amd as P
import workloads as WL
from paper_2306_00256_amd import binding as B

SPEC = WL.SPECS


def _pad(d: int) -> int:
    """Row pitch that keeps rows on 256-byte boundaries, as the benchmark lays its states out."""
    return -(-d // 64) * 64


def listed():
    q, l5, l6, p258, big = (SPEC[k] for k in ("quad31_2p", "lsq5_2p", "logistic6_2p", "paperlsq258_1p", "logistic1023_2p"))
    return [
        # the smallest call: one iteration of a small least-squares problem, called once per iteration by the
        # user's own loop (latency and launches count)
        dict(name="step_lsq6", kind="ministep", loss="lsq", n=6, d=l5.d, ld=l5.d, N=l5.N, B=l5.B, lr=l5.lr, noise=0.0, scale=0.0, port=1, iters=1),
        # a window of iterations of the same problem at five agents, two ports
        dict(name="run_lsq5", kind="run", loss="lsq", n=l5.n, d=l5.d, ld=l5.d, N=l5.N, B=l5.B, lr=l5.lr, noise=0.0, scale=0.0, port=2, iters=200),
        # the paper's own least-squares experiment: many agents, ten unknowns, full noisy gradients, 20
        # iterations at one step size
        dict(name="run_paperlsq258", kind="run", loss="lsq", n=p258.n, d=p258.d, ld=p258.d, N=p258.N, B=p258.B, lr=p258.lr, noise=p258.noise_std, scale=1.0, port=1, iters=20),
        # few agents with long rows and large batches (logistic regression on heterogeneous agents, the
        # stable step size)
        dict(name="run_logistic6", kind="run", loss="logistic", n=l6.n, d=l6.d, ld=l6.d, N=l6.N, B=l6.B, lr=0.005, noise=0.0, scale=0.0, port=2, iters=100),
        # many agents, one gradient over 16 random 16 KB rows each per iteration: the largest minibatch problem
        dict(name="run_logistic1023", kind="run", loss="logistic", n=big.n, d=big.d, ld=big.d, N=big.N, B=big.B, lr=big.lr, noise=0.0, scale=0.0, port=2, iters=50),
        # one cycle of training steps on a network-sized parameter vector with the built-in noisy quadratic
        # loss: the headline of the benchmark, and the largest case
        dict(name="step_quad31", kind="step", loss="quad", n=q.n, d=q.d, ld=_pad(q.d), noise=q.noise_std, lr=q.lr, port=2, iters=5),
        # the whole 50-iteration run of the same problem in one call
        dict(name="steps_quad31", kind="steps", n=q.n, d=q.d, ld=_pad(q.d), noise=q.noise_std, lr=q.lr, port=2, iters=q.iters),
        # a training step with gradients that the caller evaluated, on a ragged vector of odd length
        dict(name="step_gradient13", kind="step", loss="gradient", n=13, d=100003, ld=100003, noise=0.0, lr=0.1, port=2, iters=1),
        # the exact average of x and y before the first iteration (tau + 1 rounds)
        dict(name="rounds_100", kind="rounds", n=100, d=1 << 20, ld=1 << 20, port=2),
        # exact averaging at the larger size of the paper's consensus comparison
        dict(name="average_1026", kind="average", n=1026, d=1 << 17, ld=1 << 17, port=1),
        # the comparison topologies at 130 agents: ring, static and one-peer exponential graph, and a torus as
        # neighbour tables, tau rounds each, with the consensus observables of each result
        dict(name="compare_130", kind="compare", n=130, d=1 << 20, ld=1 << 20, graph_rows=10),
        # the same at 1026 agents
        dict(name="compare_1026", kind="compare", n=1026, d=1 << 17, ld=1 << 17, graph_rows=27),
    ]


def _log(rng, lo: float, hi: float) -> float:
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    kind = rng.choice(["ministep", "run", "run", "run", "step", "steps", "rounds", "average", "compare", "compare"])
    if kind in ("ministep", "run"):
        loss = rng.choice(["lsq", "logistic"])
        # the ranges of the minibatch configurations: few unknowns and full batches, small problems, long rows at
        # few agents, many agents
        n = int(_log(rng, 3, 1024))
        d = int(_log(rng, 8, 16000 if n <= 64 else 5000))
        batch = rng.randint(4, 64)
        N = batch if d <= 64 and rng.random() < 0.5 else int(_log(rng, batch, 600))
        N = max(min(N, (1 << 31) // (n * d)), 1)
        full = N == batch
        port = 1 if n % 2 == 0 and rng.random() < 0.5 else 2
        if rng.random() < 0.6:
            d = max(d // 4 * 4, 4)
        iters = 1 if kind == "ministep" else rng.randint(10, 50)
        lr = (0.5 / N if full else min(0.01, 0.5 * batch / d)) if loss == "lsq" else 0.02 * min(1.0, 2000.0 / d)
        return dict(kind=kind, loss=loss, n=n, d=d, ld=d, N=N, B=batch, lr=lr, noise=rng.choice([0.0, 0.0, 1.0]),
                    scale=1.0 if full and loss == "lsq" else 0.0, port=port, iters=iters)
    if kind == "compare":
        rows = int(_log(rng, 3, 40))
        cols = rng.randint(rows, rows + rows // 2 + 1)
        n = rows * cols
        d = max(int(_log(rng, 1 << 20, 1 << 27) / n), 8)
        if rng.random() < 0.7:
            d = max(d // 4 * 4, 8)
        ld = d if rng.random() < 0.5 else _pad(d)
        return dict(kind=kind, n=n, d=d, ld=ld, graph_rows=rows)
    n = int(_log(rng, 2, 128)) if kind in ("step", "steps") else int(_log(rng, 4, 2200))
    port = 1 if n % 2 == 0 and rng.random() < 0.5 else 2
    most = {"step": 792e6, "steps": 792e6, "rounds": 2.7e8, "average": 2.7e8}[kind]
    d = max(int(_log(rng, 1 << 17, most) / n), 8)
    if rng.random() < 0.7:
        d = max(d // 4 * 4, 8)
    ld = d if rng.random() < 0.5 else _pad(d)
    case = dict(kind=kind, n=n, d=d, ld=ld, port=port)
    if kind in ("step", "steps"):
        case["noise"] = rng.choice([0.0, 0.01, 0.01])
        case["lr"] = 0.1
        case["iters"] = rng.randint(1, 5) if kind == "step" else rng.randint(4, 50)
        if kind == "step":
            case["loss"] = rng.choice(["quad", "gradient"])
    return case


# ---- inputs ----

def _normal(gen, shape, std=1.0):
    out = torch.empty(shape, dtype=torch.float32, device="cuda")
    out.normal_(0.0, std, generator=gen)
    return out


def _minibatch_data(case, gen):
    """A (n, N, d) and targets or labels (n, N): least squares as in the paper's Sec. 5, heterogeneous logistic
    regression at few agents, 10 % non-zero features at many."""
    n, N, d = case["n"], case["N"], case["d"]
    w = _normal(gen, (d,))
    A = _normal(gen, (n, N, d))
    t = torch.empty((n, N), dtype=torch.float32, device="cuda")
    if case["loss"] == "logistic":
        if n <= 64:
            A += _normal(gen, (n, 1, d), 0.5)
        else:
            for i in range(0, n, 64):
                a = A[i:i + 64]
                a.mul_(torch.empty_like(a).uniform_(generator=gen) < 0.1)
    for i in range(0, n, 64):
        t[i:i + 64] = (A[i:i + 64] * w).sum(dim=2)
    t += _normal(gen, (n, N), 0.1)
    if case["loss"] == "logistic":
        flip = torch.empty((n, N), device="cuda").uniform_(generator=gen) < 0.05
        t = torch.where((t >= 0) ^ flip, 1.0, -1.0).contiguous()
    return A, t


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    kind, n, d, ld = case["kind"], case["n"], case["d"], case["ld"]
    st = dict(case)
    tau = st["tau"] = P.ceca_tau(n)
    if kind in ("ministep", "run"):
        st["A"], st["t"] = _minibatch_data(case, gen)
        st["loss"] = B.make_minibatch_loss(B.LOSS_LSQ if case["loss"] == "lsq" else B.LOSS_LOGISTIC, st["A"], st["t"],
                                           case["N"], case["B"], grad_scale=case["scale"], noise_std=case["noise"], seed=seed)
        if case["B"] == case["N"]:
            idx = torch.arange(case["N"], dtype=torch.int32, device="cuda").expand(case["iters"], n, -1).contiguous()
        else:
            idx = torch.randint(0, case["N"], (case["iters"], n, case["B"]), dtype=torch.int32, device="cuda", generator=gen)
        st["idx"] = idx
        nbytes = (P.dsgd_ceca_workspace_bytes if kind == "ministep" else P.dsgd_ceca_run_workspace_bytes)(n, d, st["loss"])
        st["ws"] = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        st["S"] = _normal(gen, (2 * n, ld), 0.1)
        st["r0"] = tau - 1 if kind == "ministep" else 0
        st["bufs"] = [torch.empty_like(st["S"])]
    elif kind in ("step", "steps"):
        st["S"] = _normal(gen, (2 * n, ld))
        c = st["c"] = _normal(gen, (n, ld))
        if kind == "steps" or case["loss"] == "quad":
            st["loss"] = B.make_quad_center_loss(c, case["noise"], seed)
        else:
            st["loss"] = B.make_gradient_loss(c)
        st["bufs"] = [torch.empty_like(st["S"]) for _ in range(2 if kind == "step" and case["iters"] > 1 else 1)]
    elif kind == "rounds":
        st["S"] = _normal(gen, (2 * n, ld))
        st["bufs"] = [torch.empty_like(st["S"])]
    elif kind == "average":
        st["X"] = _normal(gen, (n, ld))
        st["bufs"] = [torch.empty_like(st["X"])]
    else:
        st["X"] = _normal(gen, (n, ld))
        st["bufs"] = [torch.empty_like(st["X"]) for _ in range(4)]
        topo = (B.TOPO_RING, B.TOPO_STATIC_EXP)
        st["specs"] = [[P.ceca_topology_round(k, n)] for k in topo] + [[P.ceca_topology_round(B.TOPO_ONE_PEER_EXP, n, k) for k in range(tau)]]
        tables = WL.graph_table(n, WL.edges_of("torus", n, case["graph_rows"]))
        st["tables"] = [torch.from_numpy(t[None].copy()).cuda() for t in tables]
        st["obs"] = torch.zeros((4, 5), dtype=torch.float64, device="cuda")
        st["ws"] = torch.empty(P.consensus_error_workspace_bytes(n, d), dtype=torch.uint8, device="cuda")
    return st


# ---- one pass ----

def run(st):
    kind, n, d, ld = st["kind"], st["n"], st["d"], st["ld"]
    out = st["bufs"][0]
    if kind == "ministep":
        P.dsgd_ceca_step(st["S"], out, n, d, st["loss"], st["idx"], st["lr"], st["r0"], st["port"], workspace=st["ws"], ld=ld)
    elif kind == "run":
        P.dsgd_ceca_run(st["S"], out, n, d, st["loss"], st["idx"], st["lr"], st["r0"], st["iters"], st["port"], workspace=st["ws"], ld=ld)
    elif kind == "step":
        src = st["S"]
        for k in range(st["iters"]):
            out = st["bufs"][k % 2]
            st["loss"].k = k
            P.dsgd_ceca_step(src, out, n, d, st["loss"], None, st["lr"], k % st["tau"], st["port"], ld=ld)
            src = out
    elif kind == "steps":
        P.dsgd_ceca_steps(st["S"], out, n, d, st["loss"], st["lr"], 0, st["iters"], st["port"], ld=ld)
    elif kind == "rounds":
        P.ceca_gossip_rounds(st["S"], out, n, d, st["tau"] + 1, st["port"], ld=ld)
    elif kind == "average":
        P.ceca_average(st["X"], out, n, d, st["port"], ld=ld)
    else:
        for j, y in enumerate(st["bufs"]):
            if j < 3:
                P.ceca_mix_rounds(st["X"], y, n, d, st["specs"][j], st["tau"], ld=ld)
            else:
                P.ceca_graph_rounds(st["X"], y, n, d, *st["tables"], st["tau"], ld=ld)
            P.consensus_error(y, n, d, st["obs"][j], workspace=st["ws"], ld=ld)
        return [y[:, :d] for y in st["bufs"]] + [st["obs"]]
    return out[:, :d]


# ---- what a pass cannot do without ----

def work(case):
    n, d, kind = case["n"], case["d"], case["kind"]
    nd, tau = n * d, max(n - 1, 1).bit_length()
    if kind in ("ministep", "run"):
        it, batch = case["iters"], case["B"]
        # the state in and out once per call; the sampled rows, their targets and numbers in every iteration (rows
        # that every iteration reads again stay cached where they fit a few MB)
        rows = 4 * nd * batch + 8 * n * batch
        again = it if case["B"] < case["N"] or rows > 64e6 else 1
        return {"bytes": 16 * nd + rows * again, "flops": it * nd * (4 * batch + 10)}
    noise = 20 if case.get("noise") else 0
    if kind == "step":
        it = case["iters"]
        # x, y and c in, x and y out; round 0 does not read y
        return {"bytes": nd * (20 * it - 4 * -(-it // tau)), "flops": it * nd * (9 + noise)}
    if kind == "steps":
        return {"bytes": 16 * nd, "flops": case["iters"] * nd * (9 + noise)}
    if kind == "rounds":
        return {"bytes": 12 * nd, "flops": (tau + 1) * nd * 6}
    if kind == "average":
        return {"bytes": 8 * nd, "flops": tau * nd * 6}
    # four results and their observables: x in and x+ out per result, x+ in again for its observables
    return {"bytes": 4 * 12 * nd, "flops": nd * (tau * (5 + 2 * tau + 1 + 3 + 9) + 16)}


# ---- how far another correct fp32 implementation may be off ----

def tolerance(case):
    # against the same path in fp64 (1 ulp is 1.2e-7): up to 1.4e-6 and 2.3e-6 after 50 to 200 iterations of a
    # minibatch loss (200 cases), up to 1.2e-7 and 5.5e-7 for everything else (60 cases)
    if case["kind"] == "run":
        return {"rel": 5e-6, "max": 1e-5}
    return {"rel": 5e-7, "max": 2.5e-6}
