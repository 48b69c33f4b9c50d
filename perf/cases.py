"""The workloads this framework is timed on, through its public Python API.

listed() names the fixed cases, draw() makes more of the same ranges,
prepare() builds what a program holds before the call (instances, colonies,
batches, network parameters), run() is one pass as a program makes it, work()
its minimum traffic and arithmetic, exact() the 64-bit values of the outputs
that are computed numbers of the network and the set-up.

A colony's outputs are its tours (whole numbers), their lengths and the trails
after the iteration; a later pass on the same state is the next iteration.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2003_11902_amd import learned as L
from paper_2003_11902_amd import mmas as M

RHO = 0.02
KNN = 16    # scored neighbours per city
HID = 128   # hidden units of the edge-scoring network


def listed():
    return [
        # the smallest colony of the paper's tables (d198's size, ants = n): one
        # iteration is a few launches and a short chain, so latency counts
        dict(name="colony198", what="colony", n=198, ants=198, cand_len=32, tabu="bitmask", kind="uniform",
             problem="tsp"),
        # the default benchmark: pr1002's size, ants = n, bitmask tabu
        dict(name="colony1002", what="colony", n=1002, ants=1002, cand_len=32, tabu="bitmask", kind="clustered",
             problem="tsp"),
        # the benchmark's second line: the same colony on the compact tabu
        dict(name="colony1002_compact", what="colony", n=1002, ants=1002, cand_len=32, tabu="compact",
             kind="clustered", problem="tsp"),
        # fl3795's size, more ants than the GPU has SIMDs; also the colony the
        # learned heuristic is evaluated on
        dict(name="colony3795", what="colony", n=3795, ants=3795, cand_len=32, tabu="bitmask", kind="uniform",
             problem="tsp"),
        # no candidate list: every step weighs every unvisited city (the shape
        # of the paper's kernel comparison)
        dict(name="nolist1002", what="colony", n=1002, ants=1002, cand_len=0, tabu="bitmask", kind="clustered",
             problem="tsp"),
        # few ants with local search: the run that makes reference lengths
        dict(name="two_opt3795", what="two_opt", n=3795, ants=64, cand_len=32, ls_nn=8, pher="dense"),
        # the largest instance (d18512's size): candidate-only trails and 2-opt
        dict(name="two_opt18512", what="two_opt", n=18512, ants=64, cand_len=16, ls_nn=8, pher="candidates"),
        # uneven instances advanced together, tuned and captured once: serving
        # many requests of different sizes
        dict(name="batch_mixed", what="batch", count=20, n_lo=100, n_hi=2000),
        # many small colonies of few ants, 8 seeds per instance: making training
        # labels (captured, launch shape left at its default)
        dict(name="batch_labels", what="labels", count=20, seeds=8, ants=64, n_lo=200, n_hi=1000),
        # scoring an instance's edges with the network and installing the result
        dict(name="infer3795", what="infer", n=3795, kind="uniform"),
        # one optimisation step of the network's training (gradient, Adam, the
        # bfloat16 copies), the training loop's mini-batch
        dict(name="train65536", what="train", edges=65536, groups=256),
        # a new instance: from the distance matrix in host memory to a colony
        # that can construct
        dict(name="setup1002", what="setup", n=1002, ants=1002, cand_len=32, kind="clustered"),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))))


def draw(rng):
    what = rng.choice(["colony", "colony", "colony", "nolist", "two_opt", "batch", "labels", "infer", "train", "setup"])
    kind = rng.choice(["uniform", "clustered"])
    if what in ("colony", "nolist"):
        n = _log_int(rng, 100, 4000 if what == "colony" else 1100)
        ants = n if rng.random() < 0.7 else _log_int(rng, 64, max(64, n))
        return dict(what="colony", n=n, ants=ants, cand_len=rng.randint(8, 32) if what == "colony" else 0,
                    tabu=rng.choice(["bitmask", "bitmask", "compact", "list"]), kind=kind,
                    problem=rng.choice(["tsp", "tsp", "atsp"]))
    if what == "two_opt":
        n = _log_int(rng, 500, 12000)
        return dict(what="two_opt", n=n, ants=rng.randint(32, 64), cand_len=rng.choice([16, 24, 32]),
                    ls_nn=rng.randint(5, 10), pher="dense" if n < 5000 else "candidates")
    if what == "batch":
        lo = rng.randint(100, 400)
        return dict(what="batch", count=rng.randint(6, 20), n_lo=lo, n_hi=rng.randint(lo + 100, 2000))
    if what == "labels":
        lo = rng.randint(200, 500)
        return dict(what="labels", count=rng.randint(4, 20), seeds=8, ants=64, n_lo=lo, n_hi=rng.randint(lo + 100, 1000))
    if what == "infer":
        return dict(what="infer", n=_log_int(rng, 200, 4000), kind=kind)
    if what == "train":
        return dict(what="train", edges=_log_int(rng, 4096, 65536), groups=256)
    n = _log_int(rng, 200, 4000)
    return dict(what="setup", n=n, ants=n, cand_len=rng.randint(8, 32), kind=kind)


# ---- inputs ---------------------------------------------------------------------


def _coords(n, kind, rng):
    side = 1e6 if n > 8000 else 1e4
    if kind == "uniform":
        return rng.uniform(0.0, side, (n, 2))
    centres = rng.uniform(0.0, side, (20, 2))
    return centres[rng.integers(0, 20, n)] + rng.normal(0.0, 0.03 * side, (n, 2))


def _dist(xy, problem="tsp", rng=None):
    """Integer Euclidean distances (1 between coincident cities), as an int32
    tensor on the GPU; for the asymmetric problem with one-way surcharges up
    to 50 %."""
    n = xy.shape[0]
    p = torch.from_numpy(xy).cuda()
    out = torch.empty((n, n), dtype=torch.int32, device="cuda")
    block = max(1, (1 << 25) // n)
    for s in range(0, n, block):
        d = p[s:s + block, None, :] - p[None, :, :]
        out[s:s + block] = torch.floor(torch.sqrt((d * d).sum(-1)) + 0.5).clamp_(min=1.0).to(torch.int32)
    if problem == "atsp":
        f = torch.from_numpy(rng.random((n, n))).cuda()
        out += torch.floor(0.5 * f * out.double()).to(torch.int32)
    out.fill_diagonal_(0)
    return out


def _instance(case, seed):
    """(coordinates float64 [n, 2], distances int32 [n, n] on the GPU)."""
    rng = np.random.default_rng(seed)
    xy = _coords(case["n"], case.get("kind", "uniform"), rng)
    return xy, _dist(xy, case.get("problem", "tsp"), rng)


def _sizes(case):
    """The instances' sizes (the case's own, so that every seed has the same)."""
    rng = np.random.default_rng([case["count"], case["n_lo"], case["n_hi"]])
    return [int(n) for n in rng.integers(case["n_lo"], case["n_hi"] + 1, size=case["count"])]


def _params(seed):
    """Network parameters: the training's initial ones, the output bias at the
    log odds of a tour edge among 16 neighbours."""
    return L.init_params(seed, math.log(0.125 / 0.875))


def _edges(case, seed):
    """(X bfloat16 [E, 16], targets float32 [E]): feature rows with the ranges
    that instances give, targets in eighths."""
    g = torch.Generator().manual_seed(seed)
    E = case["edges"]
    r = (torch.arange(E) % KNN).float()
    X = torch.zeros(E, 16)
    X[:, 0] = (0.25 + 0.075 * r) * (0.8 + 0.4 * torch.rand(E, generator=g))
    X[:, 1] = r / 15.0
    X[:, 2] = torch.clamp(r + torch.randint(-3, 6, (E,), generator=g), 0, 16) / 16.0
    ang = 2 * math.pi * torch.rand(E, generator=g)
    X[:, 3] = X[:, 0] * torch.cos(ang)
    X[:, 4] = X[:, 0] * torch.sin(ang)
    X[:, 5] = torch.randint(8, 25, (E,), generator=g) / 16.0
    X[:, 6] = torch.randint(8, 25, (E,), generator=g) / 16.0
    X[:, 7] = 0.7 + 0.6 * torch.rand(E, generator=g)
    share = torch.rand(E, generator=g) < 0.9 * torch.exp(-0.45 * r)
    F = share * torch.randint(0, 9, (E,), generator=g) / 8.0
    return X.to(torch.bfloat16), F.float()


def _moments(seed):
    """Adam's moments in mid-training."""
    g = torch.Generator().manual_seed(seed + 1)
    P = M.mlp_param_count()
    return 1e-4 * torch.randn(P, generator=g), 1e-8 * (0.5 + torch.rand(P, generator=g))


ADAM_STEP, LR = 1000, 2e-3


class _State:
    pass


_STREAMS = []


def _stream():
    """The one stream all batches run on (a captured step cannot use the null
    stream), so that passes follow each other."""
    if not _STREAMS:
        _STREAMS.append(torch.cuda.Stream())
    return _STREAMS[0]


def prepare(case, seed):
    st = _State()
    st.what = case["what"]
    st.it = 0
    if st.what == "colony":
        _, d = _instance(case, seed)
        c = M.Colony(d.cpu().numpy(), case["ants"], cand_len=case["cand_len"], rho=RHO, seed=1 + seed,
                     tabu=case["tabu"], problem=case["problem"])
        st.colony, st.out = c, _colony_views(c)
    elif st.what == "two_opt":
        _, d = _instance(case, seed)
        c = M.Colony(d.cpu().numpy(), case["ants"], cand_len=case["cand_len"], rho=RHO, seed=1 + seed,
                     pher=case["pher"], ls_nn=case["ls_nn"])
        st.colony, st.out = c, _colony_views(c)
    elif st.what == "batch":
        rng = np.random.default_rng(seed)
        dists = [_dist(_coords(n, "clustered" if k % 2 else "uniform", rng)).cpu().numpy()
                 for k, n in enumerate(_sizes(case))]
        params = [M.make_params(d.shape[0], d.shape[0], cand_len=32, rho=RHO, seed=1 + k) for k, d in enumerate(dists)]
        st.batch = M.Batch(dists, params, stream=_stream())
        st.batch.tune()
        st.batch.capture()
        st.out = [_colony_views(st.batch.instance(k)) for k in range(len(dists))]
    elif st.what == "labels":
        rng = np.random.default_rng(seed)
        R = case["seeds"]
        dists, params = [], []
        for k, n in enumerate(_sizes(case)):
            d = _dist(_coords(n, "clustered" if k % 2 else "uniform", rng)).cpu().numpy()
            for r in range(R):
                dists.append(d)
                params.append(M.make_params(n, case["ants"], cand_len=32, rho=RHO, seed=1 + r))
        st.batch = M.Batch(dists, params, stream=_stream())
        st.batch.capture()
        st.out = [_seed_views(st.batch, k * R, R) for k in range(case["count"])]
    elif st.what == "infer":
        xy, st.dist = _instance(case, seed)
        st.xy = torch.from_numpy(xy.astype(np.float32)).cuda()
        st.params = torch.from_numpy(_params(seed)).cuda()
        st.colony = M.Colony(st.dist.cpu().numpy(), 64, cand_len=32, rho=RHO, seed=1 + seed)
        st.heur = st.colony.tensor(M.MMAS_BUF_HEUR)
    elif st.what == "train":
        X, F = _edges(case, seed)
        st.X, st.F = X.view(torch.int16).cuda(), F.cuda()
        st.params = torch.from_numpy(_params(seed)).cuda()
        st.m, st.v = (t.cuda() for t in _moments(seed))
        st.packed = M.mmas_mlp_pack(st.params)
        P = M.mlp_param_count()
        st.groups = case["groups"]
        st.partial = torch.empty(st.groups * (P + 1), dtype=torch.float32, device="cuda")
        st.grad = torch.empty(P + 1, dtype=torch.float32, device="cuda")
        st.out = {"grad": st.grad[:P], "loss": st.grad[P:], "params": st.params, "m": st.m, "v": st.v}
    elif st.what == "setup":
        _, d = _instance(case, seed)
        st.dist, st.case, st.seed = d.cpu().numpy(), case, seed
    else:
        raise ValueError(f"unknown case {case!r}")
    return st


def _colony_views(c):
    return [c.tensor(M.MMAS_BUF_TOURS), c.tensor(M.MMAS_BUF_LENGTHS), c.tensor(M.MMAS_BUF_PHEROMONE)]


def _seed_views(batch, first, count):
    """The same three views over `count` consecutive colonies of one size,
    which lie at one stride in the batch's workspace."""
    one, two = batch.instance(first), batch.instance(first + 1)
    out = []
    for which in (M.MMAS_BUF_TOURS, M.MMAS_BUF_LENGTHS, M.MMAS_BUF_PHEROMONE):
        t = one.tensor(which)
        step = two.buffer(which)[0] - one.buffer(which)[0]
        last = batch.instance(first + count - 1).buffer(which)[0] - one.buffer(which)[0]
        if step % t.element_size() or last != (count - 1) * step:
            raise RuntimeError("the colonies of one size do not lie at one stride")
        whole = batch.ws.view(t.dtype)
        start = (one.buffer(which)[0] - batch.ws.data_ptr()) // t.element_size()
        out.append(torch.as_strided(whole, (count, t.numel()), (step // t.element_size(), 1), start))
    return out


def run(st):
    if st.what in ("colony", "two_opt"):
        st.colony.iterate(st.it)
        st.it += 1
        return st.out
    if st.what in ("batch", "labels"):
        st.batch.step()
        return st.out
    if st.what == "infer":
        knn, X, _ = M.mmas_mlp_features(st.dist, st.xy)
        s = M.mmas_mlp_forward(X, st.params, M.mmas_mlp_pack(st.params))
        st.colony.set_learned_heuristic(knn, s)
        return {"knn": knn, "scores": s, "heuristic": st.heur}
    if st.what == "train":
        M.mmas_mlp_grad(st.X, st.F, st.params, st.packed, groups=st.groups, partial=st.partial, grad=st.grad)
        M.mmas_mlp_adam(st.params, st.grad, st.m, st.v, LR, ADAM_STEP + st.it)
        st.it += 1
        st.packed = M.mmas_mlp_pack(st.params)
        return st.out
    c = M.Colony(st.dist, st.case["ants"], cand_len=st.case["cand_len"], rho=RHO, seed=1 + st.seed)
    c.prepare_choice_info()
    return {"cand": c.tensor(M.MMAS_BUF_CAND), "nn_tour": c.tensor(M.MMAS_BUF_NN_TOUR),
            "heuristic": c.tensor(M.MMAS_BUF_HEUR), "trails": c.tensor(M.MMAS_BUF_PHEROMONE),
            "choice": c.tensor(M.MMAS_BUF_CHOICE)}


# ---- what a pass cannot do without ----------------------------------------------


# operations of one candidate's key: a quarter of a Philox4x32-10 block (20
# multiplies and 40 exclusive ors), a logarithm (about 25) and the product
KEY_OPS = 60 / 4 + 26


def _iteration(n, ants, cl, dense=True):
    """An iteration: trails and heuristic read, trails and choice_info written,
    the candidate lists and distances along the tours read, the tours and
    lengths written; one key per candidate and step (without lists, one per
    unvisited city)."""
    stored = n * n if dense else n * cl
    b = 16 * stored + 6 * n * cl + ants * n * (2 + 4) + 8 * ants
    if cl == 0:
        return b, ants * n * (n - 1) / 2 * KEY_OPS
    return b, ants * (n - 1) * cl * KEY_OPS


def work(case):
    what = case["what"]
    if what in ("colony", "two_opt"):
        n, ants = case["n"], case["ants"]
        b, f = _iteration(n, ants, case["cand_len"], case.get("pher", "dense") == "dense")
        if what == "two_opt":  # every city of every tour examined once
            b += 6 * n * case["ls_nn"] + ants * n * 4
            f += ants * n * 2 * case["ls_nn"] * 6
        return {"bytes": b, "flops": f}
    if what in ("batch", "labels"):
        tot = [(_iteration(n, case.get("ants", n), 32), case.get("seeds", 1)) for n in _sizes(case)]
        return {"bytes": sum(b * r for (b, _), r in tot), "flops": sum(f * r for (_, f), r in tot)}
    mlp = 2 * (8 * HID + HID * HID + HID)
    if what == "infer":
        n = case["n"]
        return {"bytes": 8.0 * n * n + KNN * n * (2 + 4), "flops": KNN * n * (mlp + 2 * HID * 30)}
    if what == "train":
        E = case["edges"]
        return {"bytes": E * 36 + 7 * 4 * M.mlp_param_count(), "flops": E * (3 * mlp + 2 * HID * 60)}
    n = case["n"]
    # the matrix from the host and read once; heuristic, trails, choice_info, lists
    return {"bytes": 4.0 * n * n * 5 + 2 * n * case["cand_len"] + 2 * n, "flops": 3.0 * n * n}


# ---- 64-bit values ---------------------------------------------------------------


def _network64(X, p):
    """(scores, z1, h1, z2, h2) of the network on float64 inputs [E, 16]."""
    o = np.cumsum([16 * HID, HID, HID * HID, HID, HID])
    W1, b1, W2 = p[:o[0]].view(16, HID), p[o[0]:o[1]], p[o[1]:o[2]].view(HID, HID)
    b2, w3, b3 = p[o[2]:o[3]], p[o[3]:o[4]], p[o[4]]
    z1 = X @ W1 + b1
    h1 = torch.nn.functional.gelu(z1)
    z2 = h1 @ W2 + b2
    h2 = torch.nn.functional.gelu(z2)
    return h2 @ w3 + b3, z1, h1, z2, h2


def _exact_infer(case, seed):
    xy, dist = _instance(case, seed)
    n = case["n"]
    d = dist.double()
    j = torch.arange(n, device="cuda", dtype=torch.float64)
    key = d * 65536.0 + j
    key.fill_diagonal_(math.inf)
    knn = (torch.topk(key, KNN, dim=1, largest=False, sorted=True).values % 65536.0).long()
    del key
    near = torch.gather(d, 1, knn)
    dbar = near.mean(1)
    indeg = torch.bincount(knn.reshape(-1), minlength=n).double()
    back = knn[knn] == torch.arange(n, device="cuda")[:, None, None]
    rank = torch.where(back.any(2), back.double().argmax(2), KNN).double()
    p = torch.from_numpy(xy.astype(np.float32)).cuda().double()
    rel = (p[knn] - p[:, None, :]) / dbar[:, None, None]
    r = torch.arange(KNN, device="cuda", dtype=torch.float64).expand(n, KNN)
    one = torch.ones(n, KNN, device="cuda", dtype=torch.float64)
    X = torch.stack([near / dbar[:, None], r / 15.0, rank / 16.0, rel[..., 0], rel[..., 1], indeg[knn] / 16.0,
                     indeg[:, None] / 16.0 * one, dbar[knn] / dbar[:, None]] + [0 * one] * 8, dim=2)
    s = _network64(X.reshape(-1, 16), torch.from_numpy(_params(seed)).cuda().double())[0]
    m = 2.0 * torch.sigmoid(s.view(n, KNN))
    mult = m.min(1, keepdim=True).values.expand(n, n).clone()
    mult.scatter_(1, knn, m)
    heur = (mult / d) ** 2
    heur.fill_diagonal_(0.0)
    return {"knn": None, "scores": s, "heuristic": heur.reshape(-1)}


def _exact_train(case, seed):
    X, F = _edges(case, seed)
    X, F = X.double().cuda(), F.double().cuda()
    p = torch.from_numpy(_params(seed)).cuda().double().requires_grad_(True)
    s = _network64(X, p)[0]
    loss = (torch.nn.functional.softplus(s) - F * s).sum()
    g = torch.autograd.grad(loss / X.shape[0], p)[0]
    m, v = (t.cuda().double() for t in _moments(seed))
    m, v = 0.9 * m + 0.1 * g, 0.999 * v + 0.001 * g * g
    step = (m / (1 - 0.9 ** ADAM_STEP)) / (torch.sqrt(v / (1 - 0.999 ** ADAM_STEP)) + 1e-8)
    return {"grad": g, "loss": loss.detach().reshape(1), "params": p.detach() - LR * step, "m": m, "v": v}


def _exact_setup(case, seed):
    _, dist = _instance(case, seed)
    d = dist.cpu().numpy()
    n = d.shape[0]
    left, tour, cur = np.ones(n, bool), [0], 0
    left[0] = False
    length = 0
    for _ in range(n - 1):
        nxt = int(np.where(left, d[cur], np.iinfo(np.int32).max).argmin())
        length += int(d[cur, nxt])
        left[nxt] = False
        cur = nxt
        tour.append(cur)
    length += int(d[cur, 0])
    h = 1.0 / dist.double() ** 2
    h.fill_diagonal_(0.0)
    tau = torch.full((n * n,), 1.0 / (RHO * length), dtype=torch.float64)
    h = h.reshape(-1).cpu()
    return {"cand": None, "nn_tour": None, "heuristic": h, "trails": tau, "choice": tau * h}


def exact(case, seed):
    if case["what"] == "infer":
        return _exact_infer(case, seed)
    if case["what"] == "train":
        return _exact_train(case, seed)
    if case["what"] == "setup":
        return _exact_setup(case, seed)
    return None  # tours are whole numbers; the trails follow from them
