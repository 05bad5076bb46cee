"""Timed cases of the detect-and-aggregate step.

Each case is one call a parameter server makes once per training iteration:
the replica gradients of all f = C(K,r) files are on the GPU, and the step
detects, selects and reduces them to one d-vector.  The buffers the server
keeps from one iteration to the next (detection outputs, result, selection,
workspace) are made once.

A case holds
  K, r, q       workers, replicas per file, bound on the adversaries
  d             gradient coordinates (the model's parameter count)
  mode          "median", or "paper" (the mean when detection succeeds)
  layout        "file": replicas [f][r][d]; "worker": the workers' own
                uploads [K][l][d]
  entry         "step": the whole step in one call; "noalloc": the same
                without a workspace; "parts": detect, clique and aggregate
                called one after the other
  attack        "weak": every adversary distorts every file it holds;
                "optimal": the adversaries {0..q-1} hide behind the honest
                workers {q..2q-1} (an adversary distorts a file iff most of
                its workers are adversaries and the others among those)
  distortion    "reversed" (-100 times the gradient), "alie" (mean minus one
                standard deviation over the files, the same vector from
                every adversary) or "noise" (independent N(0,1))
  dist          honest gradients: "normal" N(0, 0.01^2) or "t3" (Student-t
                with 3 degrees of freedom, times 0.01)
"""
from itertools import combinations
from math import comb, exp, log

import numpy as np
import torch

from paper_2108_02416_amd import aspis

MAX_BYTES = 61_200_000_000   # replica bytes of the largest case


def _case(name, K, r, q, d, mode="median", layout="file", entry="step", attack="optimal",
          distortion="alie", dist="normal"):
    return {"name": name, "K": K, "r": r, "q": q, "d": d, "mode": mode, "layout": layout,
            "entry": entry, "attack": attack, "distortion": distortion, "dist": dist}


def listed():
    return [
        # a softmax layer trained by seven workers: a few microseconds of
        # data, so the call's launches and synchronisations are the cost
        _case("tiny", 7, 3, 2, 7_850, attack="weak", distortion="reversed"),
        # a small network, from a serving loop that must not allocate
        _case("small_noalloc", 7, 3, 2, 100_000, entry="noalloc", attack="weak",
              distortion="reversed"),
        # a middle-sized network under Algorithm 1 as written: detection
        # succeeds and the kept files are averaged
        _case("mean_1m", 15, 3, 3, 1_000_000, mode="paper", attack="weak"),
        # parameter counts of real networks are rarely multiples of four:
        # every row but the first starts off a 16-byte boundary
        _case("odd_2m5", 15, 3, 4, 2_500_001),
        # the largest: ResNet-18's 11.2M parameters, 15 workers, the attack
        # that defeats detection
        _case("headline", 15, 3, 4, 11_200_000),
        # the same cluster aggregating the uploads as the workers send them
        _case("worker_3m", 15, 3, 4, 3_000_000, layout="worker"),
        # a smaller cluster, uploads as sent, an odd parameter count, mean
        _case("worker_mean_odd", 10, 3, 2, 1_234_567, mode="paper", layout="worker",
              attack="weak", distortion="reversed"),
        # 1,330 files, half the adversaries' files without a majority
        _case("k21_1m", 21, 3, 5, 1_250_000, attack="weak", distortion="noise"),
        # 2,300 files of heavy-tailed gradients
        _case("k25_600k", 25, 3, 6, 600_000, distortion="reversed", dist="t3"),
        # redundancy five
        _case("r5_1m", 11, 5, 3, 1_000_000, attack="weak", distortion="alie"),
        # redundancy seven
        _case("r7_400k", 10, 7, 2, 400_000, attack="weak", distortion="reversed"),
        # a server that runs the steps itself: detection, clique search on
        # the host, aggregation
        _case("parts_1m5", 15, 3, 4, 1_500_000, entry="parts"),
    ]


def draw(rng):
    r = rng.choices([3, 5, 7], [7, 2, 1])[0]
    K = rng.randint(*{3: (6, 25), 5: (8, 13), 7: (9, 11)}[r])
    q = rng.randint(1, (K - 1) // 2)
    top = min(11_200_000, MAX_BYTES // (4 * r * comb(K, r)))
    d = int(exp(rng.uniform(log(4_000), log(top))))
    if rng.random() < 0.5:
        d -= d % 4
    layout = rng.choices(["file", "worker"], [2, 1])[0]
    entry = "step" if layout == "worker" else rng.choices(["step", "noalloc", "parts"],
                                                          [4, 1, 1])[0]
    case = _case("", K, r, q, d, mode=rng.choice(["median", "median", "paper"]), layout=layout,
                 entry=entry, attack=rng.choice(["weak", "optimal"]),
                 distortion=rng.choice(["reversed", "alie", "noise"]),
                 dist=rng.choice(["normal", "t3"]))
    del case["name"]
    return case


# ------------------------------------------------------------------ inputs

def _subsets(K, r):
    return np.array(list(combinations(range(K), r)), dtype=np.int64)


def _distorted(case, subsets):
    """[f, r]: which replicas an adversary replaces."""
    q, r = case["q"], case["r"]
    bad = subsets < q
    if case["attack"] == "weak":
        return bad
    hidden = (subsets < 2 * q).all(axis=1) & (bad.sum(axis=1) >= (r + 1) // 2)
    return bad & hidden[:, None]


def _honest(case, n, gen):
    shape = (n, case["d"])
    z = torch.randn(shape, generator=gen, device="cuda")
    if case["dist"] == "t3":
        v = torch.zeros(shape, device="cuda")
        for _ in range(3):
            v.add_(torch.randn(shape, generator=gen, device="cuda").square_())
        z.div_(v.div_(3).sqrt_())
    return z.mul_(0.01)


def _replicas(case, seed):
    """The replica tensor and, per replica (i, s), its row in it."""
    K, r, d = case["K"], case["r"], case["d"]
    subsets = _subsets(K, r)
    f = len(subsets)
    if case["layout"] == "worker":
        grads = torch.empty((K, f * r // K, d), device="cuda")
        row = aspis.worker_rows(K, r)
    else:
        grads = torch.empty((f, r, d), device="cuda")
        row = np.arange(f * r).reshape(f, r)
    flat = grads.view(f * r, d)
    bad = _distorted(case, subsets)
    gen = torch.Generator(device="cuda").manual_seed(seed)
    alie = case["distortion"] == "alie"
    total = torch.zeros(d, dtype=torch.float64, device="cuda") if alie else None
    square = torch.zeros_like(total) if alie else None
    step = max(1, (1 << 26) // d)
    for i0 in range(0, f, step):
        g = _honest(case, min(step, f - i0), gen)
        if case["layout"] == "file":
            grads[i0:i0 + len(g)] = g[:, None, :]
        else:
            for j in range(len(g)):
                for s in range(r):
                    flat[int(row[i0 + j, s])] = g[j]
        if alie:
            total += g.sum(0, dtype=torch.float64)
            square += g.double().square_().sum(0)
    if alie:
        mean = total / f
        value = (mean - (square / f - mean * mean).clamp_(min=0).sqrt_()).float()
    for i, s in zip(*np.nonzero(bad)):
        target = flat[int(row[i, s])]
        if case["distortion"] == "reversed":
            target.mul_(-100.0)
        elif alie:
            target.copy_(value)
        else:
            target.normal_(generator=gen)
    return grads, flat, row


def prepare(case, seed):
    K, r, d = case["K"], case["r"], case["d"]
    grads, _, _ = _replicas(case, seed)
    dev = grads.device
    f = comb(K, r)
    state = {"case": case, "grads": grads, "bufs": aspis.DetectBuffers.empty(f, K, dev),
             "out": torch.empty(d, device=dev),
             "sel": torch.empty(f, dtype=torch.int32, device=dev),
             "ws": None if case["entry"] == "noalloc" else aspis.workspace(K, r, d, dev)}
    aspis.subsets_device(K, r, dev)
    return state


# ---------------------------------------------------------------- the call

def run(state):
    case, grads, bufs = state["case"], state["grads"], state["bufs"]
    K, r, q, mode = case["K"], case["r"], case["q"], case["mode"]
    if case["entry"] == "parts":
        aspis.detect(grads, K, r, bufs=bufs)
        res = aspis.clique(bufs.disagree.cpu().numpy().view(np.uint64), K, q)
        _, kept = aspis.aggregate(grads, K, r, bufs, res, mode=mode, out=state["out"],
                                  sel_out=state["sel"], ws=state["ws"])
    else:
        if case["entry"] == "noalloc":
            got = aspis.detect_aggregate_noalloc(grads, K, r, q, bufs, state["out"],
                                                 sel_out=state["sel"], mode=mode)
        else:
            got = aspis.detect_aggregate(grads, K, r, q, mode=mode, bufs=bufs, out=state["out"],
                                         sel_out=state["sel"], ws=state["ws"],
                                         layout=case["layout"])
        res, kept = got["clique"], got["n_selected"]
    return {"out": state["out"], "sel": state["sel"], "pair_diff": bufs.pair_diff,
            "vote": bufs.vote, "has_majority": bufs.has_majority, "disagree": bufs.disagree,
            "success": res.success, "omega": res.omega, "n_maximum": res.n_maximum,
            "honest": res.honest[0], "kept": kept}


def work(case):
    K, r, d = case["K"], case["r"], case["d"]
    f = comb(K, r)
    rows = f * r
    if case["entry"] == "parts":
        rows += f   # the second call reads the kept rows again
    # one comparison per slot pair, one step of the reduction per file
    return {"bytes": 4 * rows * d + 4 * d + f * 10 + 8 * K,
            "flops": f * d * (r * (r - 1) // 2 + 1)}


def tolerance(case):
    if case["mode"] == "median":
        return "exact"   # the result is one of the inputs
    # 64-bit sums rounded once to 32 bits: half a unit in the last place,
    # whichever order the sum takes
    return {"rel": 6e-8, "max": 1.2e-7}


# -------------------------------------------------------------- reference

def _cliques(adj, K):
    """Every maximal clique of the graph, as bit masks."""
    found = []

    def expand(R, P, X):
        if not P and not X:
            found.append(R)
            return
        pivot = max((v for v in range(K) if (P | X) >> v & 1),
                    key=lambda v: (P & adj[v]).bit_count())
        for v in range(K):
            if (P & ~adj[pivot]) >> v & 1:
                expand(R | 1 << v, P & adj[v], X & adj[v])
                P &= ~(1 << v)
                X |= 1 << v

    expand(0, (1 << K) - 1, 0)
    return found


def exact(case, seed):
    K, r, q, d = case["K"], case["r"], case["q"], case["d"]
    f = comb(K, r)
    if f * d > 2_000_000_000:
        return None   # sorting 455 x 11.2M values takes too long
    _, flat, row = _replicas(case, seed)
    words = flat.view(torch.int32)
    subsets = _subsets(K, r)
    pairs = list(combinations(range(r), 2))
    differ = torch.stack([torch.stack([(words[int(row[i, s])] != words[int(row[i, t])]).any()
                                       for s, t in pairs]) for i in range(f)]).cpu().numpy()
    pair_diff = (differ.astype(np.int64) << np.arange(len(pairs))).sum(axis=1).astype(np.int32)
    same = np.zeros((f, r, r), dtype=bool)
    disagree = [0] * K
    for p, (s, t) in enumerate(pairs):
        same[:, s, t] = same[:, t, s] = ~differ[:, p]
        for i in np.flatnonzero(differ[:, p]):
            u, v = int(subsets[i, s]), int(subsets[i, t])
            disagree[u] |= 1 << v
            disagree[v] |= 1 << u
    size = 1 + same.sum(axis=2)
    vote = size.argmax(axis=1)
    majority = size.max(axis=1) >= (r + 1) // 2
    everyone = (1 << K) - 1
    cliques = _cliques([everyone & ~disagree[u] & ~(1 << u) for u in range(K)], K)
    omega = max(c.bit_count() for c in cliques)
    largest = [c for c in cliques if c.bit_count() == omega]
    success = len(largest) == 1 and omega >= K - q
    honest = largest[0] if success else 0
    if success:
        member = (honest >> subsets & 1).astype(bool)
        sel = np.where(member.any(axis=1), member.argmax(axis=1), -1)
    else:
        sel = vote
    kept = np.flatnonzero(sel >= 0)
    rows = torch.from_numpy(row[kept, sel[kept]].astype(np.int64)).to(flat.device)
    out = torch.empty(d, dtype=torch.float64, device=flat.device)
    step = max(1, (1 << 26) // len(kept))
    for k in range(0, d, step):
        x = flat[:, k:k + step].index_select(0, rows).t().contiguous()
        if case["mode"] != "median" and success:
            out[k:k + step] = x.double().mean(1)
        else:
            out[k:k + step] = x.sort(dim=1).values[:, (len(kept) - 1) // 2].double()
    return {"out": out, "sel": sel.astype(np.int32), "pair_diff": pair_diff,
            "vote": vote.astype(np.int8), "has_majority": majority.astype(np.uint8),
            "disagree": np.array(disagree, dtype=np.int64), "success": int(success),
            "omega": omega, "n_maximum": len(largest), "honest": honest, "kept": len(kept)}
