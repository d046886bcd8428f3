"""The work that a program has this library do, as measurable cases.

Four kinds of pass, each through the public calls of paper_2606_22768_amd:

  step       the fused outer step of one synchronization round
             (Engine.outer_step), with the round's edge masks uploaded first
             where links drop
  split      the same round in two halves (Engine.mix1 at the round's start,
             Engine.outer_step_blocking at its end)
  consensus  the consensus distance of one array (Engine.consensus_distance),
             as a program monitors it between rounds
  js         the Jensen--Shannon distance of the workers' logits on a batch of
             tokens (js_distance), as an evaluation runs it

Sizes: 2 to 64 workers, from a quarter of a million to 400 million parameters
each, float32 and bf16 storage, every Mix configuration of the method, row
lengths that are and are not multiples of a tile; 1 to 1024 tokens over
vocabularies of 5 000 to 152 064, any top-k up to 1024.  A state takes at
most 26 GB, so that several fit one device; the arrays of a state lie in one
buffer, packed (Engine.alloc_state(spread=False)).
"""

import math

import numpy as np
import torch

import paper_2606_22768_amd as fgd

LR, MU = 0.7, 0.9
SUBSET = ((0.0, 0.33), (0.90, 1.0))  # the Mix2 subset: 43% of the parameters, at both ends of the vector
MASK_SETS = 4                        # rounds of edge masks a state holds, used in turn
HEAD = 48                            # tokens of each position whose logits are lifted

_STEP = dict(op="step", mix1="global", k1=1, mix2="local", k2=1, drop=0.0, nesterov=True, mix_state=False,
             subset=False, cd=True, mom_std=1e-4, drift=1e-3)


def listed():
    step = lambda name, **k: dict(_STEP, name=name, **k)  # noqa: E731
    return [
        # The smallest round: a model of a million parameters on four
        # workers, first step (momentum zero).  The arrays fit the caches;
        # launches and latency count.
        step("step_m4_p1m_f32", M=4, P=1_048_576, dtype="f32", graph="ring", mom_std=0.0),
        # An ordinary round of a 150M-parameter model in float32.
        step("step_m8_p150m_f32", M=8, P=150_000_000, dtype="f32", graph="ring"),
        # The largest: bf16 weights, links that drop anew every round, and a
        # row length that ends inside a tile.
        step("step_m8_p400m_bf16_drops", M=8, P=400_000_005, dtype="bf16", graph="ring", drop=0.1),
        # Two rounds over a directed exponential graph on 16 workers.
        step("step_m16_p60m_f32_exp", M=16, P=60_000_000, dtype="f32", graph="exp", k2=2),
        # 64 workers on a sparse regular graph, one round of Mix1 and three of Mix2.
        step("step_m64_p12m_f32_regular", M=64, P=12_400_000, dtype="f32", graph="regular", mix1="local", k2=3,
             drift=2e-3),
        # A worker count that is no power of two, both mixes by gossip.
        step("step_m12_p7m_bf16_gossip", M=12, P=7_000_003, dtype="bf16", graph="pairs", mix1="local", drop=0.0),
        # 32 workers, the optimizer state averaged too, Mix2 on a subset.
        step("step_m32_p10m_bf16_state", M=32, P=10_000_000, dtype="bf16", graph="exp", mix_state=True, subset=True),
        # A round in two halves, the blocking half writing the next inner start.
        step("split_m8_p100m_bf16", M=8, P=100_000_000, dtype="bf16", graph="ring", drop=0.1) | dict(op="split"),
        # Monitoring the disagreement of 24 workers' weights.
        dict(name="consensus_m24_p40m_bf16", op="consensus", M=24, P=40_000_001, dtype="bf16"),
        # The functional distance over a batch of 1024 tokens, top 100.
        dict(name="js_m8_u1024_v128256_bf16", op="js", M=8, U=1024, K=128_256, dtype="bf16", k=100),
        # A few tokens of a small model: latency.
        dict(name="js_m4_u16_v32000_f32", op="js", M=4, U=16, K=32_000, dtype="f32", k=100),
        # float32 logits, a vocabulary that ends inside a vector, a longer list of tokens.
        dict(name="js_m8_u256_v50257_f32_k300", op="js", M=8, U=256, K=50_257, dtype="f32", k=300),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choices(("step", "split", "consensus", "js"), (9, 2, 2, 6))[0]
    dtype = rng.choice(("f32", "bf16"))
    if op == "js":
        M, K = rng.choice((1, 2, 3, 4, 6, 8, 8, 12, 16)), _log_uniform(rng, 5_000, 152_064)
        es = 4 if dtype == "f32" else 2
        U = _log_uniform(rng, 1, max(2, min(1024, 2_300_000_000 // ((M + 1) * K * es))))
        k = min(K, rng.choice((100, 100, _log_uniform(rng, 1, 1024))))
        return dict(op="js", M=M, U=U, K=K, dtype=dtype, k=k)
    M = rng.choice((2, 3, 4, 4, 6, 8, 8, 8, 12, 16, 16, 24, 32, 48, 64, rng.randint(2, 64)))
    P = _log_uniform(rng, 1 << 18, 1_000_000_000 // M)
    if op == "consensus":
        return dict(op=op, M=M, P=P, dtype=dtype)
    mix1, mix2 = rng.choices((("global", "local"), ("local", "local"), ("global", "identity"), ("identity", "global")),
                             (5, 4, 1, 1))[0]
    graph, k2 = rng.choice(("ring", "exp", "regular", "pairs")), rng.choice((1, 1, 2, 3))
    # Rounds that average completely leave a disagreement of rounding errors
    # alone, which nothing can be compared with: no complete graphs, and few
    # rounds of matchings among few workers.
    if len(_structure(graph, M)[0]) == M - 1:
        graph = "pairs" if M < 4 else "ring"
    if graph == "pairs":
        k2 = 1 if M <= 4 else min(k2, 2)
    state = mix1 == "global" and rng.random() < 0.15
    return dict(_STEP, op=op, M=M, P=P, dtype=dtype, mix1=mix1, mix2=mix2, graph=graph, k2=k2,
                drop=0.1 if graph in ("ring", "regular") and rng.random() < 0.5 else 0.0,
                nesterov=rng.random() < 0.85, mix_state=state, subset=mix2 == "local" and rng.random() < 0.15,
                cd=rng.random() < 0.8)


# ---------------------------------------------------------------- topologies

def _structure(graph, M):
    """Neighbour lists (without the worker itself)."""
    if graph == "pairs":
        return [[j for j in range(M) if j != i] for i in range(M)]
    if graph == "exp":
        hops = [1 << b for b in range(4) if (1 << b) < M]
    elif graph == "regular":
        far = max(2, int(round(M * 0.3)))
        hops = [1, -1, far, -far]
    else:
        hops = [1, -1]
    return [sorted({(i + h) % M for h in hops} - {i}) for i in range(M)]


def _csr(neighbours):
    rows = [sorted(n + [i]) for i, n in enumerate(neighbours)]
    row_ptr = np.cumsum([0] + [len(r) for r in rows]).astype(np.int32)
    return row_ptr, np.array([j for r in rows for j in r], dtype=np.int32)


def _masks(case, rounds, rng, row_ptr, col_idx):
    """One uint8 mask of live entries per round, symmetric, diagonals live;
    None where every link is up."""
    M = case["M"]
    if case["graph"] != "pairs" and case["drop"] == 0.0:
        return None
    out = np.zeros((rounds, col_idx.size), dtype=np.uint8)
    rows = np.repeat(np.arange(M), np.diff(row_ptr))
    for r in range(rounds):
        live = np.zeros((M, M), dtype=bool)
        if case["graph"] == "pairs":  # a random matching
            order = rng.permutation(M)
            for a, b in zip(order[0::2], order[1::2]):
                live[a, b] = True
        else:
            live = np.triu(rng.random((M, M)) >= case["drop"], 1)
        live = live | live.T | np.eye(M, dtype=bool)
        out[r] = live[rows, col_idx]
    return out


def _weights(case, row_ptr, col_idx):
    """(weights or None, reweight): a directed graph has equal weights, the
    others Metropolis weights of each round's live links."""
    if case["graph"] == "exp":
        return np.repeat((1.0 / np.diff(row_ptr)).astype(np.float32), np.diff(row_ptr)), "none"
    return None, "metropolis"


def _topologies(case, seed):
    """Arguments of set_topology: one for Mix1, MASK_SETS of them for Mix2
    (one where nothing drops)."""
    row_ptr, col_idx = _csr(_structure(case["graph"], case["M"]))
    weights, reweight = _weights(case, row_ptr, col_idx)
    rng = np.random.default_rng(seed)

    def one(kind, rounds):
        if kind != "local":
            return dict(kind=kind)
        return dict(kind="csr", row_ptr=row_ptr, col_idx=col_idx, weights=weights, rounds=rounds,
                    masks=_masks(case, rounds, rng, row_ptr, col_idx), reweight=reweight)

    mix1 = one(case["mix1"], case["k1"])
    mix2 = [one(case["mix2"], case["k2"])]
    if mix2[0].get("masks") is not None:
        mix2 += [one(case["mix2"], case["k2"]) for _ in range(MASK_SETS - 1)]
    return mix1, mix2


def _dense(topology, M, r):
    """The mixing matrix of round r in float64 (from the float32 weights that
    a round uses)."""
    W = np.zeros((M, M))
    rows = np.repeat(np.arange(M), np.diff(topology["row_ptr"]))
    cols, masks = topology["col_idx"], topology["masks"]
    live = np.ones(cols.size, dtype=bool) if masks is None else masks[r].astype(bool)
    if topology["reweight"] == "none":
        W[rows, cols] = topology["weights"].astype(np.float64)
        return W
    off = live & (rows != cols)
    degree = np.bincount(rows[off], minlength=M)
    W[rows[off], cols[off]] = 1.0 / (1.0 + np.maximum(degree[rows[off]], degree[cols[off]]))
    W[np.arange(M), np.arange(M)] = 1.0 - W.sum(axis=1)
    return W.astype(np.float32).astype(np.float64)


# -------------------------------------------------------------------- inputs

def _fill(t, P, std, gen, base=None):
    """Rows of N(0, std) draws (added to base's rows), zero past P."""
    for m in range(t.shape[0]):
        row = torch.randn(P, generator=gen, device=t.device).mul_(std)
        if base is not None:
            row += base[m, :P]
        t[m, :P] = row
        t[m, P:] = 0


def _ld(P):
    return (P + 7) // 8 * 8


def _logits(case, seed):
    """Averaged and worker logits: a broad normal over the vocabulary with a
    lifted head of a few dozen tokens, the workers' around the averaged
    model's."""
    M, U, K = case["M"], case["U"], case["K"]
    per = 4 if case["dtype"] == "f32" else 8
    ldk = (K + per - 1) // per * per
    dt = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    gen = torch.Generator(device="cuda").manual_seed(seed)
    avg = torch.zeros((U, ldk), dtype=dt, device="cuda")
    workers = torch.zeros((M, U, ldk), dtype=dt, device="cuda")
    lift = 8.0 / torch.sqrt(1.0 + torch.arange(HEAD, device="cuda"))
    for u0 in range(0, U, 256):
        n = min(256, U - u0)
        z = torch.randn((n, K), generator=gen, device="cuda") * 2.0
        # One position in each of HEAD equal parts of the vocabulary, its rank drawn too.
        at = torch.randint(0, K // HEAD, (n, HEAD), generator=gen, device="cuda")
        at += torch.arange(HEAD, device="cuda") * (K // HEAD)
        rank = torch.rand((n, HEAD), generator=gen, device="cuda").argsort(1)
        z.scatter_(1, at, z.gather(1, at) + lift[rank])
        avg[u0:u0 + n, :K] = z
        for m in range(M):
            workers[m, u0:u0 + n, :K] = z + torch.randn((n, K), generator=gen, device="cuda") * 0.2
    return avg, workers


def prepare(case, seed):
    if case["op"] == "js":
        avg, workers = _logits(case, seed)
        topk = torch.empty((case["U"], case["k"]), dtype=torch.int32, device="cuda")
        return dict(case=case, avg=avg, workers=workers, topk=topk)
    M, P = case["M"], case["P"]
    gen = torch.Generator(device="cuda").manual_seed(seed)
    if case["op"] == "consensus":
        eng = fgd.Engine(M, P, _ld(P), case["dtype"])
        x = torch.empty((M, _ld(P)), dtype=torch.float32 if case["dtype"] == "f32" else torch.bfloat16, device="cuda")
        shared = torch.randn(P, generator=gen, device="cuda").mul_(0.02)  # the workers stay near one another
        _fill(x, P, 2e-3, gen, shared.expand(M, P))
        return dict(case=case, eng=eng, x=x, out=torch.zeros(M, dtype=torch.float64, device="cuda"))
    eng = fgd.Engine(M, P, _ld(P), case["dtype"], outer_lr=LR, momentum=MU, nesterov=case["nesterov"],
                     mix1_state=case["mix_state"])
    mem = eng.alloc_state(spread=False, with_x=case["op"] == "split")
    _fill(mem["theta_prev"], P, 0.02, gen)
    _fill(mem["theta_local"], P, case["drift"], gen, mem["theta_prev"])
    if case["mom_std"]:
        _fill(mem["momentum"], P, case["mom_std"], gen)
    else:
        mem["momentum"].zero_()
    mix1, mix2 = _topologies(case, seed)
    eng.set_topology("mix1", **mix1)
    eng.set_topology("mix2", **mix2[0])
    if case["subset"]:
        cut = lambda f: P if f == 1.0 else int(f * P) // 8 * 8  # noqa: E731
        eng.set_mix2_subset([(cut(a), cut(b)) for a, b in SUBSET])
    st = dict(case=case, eng=eng, mem=mem, mix2=mix2, round=0)
    theta, mom = mem["theta_prev"][:, :P], mem["momentum"][:, :P]
    new = lambda rows: torch.zeros((rows, M), dtype=torch.float64, device="cuda") if case["cd"] else None  # noqa: E731
    rows = lambda cd: [] if cd is None else list(cd.unbind(0))  # noqa: E731
    if case["op"] == "split":
        r1, r2 = eng.num_cd_rows_split()
        st["cd1"], st["cd2"] = new(r1), new(r2)
        st["outputs"] = [theta, mom, mem["x"][:, :P], mem["theta_local"][:, :P], rows(st["cd1"]), rows(st["cd2"])]
    else:
        st["cd"] = new(eng.num_cd_rows())
        st["outputs"] = [theta, mom, rows(st["cd"])]
    return st


def run(state):
    case = state["case"]
    op = case["op"]
    if op == "js":
        d, mean = fgd.js_distance(state["avg"], state["workers"], top_k=case["k"], vocab=case["K"],
                                  topk_out=state["topk"])
        return [d, mean, state["topk"]]
    eng = state["eng"]
    if op == "consensus":
        eng.consensus_distance(state["x"], state["out"])
        return state["out"]
    mem = state["mem"]
    if len(state["mix2"]) > 1:  # this round's links
        eng.set_topology("mix2", **state["mix2"][state["round"] % MASK_SETS])
        state["round"] += 1
    if op == "split":
        eng.mix1(mem["theta_prev"], mem["x"], mem["momentum"], state["cd1"])
        eng.outer_step_blocking(mem["x"], mem["theta_prev"], mem["theta_local"], mem["momentum"], state["cd2"],
                                write_local=True)
    else:
        eng.outer_step(mem["theta_prev"], mem["theta_local"], mem["momentum"], state["cd"])
    return state["outputs"]


# ---------------------------------------------------------- work, tolerances

def work(case):
    e = 4 if case["dtype"] == "f32" else 2
    M = case["M"]
    if case["op"] == "js":
        logits = (M + 1) * case["U"] * case["K"]
        return {"bytes": logits * e + 8 * M * (case["U"] + 1) + 4 * case["U"] * case["k"], "flops": 2 * logits}
    n = M * case["P"]
    if case["op"] == "consensus":
        return {"bytes": n * e + 8 * M, "flops": 4 * n}
    rounds = sum(k for mix, k in ((case["mix1"], case["k1"]), (case["mix2"], case["k2"])) if mix == "local")
    width = 2 if case["graph"] == "pairs" else 1 + len(_structure(case["graph"], M)[0])
    flops = n * (6 + 2 * width * rounds + (4 * (rounds + 3) if case["cd"] else 0))
    state = 8 if case["mix_state"] and case["op"] == "split" else 0
    if case["op"] == "split":  # theta_prev, x; then x, theta_prev, theta_local, v read, theta' twice and v' written
        return {"bytes": n * (2 * e + state + 5 * e + 8), "flops": flops}
    return {"bytes": n * (3 * e + 8), "flops": flops}


def tolerance(case):
    if case["op"] == "js":
        # float64 throughout: 6e-15 from the 64-bit answer for distances of a
        # few hundredths; one near 0 loses digits to its square root.
        return {"rel": 1e-10, "max": 1e-8}
    if case["op"] == "consensus":
        return {"rel": 1e-6, "max": 1e-5}  # float32 deviations: up to 1.4e-7 seen
    if case["dtype"] == "f32":
        return {"rel": 1e-6, "max": 1e-5}  # 6e-8 a pass, three passes in a row compared
    # bf16 weights: another order of the float32 sums moves one in some ten
    # thousand of them by a unit in the last place (up to 2^-7 of its value),
    # twice over three passes.
    return {"rel": 2e-4, "max": 0.016}


# -------------------------------------------------------------- 64-bit answer

def _exact_js(case, seed):
    avg, workers = _logits(case, seed)
    M, U, K, k = case["M"], case["U"], case["K"], case["k"]
    d = torch.empty((M, U), dtype=torch.float64, device="cuda")
    topk = torch.empty((U, k), dtype=torch.int32, device="cuda")
    for u0 in range(0, U, 64):
        u = slice(u0, min(U, u0 + 64))
        a = avg[u, :K].double()
        top = torch.sort(a, dim=1, descending=True, stable=True).indices[:, :k].sort(dim=1).values
        topk[u] = top.int()
        lq = (a - torch.logsumexp(a, 1, keepdim=True)).gather(1, top)
        for m in range(M):
            z = workers[m, u, :K].double()
            lp = (z - torch.logsumexp(z, 1, keepdim=True)).gather(1, top)
            p, q = lp.exp(), lq.exp()
            mix = torch.log(0.5 * (p + q))
            js = 0.5 * (p * (lp - mix) + q * (lq - mix)).sum(1)
            d[m, u] = torch.sqrt(js.clamp_min(0) / math.log(2.0))
    return [d, d.mean(1), topk]


def _spread(u):
    return (u - u.mean(0, keepdim=True)).square().sum(1)


def exact(case, seed):
    if case["op"] == "js":
        return _exact_js(case, seed)
    state = prepare(case, seed)  # the same inputs; the engine is not used
    M, P = case["M"], case["P"]
    chunk = max(1, (1 << 27) // M)
    cuts = [(a, min(P, a + chunk)) for a in range(0, P, chunk)]
    if case["op"] == "consensus":
        return sum(_spread(state["x"][:, a:b].double()) for a, b in cuts)
    mem, bf16, split = state["mem"], case["dtype"] == "bf16", case["op"] == "split"
    mix1, mix2 = _topologies(case, seed)
    to = lambda t, kind, k: [torch.from_numpy(_dense(t, M, r)).cuda() for r in range(k)] if kind == "local" else []  # noqa: E731
    W1, W2 = to(mix1, case["mix1"], case["k1"]), to(mix2[0], case["mix2"], case["k2"])

    def mix(u, kind, W, keep=None):
        """Every round's output, the input first."""
        if kind == "global":
            return [u, u.mean(0, keepdim=True).expand_as(u)]
        out = [u]
        for w in W:
            v = w @ out[-1]
            out.append(v if keep is None else torch.where(keep, v, out[-1]))
        return out

    theta = torch.empty((M, P), dtype=torch.float64, device="cuda")
    mom = torch.empty_like(theta)
    xs = torch.empty_like(theta) if split else None
    cd1, cd2, cdt = [], [], []

    def add(cd, rows, kind):
        for i, u in enumerate(rows):
            s = torch.zeros(M, dtype=torch.float64, device="cuda") if kind == "global" and i else _spread(u)
            if i < len(cd):
                cd[i] = cd[i] + s
            else:
                cd.append(s)

    for a, b in cuts:
        prev, local = mem["theta_prev"][:, a:b].double(), mem["theta_local"][:, a:b].double()
        v = mem["momentum"][:, a:b].double()
        keep = None
        if case["subset"]:
            at = torch.arange(a, b, device="cuda")
            keep = torch.zeros(b - a, dtype=torch.bool, device="cuda")
            for f0, f1 in SUBSET:
                keep |= (at >= int(f0 * P) // 8 * 8) & (at < (P if f1 == 1.0 else int(f1 * P) // 8 * 8))
        g = mix(prev - local, case["mix2"], W2, keep)
        x = mix(prev, case["mix1"], W1)
        if case["mix_state"]:
            v = mix(v, case["mix1"], W1)[-1]
        if case["cd"]:
            add(cd2, g, case["mix2"])
            add(cd1, x, case["mix1"])
        x = x[-1]
        if split:
            xs[:, a:b] = x
            if bf16:  # x is stored between the halves
                x = x.bfloat16().double()
        mom[:, a:b] = MU * v + g[-1]
        step = g[-1] + MU * mom[:, a:b] if case["nesterov"] else mom[:, a:b]
        theta[:, a:b] = x - LR * step
        if case["cd"]:
            t = theta[:, a:b]
            add(cdt, [t.bfloat16().double() if bf16 else t], "")
    if split:
        return [theta, mom, xs, theta, cd1, cd2 + cdt]
    return [theta, mom, cd2 + cd1 + cdt]
