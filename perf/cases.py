"""The calls that users of this library make, as measured cases.

Every case is a knowledge base of one shape, a batch width and one operation,
through the public entry points of ``paper_2002_06115_amd``:

  follow      one query: Y = kb.follow(X, R)
  hops2       two-hop inference: kb.follow(kb.follow(X, R), R)
  step        one differentiable hop, forward and backward (autograd)
  residual    the same for the residual hop follow(X, R) + gamma * X
  accumulate  Y = follow(X, R) + gamma * Z, then the gradients of the hop
  chain       a training step of the three-hop model: softmax over relations,
              follow, L1 normalisation, softmax cross-entropy, full backward
  head        the softmax cross-entropy of the last hop alone

Activations are entity-major [N][b] float32.  Triples are drawn on the GPU
from Zipf or uniform marginals, distinct, and handed to the library as host
int32 arrays, as a program that loads a KB from disk would.
"""
import math

import torch

import paper_2002_06115_amd as kbf

HOPS = 3
GAMMA = 0.5


def _case(name, op, entities, relations, triples, batch, subj=0.0, obj=0.0, rel=0.0,
          inverse=False, soft=False, grid=0, x="softmax", graph=False):
    """subj / obj / rel: Zipf exponents of the marginals (0: uniform); inverse:
    the second half of the relations are the inverses of the first; soft:
    triples carry confidences; grid: the side of a grid KB instead of drawn
    triples; x: how the entity sets look (softmax, sparse, khot)."""
    return dict(name=name, op=op, entities=entities, relations=relations, triples=triples,
                batch=batch, subj=subj, obj=obj, rel=rel, inverse=inverse, soft=soft, grid=grid,
                x=x, graph=graph)


def listed():
    return [
        # A few questions at once over a small KB: the smallest call, all latency.
        _case("query_small_b4", "follow", 1_000, 10, 5_000, 4, x="khot"),
        # One question over a KB of 20 M facts: a single column, rows of 4 bytes.
        _case("query_one_b1", "follow", 2_000_000, 1_000, 20_000_000, 1, subj=1.1, x="khot"),
        # One hop's training step on a KB of the size of MetaQA's, minibatch 128.
        _case("step_metaqa_b128", "step", 43_000, 18, 190_000, 128, subj=1.1, inverse=True),
        # The last, ragged minibatch of an epoch on the same KB.
        _case("step_metaqa_b93", "step", 43_000, 18, 190_000, 93, subj=1.1, inverse=True),
        # The three-hop model on the small KB, its step captured in a HIP graph.
        _case("chain_small_b256", "chain", 1_000, 10, 5_000, 256, x="khot", graph=True),
        # The three-hop model on the MetaQA-sized KB, run eagerly.
        _case("chain_metaqa_b128", "chain", 43_000, 18, 190_000, 128, subj=1.1, inverse=True,
              x="khot"),
        # A residual hop of KB completion at the paper's sizes (75 k entities,
        # 200 relations, 154 k facts) and its minibatch of 10.
        _case("residual_completion_b10", "residual", 75_492, 200, 154_213, 10, subj=1.05, obj=1.05,
              rel=1.2),
        # A hop over a KB with uncertain facts, added to what other hops gave.
        _case("accumulate_soft_b64", "accumulate", 1_000_000, 200, 8_000_000, 64, subj=1.05,
              obj=1.05, rel=1.2, soft=True),
        # The grid scalability experiment: two-hop inference, 128 queries.
        _case("hops2_grid_b128", "hops2", 1_000_000, 100, 3_996_000, 128, grid=1_000, x="khot"),
        # A Freebase-subset-sized KB (12.9 M entities, 43.7 M facts) at the
        # paper's minibatch of 10.
        _case("step_freebase_b10", "step", 12_942_798, 616, 43_724_175, 10, subj=1.05, obj=1.05,
              rel=1.2, x="sparse"),
        # The headline benchmark: 10 M entities, 50 M facts, minibatch 32.
        _case("step_large_b32", "step", 10_000_000, 600, 50_000_000, 32, subj=1.05, obj=1.05,
              rel=1.2, x="sparse"),
        # The training-shaped benchmark: wide minibatches, hub subjects.
        _case("step_train_b256", "step", 2_000_000, 1_000, 20_000_000, 256, subj=1.1),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["follow", "follow", "step", "step", "step", "residual", "accumulate",
                     "chain", "head"])
    entities = _log_int(rng, 1_000, 100_000 if op in ("chain", "head") else 3_000_000)
    triples = int(entities * rng.uniform(3.0, 10.0))
    relations = _log_int(rng, 4, 1_200)
    # From one query to a wide minibatch; whatever width the data leaves.
    batch = _log_int(rng, 1, 256)
    if rng.random() < 0.5:
        batch = min(256, max(4, 4 * round(batch / 4)))
    # Nothing costlier than the largest listed case.
    batch = max(1, min(batch, int(400e6 / triples)))
    return dict(op=op, entities=entities, relations=relations, triples=triples, batch=batch,
                subj=rng.choice([0.0, 1.05, 1.1]), obj=rng.choice([0.0, 1.05]),
                rel=rng.choice([0.0, 1.2]), inverse=False,
                soft=op != "chain" and rng.random() < 0.3, grid=0,
                x="khot" if op == "chain" else rng.choice(["softmax", "sparse", "khot"]),
                graph=op == "chain" and rng.random() < 0.5)


# -- inputs ------------------------------------------------------------------

def _generator(seed, what):
    return torch.Generator(device="cuda").manual_seed(seed * 1_000_003 + what)


def _ids(law, n, count, gen, ranking):
    """``count`` ids below n: uniform (law 0), or Zipf(law) over a ranking of
    the ids that ``ranking``'s seed alone decides.  Ranks by inversion of the
    power law's integral over [1/2, n + 1/2], element by element: a running sum
    of the probabilities would differ from run to run in its last bits."""
    if law == 0:
        return torch.randint(0, n, (count,), device="cuda", generator=gen)
    lo, hi = 0.5 ** (1.0 - law), (n + 0.5) ** (1.0 - law)
    u = torch.rand(count, device="cuda", generator=gen, dtype=torch.float64)
    rank = u.mul_(hi - lo).add_(lo).pow_(1.0 / (1.0 - law)).add_(0.5).long().sub_(1).clamp_(0, n - 1)
    return torch.randperm(n, device="cuda", generator=ranking)[rank]


def _drawn_triples(case, seed):
    """Distinct (s, r, o) triples in random order, int64 on the GPU."""
    n_e, n_t = case["entities"], case["triples"]
    n_r = case["relations"]
    if case["inverse"]:
        n_r, n_t = n_r // 2, n_t // 2
    keys, rounds = None, 0
    while keys is None or keys.numel() < n_t:
        gen = _generator(seed, 10 + rounds)
        count = n_t + n_t // 16 + 64 if keys is None else 2 * (n_t - keys.numel()) + 1024
        s, r, o = (_ids(case[law], n, count, gen, _generator(seed, k))
                   for k, law, n in ((1, "subj", n_e), (2, "rel", n_r), (3, "obj", n_e)))
        new = (s * n_r + r) * n_e + o
        del s, r, o
        keys = torch.unique(new if keys is None else torch.cat([keys, new]))
        rounds += 1
    keys = keys[torch.randperm(keys.numel(), device="cuda", generator=_generator(seed, 4))[:n_t]]
    s, r, o = keys // (n_r * n_e), keys // n_e % n_r, keys % n_e
    if case["inverse"]:
        s, r, o = torch.cat([s, o]), torch.cat([r, r + n_r]), torch.cat([o, s])
    return s, r, o


def _grid_triples(case, seed):
    """Every cell linked to its four neighbours; each edge gets one of the
    relation names at random."""
    n = case["grid"]
    cell = torch.arange(n * n, device="cuda").view(n, n)
    pairs = [(cell[1:], cell[:-1]), (cell[:-1], cell[1:]), (cell[:, :-1], cell[:, 1:]),
             (cell[:, 1:], cell[:, :-1])]
    s = torch.cat([a.reshape(-1) for a, _ in pairs])
    o = torch.cat([b.reshape(-1) for _, b in pairs])
    r = torch.randint(0, case["relations"], s.shape, device="cuda", generator=_generator(seed, 1))
    return s, r, o


def _triples(case, seed):
    """(s, r, o, weight or None) on the GPU."""
    s, r, o = _grid_triples(case, seed) if case["grid"] else _drawn_triples(case, seed)
    w = None
    if case["soft"]:
        w = 1.0 - torch.rand(s.shape, device="cuda", generator=_generator(seed, 5))
    return s, r, o, w


def _khot(n, b, gen, of=None, most=5):
    """Between one and ``most`` entities per column, among ``of`` when given."""
    X = torch.zeros((n, b), device="cuda")
    cols = torch.arange(b, device="cuda")
    k = torch.randint(1, most + 1, (b,), device="cuda", generator=gen)
    for j in range(most):
        rows = torch.randint(0, n if of is None else of.numel(), (b,), device="cuda", generator=gen)
        rows = rows if of is None else of[rows]
        X[rows[k > j], cols[k > j]] = 1.0
    return X


def _entity_sets(case, gen, s):
    n, b = case["entities"], case["batch"]
    if case["x"] == "khot":  # entities that facts are about
        return _khot(n, b, gen, of=s)
    if case["x"] == "sparse":
        X = 1.0 - torch.rand((n, b), device="cuda", generator=gen)
        X *= torch.rand((n, b), device="cuda", generator=gen) < 0.01
        return X / X.sum(0, keepdim=True).clamp_(min=1e-6)
    return torch.softmax(torch.randn((n, b), device="cuda", generator=gen), 0)


def _relation_sets(case, gen):
    n, b = case["relations"], case["batch"]
    if case["grid"]:
        return 1.0 + 0.001 * torch.rand((n, b), device="cuda", generator=gen)
    z = torch.randn((n, b), device="cuda", generator=gen)
    return torch.softmax(2.0 * z if case["x"] == "sparse" else z, 0)


def _targets(case, gen):
    t = _khot(case["entities"], case["batch"], gen)
    return t / t.sum(0, keepdim=True)


def _with_path(case, s, o):
    """Entities that start a path of HOPS edges."""
    alive = torch.ones(case["entities"], dtype=torch.bool, device="cuda")
    for _ in range(HOPS):
        step = torch.zeros_like(alive)
        step[s[alive[o]]] = True
        alive = step
    return alive.nonzero().view(-1)


def _arrays(case, seed, s, o):
    """The case's activations, as the operation takes them."""
    n, b, op = case["entities"], case["batch"], case["op"]
    gen = _generator(seed, 6)
    if op == "head":
        return {"z": torch.randn((n, b), device="cuda", generator=gen), "t": _targets(case, gen)}
    if op == "chain":
        return {"X": _khot(n, b, gen, of=_with_path(case, s, o), most=1),
                "rho": [torch.randn((case["relations"], b), device="cuda", generator=gen)
                        for _ in range(HOPS)],
                "t": _targets(case, gen)}
    a = {"X": _entity_sets(case, gen, s), "R": _relation_sets(case, gen)}
    if op in ("step", "residual", "accumulate"):
        a["dY"] = torch.randn((n, b), device="cuda", generator=gen)
    if op == "accumulate":
        a["Z"] = torch.rand((n, b), device="cuda", generator=gen) / n
    return a


# -- the library's side --------------------------------------------------------

def prepare(case, seed):
    if case["op"] == "head":
        return {"op": "head", **_arrays(case, seed, None, None)}
    s, r, o, w = _triples(case, seed)
    state = {"op": case["op"], **_arrays(case, seed, s, o)}
    host = [x.to(torch.int32).cpu().numpy() for x in (s, r, o)]
    del s, r, o
    state["kb"] = kbf.KB(*host, case["entities"], case["relations"],
                         weight=None if w is None else w.cpu().numpy())
    if case["op"] in ("step", "residual"):
        state["X"].requires_grad_()
        state["R"].requires_grad_()
    if case["graph"]:
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            _chain(state)
        torch.cuda.current_stream().wait_stream(side)
        state["graph"] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(state["graph"]):
            state["out"] = _chain(state)
    return state


def _chain(state):
    from paper_2002_06115_amd import chain
    kb, xs, rs, sums = state["kb"], [state["X"]], [], []
    for t in range(HOPS):
        rs.append(chain.softmax(state["rho"][t]))
        x, total = chain.l1_normalize(kb.follow(xs[-1], rs[-1]))
        xs.append(x)
        sums.append(total)
    loss, _, dx = chain.softmax_xent(xs[-1], state["t"])
    drho = [None] * HOPS
    for t in reversed(range(HOPS)):
        du = chain.l1_normalize_backward(xs[t + 1], sums[t], dx)
        dx, dr = kb.follow_backward(xs[t], rs[t], du)
        drho[t] = chain.softmax_backward(rs[t], dr)
    return {"logits": xs[-1], "loss": loss, "dx": dx, "drho": drho}


def run(state):
    op = state["op"]
    if op == "head":
        from paper_2002_06115_amd import chain
        loss, columns, dz = chain.softmax_xent(state["z"], state["t"])
        return {"loss": loss, "columns": columns, "dz": dz}
    kb = state["kb"]
    if op == "chain":
        if "graph" in state:
            state["graph"].replay()
            return state["out"]
        return _chain(state)
    X, R = state["X"], state["R"]
    if op == "follow":
        return {"Y": kb.follow(X, R)}
    if op == "hops2":
        return {"Y": kb.follow(kb.follow(X, R), R)}
    if op == "accumulate":
        Y = kb.follow_accumulate(X, R, state["Z"], GAMMA)
        dX, dR = kb.follow_backward(X, R, state["dY"])
        return {"Y": Y, "dX": dX, "dR": dR}
    Y = kbf.follow(kb, X, R) if op == "step" else kbf.follow_residual(kb, X, R, GAMMA)
    dX, dR = torch.autograd.grad(Y, (X, R), state["dY"])
    return {"Y": Y, "dX": dX, "dR": dR}


# -- what a pass cannot do without ----------------------------------------------

def work(case):
    """Each call of a pass reads its inputs once and writes its outputs once:
    the triples (three ids, and a confidence in a soft KB), the activations."""
    n, m, b, l = case["entities"], case["relations"], case["batch"], case["triples"]
    ent, rel, kb = 4 * n * b, 4 * m * b, (16 if case["soft"] else 12) * l
    mul = 3 if case["soft"] else 2
    head = {"bytes": 3 * ent, "flops": 12 * n * b}
    if case["op"] == "head":
        return head
    forward = {"bytes": kb + 2 * ent + rel, "flops": mul * l * b}
    backward = {"bytes": kb + 3 * ent + 2 * rel, "flops": 2 * mul * l * b}
    if case["op"] == "residual":
        forward["flops"] += 2 * n * b
        backward["flops"] += 2 * n * b
    if case["op"] == "accumulate":
        forward = {"bytes": forward["bytes"] + ent, "flops": forward["flops"] + 2 * n * b}
    if case["op"] == "follow":
        return forward
    if case["op"] == "hops2":
        return {k: 2 * v for k, v in forward.items()}
    if case["op"] == "chain":
        # Per hop: softmax and its backward (2 + 3 relation arrays),
        # normalisation and its backward (2 + 3 entity arrays).
        hop = {"bytes": forward["bytes"] + backward["bytes"] + 5 * ent + 5 * rel,
               "flops": forward["flops"] + backward["flops"] + 6 * n * b + 12 * m * b}
        return {k: HOPS * hop[k] + head[k] for k in hop}
    return {k: forward[k] + backward[k] for k in forward}


def tolerance(case):
    """One float rounding of a 64-bit sum per output of a hop (2 to 5e-8 was
    seen against exact()); the chains round after every operation (up to
    3.5e-7)."""
    return {"rel": 1.5e-6} if case["op"] == "chain" else {"rel": 2e-7}


# -- the same in 64 bits ----------------------------------------------------------

def _segment_sum(out, row, a_id, A, b_id, B, w):
    """out[row] += w * A[a_id] * B[b_id] over all triples, in float64."""
    order = torch.argsort(row)
    chunk = max(1, min(1 << 20, (1 << 28) // max(1, A.shape[1])))
    for i in range(0, order.numel(), chunk):
        at = order[i:i + chunk]
        v = A[a_id[at]].double()
        v *= B[b_id[at]]
        if w is not None:
            v *= w[at].double()[:, None]
        # Pieces of at most 64 triples of a row first, then the pieces: a hub
        # row's sum is then not one long chain of atomic additions.
        rows = row[at]
        new = torch.ones_like(rows, dtype=torch.bool)
        new[1:] = (rows[1:] != rows[:-1])
        new |= torch.arange(rows.numel(), device="cuda") % 64 == 0
        piece = new.cumsum(0) - 1
        part = torch.zeros((int(piece[-1]) + 1, A.shape[1]), dtype=torch.float64, device="cuda")
        part.index_add_(0, piece, v)
        out.index_add_(0, rows[new], part)
    return out


def _forward(kb, X, R):
    s, r, o, w = kb
    return _segment_sum(torch.zeros(X.shape, dtype=torch.float64, device="cuda"), o, s, X, r, R, w)


def _backward(kb, X, R, dY):
    s, r, o, w = kb
    zeros = lambda t: torch.zeros(t.shape, dtype=torch.float64, device="cuda")  # noqa: E731
    dX = _segment_sum(zeros(X), s, o, dY, r, R, w)
    return dX, _segment_sum(zeros(R), r, o, dY, s, X, w)


def _head(z, t):
    z, t = z.double(), t.double()
    logp = torch.log_softmax(z, 0)
    columns = -(t * logp).sum(0)
    dz = (logp.exp() * t.sum(0, keepdim=True) - t) / z.shape[1]
    return columns.mean(), columns, dz


def exact(case, seed):
    op = case["op"]
    if op == "head":
        a = _arrays(case, seed, None, None)
        loss, columns, dz = _head(a["z"], a["t"])
        return {"loss": loss, "columns": columns, "dz": dz}
    kb = _triples(case, seed)
    a = _arrays(case, seed, kb[0], kb[2])
    X = a["X"]
    if op == "chain":
        xs, rs, sums = [X.double()], [], []
        for t in range(HOPS):
            rs.append(torch.softmax(a["rho"][t].double(), 0))
            u = _forward(kb, xs[-1], rs[-1])
            sums.append(u.sum(0, keepdim=True))
            xs.append(u / sums[-1])
        loss, _, dx = _head(xs[-1], a["t"])
        drho = [None] * HOPS
        for t in reversed(range(HOPS)):
            du = (dx - (dx * xs[t + 1]).sum(0, keepdim=True)) / sums[t]
            dx, dr = _backward(kb, xs[t], rs[t], du)
            drho[t] = rs[t] * (dr - (dr * rs[t]).sum(0, keepdim=True))
        return {"logits": xs[-1], "loss": loss, "dx": dx, "drho": drho}
    R = a["R"]
    Y = _forward(kb, X, R)
    if op == "follow":
        return {"Y": Y}
    if op == "hops2":
        return {"Y": _forward(kb, Y, R)}
    if op == "residual":
        Y += GAMMA * X.double()
    if op == "accumulate":
        Y += GAMMA * a["Z"].double()
    dX, dR = _backward(kb, X, R, a["dY"])
    if op == "residual":
        dX += GAMMA * a["dY"].double()
    return {"Y": Y, "dX": dX, "dR": dR}
