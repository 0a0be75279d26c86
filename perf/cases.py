"""The work this library is measured on: drafting and verifying batches of token trees.

Every case is one step of multi-draft speculative decoding through the Python binding of the C ABI.
`call` says how a program drives it:

  step   binding.StepPlan.run(): a serving loop that marshalled its arguments once
  path   StepPlan.draft() and StepPlan.verify_path(): only the nodes that decide what is emitted
  calls  binding.<method>_draft() and binding.<method>_verify(), nothing kept between the two
  mass   binding.<method>_verify() on tokens that were drafted before, with the residual mass of every
         node asked for (what an acceptance study reads)

The rows are those of workloads.py: heavy-tailed target logits and a noisy copy as the draft, the
pairs of the toy experiment, or the softmax of such logits where a program hands in probabilities.
"""
import math

import torch

from paper_2411_05289_amd import binding
from paper_2411_05289_amd import workloads

# Node 0 has children (1, 2), node 1 (3, 4), node 3 (5, 6), node 5 (7, 8): a left spine, as a tree
# search over measured acceptance rates gives it.  `tree` = "spine" hands it over as a table.
SPINE = (1, 3, -1, 5, -1, 7, -1, -1, -1)


def _case(name, call, method, B, V, depth, dtype, *, k=2, kind="logits", T=1.0, noise="spread", rows="llm",
          near_uniform=0, tree="complete"):
    return dict(name=name, call=call, method=method, B=B, V=V, k=k, depth=depth, dtype=dtype, kind=kind, T=T,
                noise=noise, rows=rows, near_uniform=near_uniform, tree=tree)


def listed():
    return [
        # one user, the paper's own setting: fp32 logits, 15 nodes; nothing but latency
        _case("one_sequence", "step", "spechub", 1, 32000, 4, "fp32", noise="1.5"),
        # the benchmark's step: a serving batch of 64 sequences, 31-node binary trees
        _case("serving_batch", "step", "spechub", 64, 32000, 5, "bf16"),
        # the same batch with the baseline method
        _case("serving_batch_rrs", "step", "rrs", 64, 32000, 5, "bf16"),
        # the same batch, verifying only along the accepted path
        _case("serving_batch_path", "path", "spechub", 64, 32000, 5, "bf16"),
        # a large vocabulary and a large batch at temperature 0.7: the largest step
        _case("large_vocabulary", "step", "spechub", 256, 128256, 5, "bf16", T=0.7, noise="1.5"),
        # four drafts per node on the longest rows, a quarter of the sequences nearly uniform
        _case("four_drafts_rrs", "step", "rrs", 128, 152064, 3, "bf16", k=4, noise="2.0", near_uniform=4),
        _case("four_drafts_rrsw", "step", "rrsw", 128, 152064, 3, "bf16", k=4, noise="2.0", near_uniform=4),
        # a vocabulary that is no whole number of 16-byte chunks, so that rows start anywhere, and a
        # tree of its own shape
        _case("odd_vocabulary", "step", "rrsw", 48, 50257, 5, "bf16", tree="spine"),
        # a program whose sampler hands over probabilities, calling function by function
        _case("probabilities", "calls", "spechub", 32, 32000, 4, "fp32", kind="probs", noise="1.5"),
        # an acceptance study: residual masses of a serving batch
        _case("residual_mass", "mass", "rrs", 64, 32000, 4, "bf16"),
        # many independent tiny problems: one draft step over 16 tokens each
        _case("tiny_rows", "calls", "spechub", 4096, 16, 2, "fp32", kind="probs", rows="dirichlet"),
        # the toy experiment: 102400 one-step trees over 50 tokens
        _case("toy_pairs", "step", "spechub", 102400, 50, 2, "fp32", T=0.25, rows="toy"),
    ]


def draw(rng):
    call = rng.choice(["step", "step", "step", "path", "calls", "mass"])
    method = rng.choice(["spechub", "spechub", "rrs", "rrsw"])
    kind = "probs" if call in ("calls", "mass") and rng.random() < 0.5 else "logits"
    dtype = "fp32" if kind == "probs" or rng.random() < 0.25 else "bf16"
    V = int(round(math.exp(rng.uniform(math.log(16), math.log(152064)))))
    if rng.random() < 0.5 and V > 64:
        V -= V % 64              # half of the vocabularies are padded to a round size
    k = 2 if method == "spechub" else rng.choice([2, 2, 3, 4])
    tree = "spine" if k == 2 and rng.random() < 0.2 else "complete"
    depth = 5 if tree == "spine" else rng.choice([2, 3, 4, 5] if k == 2 else [2, 3])
    case = dict(call=call, method=method, B=1, V=V, k=k, depth=depth, dtype=dtype, kind=kind,
                T=rng.choice([0.7, 1.0, 1.0]), noise=rng.choice(["spread", "1.5", "2.0"]), rows="llm",
                near_uniform=4 if rng.random() < 0.2 else 0, tree=tree)
    # from one sequence to about an eighth of the largest listed step's rows
    most = min(4.0e8 / (_nodes(case) * V * _size(case)), 100000.0 / _nodes(case))
    case["B"] = int(max(1, round(math.exp(rng.uniform(0.0, math.log(max(1.0, most)))))))
    return case


def _size(case):
    return 4 if case["dtype"] == "fp32" else 2


def _nodes(case):
    return len(SPINE) if case["tree"] == "spine" else workloads.tree_nodes(case["k"], case["depth"])


def _first_children(case):
    """Number of the first child of every node, -1 for leaves."""
    if case["tree"] == "spine":
        return list(SPINE)
    N, k = _nodes(case), case["k"]
    return [k * n + 1 if k * n + k < N else -1 for n in range(N)]


def _internal(case):
    return sum(c >= 0 for c in _first_children(case))


def _rows(case, seed):
    B, N, V = case["B"], _nodes(case), case["V"]
    dtype = torch.float32 if case["dtype"] == "fp32" else torch.bfloat16
    if case["rows"] == "toy":
        wl = workloads.toy_pairs(case["T"], 0.7, 400, repeats=B // 400, seed=seed, device="cuda")
        return wl.target, wl.draft
    if case["rows"] == "dirichlet":
        return workloads.dirichlet_rows(B, N, V, seed=seed, device="cuda")
    gen = torch.Generator().manual_seed(seed + 1000)
    noise = 0.5 + 2.0 * torch.rand(B, generator=gen) if case["noise"] == "spread" else float(case["noise"])
    std = torch.full((B,), 3.0)
    if case["near_uniform"]:
        std[case["near_uniform"] - 1::case["near_uniform"]] = 0.5
    probs = case["kind"] == "probs"
    t, d = workloads.llm_like_logits(B, N, V, logit_std=std, draft_noise_std=noise, seed=seed, device="cuda",
                                     dtype=torch.float32 if probs else dtype, chunk_rows=max(N, (1 << 25) // V))
    if probs:
        t, d = (torch.softmax(x / case["T"], -1).to(dtype) for x in (t, d))
    return t, d


def prepare(case, seed):
    B, N, k = case["B"], _nodes(case), case["k"]
    target, draft = _rows(case, seed)
    gen = torch.Generator(device="cuda").manual_seed(seed + 77)
    u_draft = torch.rand((B, N, k), generator=gen, device="cuda")
    u_verify = torch.rand((B, N, k + 1), generator=gen, device="cuda")
    table = None
    if case["tree"] != "complete":
        table = torch.tensor(_first_children(case), dtype=torch.int32, device="cuda")
    logits = case["kind"] == "logits"
    pb = binding.Problem(target, draft, binding.LOGITS if logits else binding.PROBS, k, case["depth"],
                         case["T"] if logits else 1.0, case["T"] if logits else 1.0, table)
    state = dict(call=case["call"], pb=pb, u_draft=u_draft, u_verify=u_verify)
    if case["call"] in ("step", "path"):
        plan = binding.StepPlan(case["method"], pb, u_draft, u_verify)
        out = dict(plan.out)
        records = plan.pb.draft_stats
        out.update(tokens=plan.tokens, draft_flags=plan.draft_flags, largest=records[..., 0],
                   rest_mass=records[..., 1], record_hub=records.view(torch.int32)[..., 2])
        if case["method"] == "spechub":
            out["hub"] = plan.hub
        state.update(plan=plan, out=out)
    else:
        state.update(draft=getattr(binding, case["method"] + "_draft"),
                     verify=getattr(binding, case["method"] + "_verify"))
        if case["call"] == "mass":
            state["tokens"] = _drafted(case, draft, u_draft)["tokens"].to(torch.int32)
    return state


def run(state):
    if state["call"] == "step":
        state["plan"].run()
        return state["out"]
    if state["call"] == "path":
        state["plan"].draft()
        state["plan"].verify_path()
        return state["out"]
    if state["call"] == "mass":
        return state["verify"](state["pb"], state["tokens"], state["u_verify"], resid_mass=True)
    drafted = state["draft"](state["pb"], state["u_draft"])
    out = state["verify"](state["pb"], drafted["tokens"], state["u_verify"])
    out = dict(out, tokens=drafted["tokens"], draft_flags=drafted["flags"])
    if "hub" in drafted:
        out["hub"] = drafted["hub"]
    return out


def work(case):
    B, N, V, k = case["B"], _nodes(case), case["V"], case["k"]
    inner = _internal(case)
    # draft rows of internal nodes and target rows once each; a step that verifies along the accepted
    # path reads about accepted + 1 target rows per tree, at least the root's
    target_rows = 1 if case["call"] == "path" else N
    rows = B * (inner + target_rows)
    outputs = B * N * (16 + 8 * k + 4)
    if case["call"] in ("step", "path"):
        outputs += B * N * 16
    return {"bytes": rows * V * _size(case) + outputs, "flops": 4 * rows * V}


def tolerance(case):
    # Against 64 bits the draft masses are off by up to 2e-7 (one of them by 1e-6), residual masses by
    # 6e-8 (3e-7).  A token or outcome differs where a uniform lies that close to a threshold: of 40
    # cases three nodes in a thousand at most (long, flat rows), and one tree's walk in 128 with one of
    # them, which is 0.008 of the accepted depths.
    return {"rel": 1e-6, "max": 5e-6, "differ": 0.01}


# ---------------------------------------------------------------- the same step in 64 bits
def _weights(rows, case):
    """Probabilities of stored rows in 64 bits: as given, or the softmax at the case's temperature."""
    x = rows.double()
    return torch.softmax(x / case["T"], -1) if case["kind"] == "logits" else x


def _pick(w, u):
    """Smallest index whose running sum exceeds u * sum per row; -1 where the row has no mass."""
    c = torch.cumsum(w, -1)
    t = u.double() * c[:, -1]
    v = torch.searchsorted(c, t[:, None], right=True).squeeze(1)
    last = w.shape[1] - 1 - torch.argmax((w > 0).flip(-1).to(torch.uint8), -1)
    return torch.where(c[:, -1] > 0, torch.minimum(v, last), torch.full_like(v, -1))


def _at(w, x):
    return w.gather(1, x[:, None].clamp(min=0)).squeeze(1)


def _without(w, x):
    return w.scatter(1, x[:, None].clamp(min=0), 0.0)


def _draft_nodes(case, stored, u):
    """Drafted tokens [R,k], flags, hub, largest stored element and rest mass of R internal nodes."""
    q = _weights(stored, case)
    largest = stored.float().amax(-1)
    flags = torch.zeros_like(u[:, 0], dtype=torch.int32)
    hub = torch.where(stored.float() == largest[:, None], torch.arange(q.shape[1], device=q.device), q.shape[1]).amin(-1)
    w = q if case["kind"] == "probs" else torch.exp((stored.double() - largest.double()[:, None]) / case["T"])
    tokens = []
    if case["method"] == "spechub":
        rest = _without(w, hub).sum(-1)
        x = _pick(q, u[:, 0])
        y = _pick(_without(q, hub), u[:, 1])
        second = x == hub
        flags += torch.where(second & (y < 0), 1, 0).to(torch.int32)
        y = torch.where(y < 0, hub, y)
        tokens = [torch.where(second, hub, x), torch.where(second, y, hub)]
    else:
        rest = w.sum(-1)
        left, previous = q, torch.zeros_like(hub)
        for i in range(case["k"]):
            x = _pick(left, u[:, i])
            flags |= torch.where(x < 0, 4, 0).to(torch.int32)
            if case["method"] == "rrsw":
                left = torch.where((x >= 0)[:, None], _without(left, x), left)
            previous = torch.where(x < 0, previous, x)
            tokens.append(previous)
        hub = torch.full_like(hub, -1)
    return torch.stack(tokens, 1), flags, hub, largest, rest


def _verify_spechub(p, q, hub, x, u):
    """Alg. 3 on R nodes: outcome, token, flags, residual mass."""
    a = hub
    pa, qa = _at(p, a), _at(q, a)
    rest = _without(q, a).sum(-1)
    c = torch.where(rest > 0, qa / rest, torch.zeros_like(qa))
    first = x[:, 1] == a                                    # the pair is (x, a)
    other = torch.where(first, x[:, 0], x[:, 1])
    po, qo = _at(p, other), _at(q, other)
    p1 = (p - q).clamp(min=0)
    q_ax = _without(q * c[:, None], a)
    S_ax = _without((q_ax - p1).clamp(min=0), a).sum(-1)
    S_xa = _without((q - p).clamp(min=0), a).sum(-1)
    resid = _without((p1 - q_ax).clamp(min=0), a)
    alone = rest <= 0                                       # all draft mass on the hub
    resid = torch.where(alone[:, None], _without(p, a), resid)
    mass = resid.sum(-1)
    take_other = torch.where(first, u[:, 0] * qo < po, u[:, 0] * (c * qo) < (po - qo).clamp(min=0)) & ~alone
    take_hub = torch.where(first, u[:, 1] * S_xa < (pa - S_ax).clamp(min=0), u[:, 1] * S_ax < pa)
    take_hub = torch.where(alone, u[:, 0] * qa < pa, take_hub)
    drawn = _pick(resid, u[:, 2])
    drawn_p = _pick(p, u[:, 2])
    empty = drawn < 0
    slot_other = torch.where(first, 0, 1)
    slot_hub = torch.where(alone, 0, torch.where(first, 1, 0))
    outcome = torch.where(take_other, slot_other, torch.where(take_hub, slot_hub, -1))
    token = torch.where(take_other, other, torch.where(take_hub, a, torch.where(empty & ~alone, drawn_p, drawn)))
    flags = torch.where(alone, 1, 0) + torch.where((outcome < 0) & empty, 2, 0)
    return outcome, token, flags, mass


def _verify_rounds(case, p, q, x, u):
    """Alg. 1 on R nodes, round by round on the distributions themselves."""
    k, without = case["k"], case["method"] == "rrsw"
    outcome = torch.full_like(x[:, 0], -1)
    token = torch.full_like(outcome, -1)
    flags = torch.zeros_like(outcome)
    mass = torch.ones_like(p[:, 0])
    live = torch.ones_like(outcome, dtype=torch.bool)       # still in its rounds
    done = torch.zeros_like(live)                           # accepted
    for i in range(k):
        xi = x[:, i]
        accept = live & (u[:, i] * _at(q, xi) < _at(p, xi))
        outcome = torch.where(accept, i, outcome)
        token = torch.where(accept, xi, token)
        done |= accept
        live &= ~accept
        r = (p - q).clamp(min=0)
        m = r.sum(-1)
        step = live & (m > 0)
        p = torch.where(step[:, None], r / m.clamp(min=1e-300)[:, None], p)
        mass = torch.where(step, mass * m, mass)
        flags |= torch.where(live & (m <= 0), 2, 0)
        if without:
            r = _without(q, xi)
            m = r.sum(-1)
            q = torch.where((live & (m > 0))[:, None], r / m.clamp(min=1e-300)[:, None], q)
            out = live & (m <= 0)
            flags |= torch.where(out, 4, 0)
            live &= ~out
    drawn = _pick(p, u[:, k])
    return outcome, torch.where(done, token, drawn), flags, mass


def _parts(case):
    """Slices of the batch that are worked on at once, and the nodes with and without children."""
    B, children = case["B"], _first_children(case)
    trees = max(1, (1 << 24) // (case["V"] * len(children)))
    inner = torch.tensor([n for n, c in enumerate(children) if c >= 0], device="cuda")
    leaf = torch.tensor([n for n, c in enumerate(children) if c < 0], device="cuda")
    return [slice(b, min(B, b + trees)) for b in range(0, B, trees)], inner, leaf


def _flat(t, part, nodes):
    return t[part].index_select(1, nodes).flatten(0, 1)


def _put(into, part, nodes, value):
    into[part, nodes] = value.view(part.stop - part.start, -1).to(into.dtype)


def _whole(case, value, dtype=torch.int64):
    return torch.full((case["B"], _nodes(case)), value, dtype=dtype, device="cuda")


def _drafted(case, draft, u_draft):
    out = dict(tokens=_whole(case, -1), flags=_whole(case, 0), hub=_whole(case, -1),
               largest=_whole(case, 0, torch.float64), rest=_whole(case, 0, torch.float64))
    parts, inner, _ = _parts(case)
    first = torch.tensor(_first_children(case), device="cuda")[inner]
    for part in parts:
        x, *others = _draft_nodes(case, _flat(draft, part, inner), _flat(u_draft, part, inner))
        for j in range(case["k"]):
            _put(out["tokens"], part, first + j, x[:, j])
        for name, value in zip(("flags", "hub", "largest", "rest"), others):
            _put(out[name], part, inner, value)
    return out


def exact(case, seed):
    state = prepare(case, seed)
    pb, u_v = state["pb"], state["u_verify"]
    B, k = case["B"], case["k"]
    dev = pb.draft.device
    drafted = _drafted(case, pb.draft, state["u_draft"])
    tokens = drafted["tokens"]
    outcome, token, flags = _whole(case, -1), _whole(case, -1), _whole(case, 0)
    mass = _whole(case, 0, torch.float64)
    parts, inner, leaf = _parts(case)
    first = torch.tensor(_first_children(case), device=dev)
    for part in parts:
        p = _weights(_flat(pb.target, part, leaf), case)
        _put(token, part, leaf, _pick(p, _flat(u_v, part, leaf)[:, k]))
        _put(mass, part, leaf, p.sum(-1))
        p, q = (_weights(_flat(rows, part, inner), case) for rows in (pb.target, pb.draft))
        u = _flat(u_v, part, inner).double()
        x = torch.stack([_flat(tokens, part, first[inner] + j) for j in range(k)], 1)
        if case["method"] == "spechub":
            got = _verify_spechub(p, q, _flat(drafted["hub"], part, inner), x, u)
        else:
            got = _verify_rounds(case, p, q, x, u)
        for into, value in zip((outcome, token, flags, mass), got):
            _put(into, part, inner, value)

    # the walk: follow accepted children from the root
    node = torch.zeros(B, dtype=torch.int64, device=dev)
    on = torch.ones(B, dtype=torch.bool, device=dev)
    depth = torch.zeros(B, dtype=torch.int64, device=dev)
    emitted = torch.full((B, case["depth"]), -1, dtype=torch.int64, device=dev)
    seen = torch.zeros_like(tokens, dtype=torch.bool)
    every = torch.arange(B, device=dev)
    for level in range(case["depth"]):
        seen[every, node] |= on
        oc = outcome[every, node]
        emitted[:, level] = torch.where(on, token[every, node], -1)
        on = on & (oc >= 0)
        depth += on
        node = torch.where(on, first[node] + oc, node)
    if case["call"] == "path":
        outcome = torch.where(seen, outcome, -4)
        token = torch.where(seen, token, -1)
        flags = torch.where(seen, flags, 0)

    out = dict(outcome=outcome, token=token, flags=flags, accept_depth=depth, emitted=emitted)
    if case["call"] == "mass":
        return dict(out, resid_mass=mass)
    out.update(tokens=tokens, draft_flags=drafted["flags"])
    if case["method"] == "spechub":
        out["hub"] = drafted["hub"]
    if case["call"] in ("step", "path"):
        out.update(largest=drafted["largest"], rest_mass=drafted["rest"], record_hub=drafted["hub"])
    return out
