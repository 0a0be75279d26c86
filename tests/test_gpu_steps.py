"""StepPlan.run(), which drafts and verifies a node in one kernel where there is one for its rows, against the CPU oracle
at the edges of those kernels, and against the two calls on rows with little or nothing to draw from."""
import ctypes as C

import numpy as np
import pytest
import torch

from paper_2411_05289_amd import binding as B
from paper_2411_05289_amd import workloads as W
from parity import BAND, METHODS, _check_stats, _compare_nodes, _compare_walk, _internal_mask, _np, check_case
from parity import mismatch_allowance, oracle_kwargs, uniforms
from test_gpu_routes import _workload
import oracle

pytestmark = pytest.mark.gpu
DEV = "cuda"
ALL = ["spechub", "rrs", "rrsw"]


def _poison(plan):
    for t in (*plan.out.values(), plan.tokens, plan.draft_flags, plan.hub, plan.pb.draft_stats):
        if t is not None:
            t.fill_(-9)


def _check_step(method, wl, seqs):
    """The drafted tokens are the oracle's except at nodes with a uniform near a boundary; the rest of the step is
    compared with the oracle on the tokens that the step drafted."""
    pb = B.Problem.from_workload(wl)
    u_d, u_v = uniforms(wl, wl.V)
    ok = oracle_kwargs(wl)
    idx = torch.as_tensor(seqs, device=DEV)
    t_np, d_np = W.rows_as_numpy(wl.target[idx]), W.rows_as_numpy(wl.draft[idx])
    o_d = oracle.batch_draft(METHODS[method], d_np, _np(u_d[idx]), temp_draft=wl.temp_draft, nthreads=8, **ok)
    internal = _internal_mask(wl)
    sure = np.zeros((len(seqs), wl.N), dtype=bool)
    first = _np(wl.first_child) if wl.first_child is not None else wl.k * np.arange(wl.N) + 1
    for n in np.nonzero(internal)[0]:
        sure[:, first[n]:first[n] + wl.k] = (o_d["margin"][:, n] >= BAND)[:, None]
    for placement in (True, False):
        plan = B.StepPlan(method, pb, u_d, u_v, walk_in_verify=placement)
        for _ in range(2):
            _poison(plan)
            out = plan.run()
            torch.cuda.synchronize()
            assert not plan.workspace.any()
            tokens = _np(plan.tokens[idx])
            assert (tokens == o_d["tokens"])[sure].all() and (tokens[:, 0] == -1).all()
            assert (_np(plan.draft_flags[idx]) == o_d["flags"])[:, internal].all()
            assert not plan.draft_flags[:, torch.as_tensor(~internal, device=DEV)].any()
            if method == "spechub":
                assert (_np(plan.hub[idx]) == np.where(internal, o_d["hub"], -1)).all()
            _check_stats(wl, _np(plan.pb.draft_stats[idx]), d_np, o_d["hub"] if method == "spechub" else None, internal)
            o_v = oracle.batch_verify(METHODS[method], t_np, d_np, tokens, _np(u_v[idx]), temp_target=wl.temp_target,
                                      temp_draft=wl.temp_draft, nthreads=8, **ok)
            near = o_v["margin"] < BAND
            ctx = dict(method=method, wl=wl, t_np=t_np, d_np=d_np, tokens=tokens, uv=_np(u_v[idx]))
            assert _compare_nodes(out, o_v, idx, near, "step", ctx) <= mismatch_allowance(near)
            _compare_walk(wl, out, o_v, idx, near)


@pytest.mark.parametrize("method,k", [("spechub", 2), ("rrs", 2), ("rrsw", 2), ("rrs", 5), ("rrsw", 4), ("rrsw", 1)])
@pytest.mark.parametrize("dtype,V,off,Bn", [
    ("bf16", 8185, 0, 5), ("bf16", 16369, 0, 5), ("fp32", 8188, 0, 5), ("fp32", 4101, 3, 5),  # four chunks per lane
    ("bf16", 16384, 0, 5), ("bf16", 32737, 7, 5), ("fp32", 16380, 0, 5),                      # eight
    ("bf16", 32768, 0, 5), ("bf16", 65521, 1, 5), ("fp32", 20001, 2, 5),                      # sixteen, drafted from memory
    ("bf16", 9001, 3, 1000), ("fp32", 16384, 0, 1000), ("bf16", 16400, 0, 1000),              # 256 threads per node
    ("bf16", 2049, 0, 5), ("bf16", 4081, 3, 5), ("fp32", 1021, 2, 5), ("fp32", 2041, 1, 5),     # 128
    ("bf16", 4089, 0, 5), ("bf16", 8177, 5, 5), ("fp32", 4085, 3, 5),                         # 256, four chunks
    ("bf16", 32768, 0, 200), ("bf16", 65521, 1, 200),                                         # 512, sixteen
])
def test_rows_in_registers(method, k, dtype, V, off, Bn):
    wl = _workload(Bn, W.tree_nodes(k, 2), V, k, 2, dtype, "logits", off)
    _check_step(method, wl, range(Bn) if Bn < 9 else [0, 1, 7, 8, Bn - 1])


@pytest.mark.parametrize("method,k", [("spechub", 2), ("rrs", 2), ("rrsw", 3)])
@pytest.mark.parametrize("dtype,V,off,Bn", [
    ("bf16", 65600, 0, 3), ("bf16", 131073, 3, 3), ("bf16", 163000, 1, 3), ("fp32", 70001, 1, 3),  # 1024 threads, up to 20 chunks
    ("bf16", 66001, 1, 800), ("fp32", 33001, 0, 800), ("bf16", 200000, 0, 3),                      # from memory
])
def test_long_rows(method, k, dtype, V, off, Bn):
    wl = _workload(Bn, W.tree_nodes(k, 2), V, k, 2, dtype, "logits", off)
    _check_step(method, wl, range(Bn) if Bn < 9 else [0, 1, Bn - 1])


@pytest.mark.parametrize("method,k", [("spechub", 2), ("rrs", 2), ("rrsw", 2), ("rrsw", 4)])
@pytest.mark.parametrize("dtype,V,off,nodes", [
    ("bf16", 32000, 0, 300), ("bf16", 50304, 0, 300), ("bf16", 131080, 0, 300), ("bf16", 140001, 1, 300),  # 1024 threads
    ("bf16", 152064, 0, 30), ("bf16", 152064, 0, 300), ("bf16", 152064, 0, 600), ("fp32", 20000, 0, 300), ("fp32", 70000, 0, 300),
    ("bf16", 50304, 0, 600), ("bf16", 131080, 0, 600),
    ("fp32", 7000, 0, 3000), ("fp32", 7001, 1, 3000), ("bf16", 9000, 0, 3000),                             # 256, eight chunks
    ("bf16", 20001, 3, 3000), ("fp32", 12000, 0, 3000), ("fp32", 12001, 3, 3000),                          # ... sixteen
    ("bf16", 6000, 0, 30), ("fp32", 3000, 0, 30), ("fp32", 1500, 0, 30),                                   # ... four; 128
    ("bf16", 20001, 1, 900), ("fp32", 12001, 1, 900), ("fp32", 20001, 1, 600), ("fp32", 20000, 0, 600),    # 512
    ("fp32", 33001, 0, 1400), ("fp32", 66000, 0, 2800),                                                    # ... from memory
    ("fp32", 12001, 1, 300), ("fp32", 40001, 1, 300), ("fp32", 70001, 1, 300),                             # 1024, unaligned
])
def test_builds_by_batch_size(method, k, dtype, V, off, nodes):
    """Batches that take another number of threads per node than the smallest ones."""
    N = W.tree_nodes(k, 3)
    Bn = -(-nodes // N)
    _check_step(method, _workload(Bn, N, V, k, 3, dtype, "logits", off), [0, Bn // 2, Bn - 1])


@pytest.mark.parametrize("method,k", [("spechub", 2), ("rrs", 2), ("rrs", 7), ("rrsw", 3), ("rrsw", 8), ("rrs", 1)])
@pytest.mark.parametrize("V,dtype,Bn", [(16, "fp32", 1), (50, "fp32", 17), (60, "bf16", 700), (200, "bf16", 401),
                                        (1025, "bf16", 9), (2041, "bf16", 33), (1019, "fp32", 9), (50, "fp32", 30001),
                                        (600, "bf16", 9000)])
def test_short_rows(method, k, V, dtype, Bn):
    """Groups of 4 to 64 lanes: whole trees in a workgroup, a wavefront per node number, nodes in any order."""
    for depth in (2, 3) if k == 2 and Bn < 9000 else (2,):
        wl = _workload(Bn, W.tree_nodes(k, depth), V, k, depth, dtype, "logits", off=1)
        _check_step(method, wl, sorted({0, Bn // 2, Bn - 1}))


@pytest.mark.parametrize("method", ALL)
@pytest.mark.parametrize("what", ["step", "logits", "probs"])
@pytest.mark.parametrize("dtype,V,depth,Bn", [
    ("bf16", 16, 2, 1), ("bf16", 16, 4, 1), ("bf16", 16, 4, 1101),      # 4 lanes per node: a wavefront per node number, whole
    ("bf16", 30, 2, 1), ("bf16", 30, 4, 1), ("bf16", 240, 4, 1101),     # trees in a workgroup, nodes in any order; 8 lanes
    ("bf16", 60, 2, 1), ("bf16", 60, 4, 1), ("bf16", 250, 4, 1101),     # 16
    ("bf16", 250, 2, 700), ("bf16", 250, 4, 1), ("bf16", 900, 5, 201),  # 32
    ("bf16", 250, 2, 1), ("bf16", 250, 5, 1),                           # 64, no wavefront per node number
    ("fp32", 16, 2, 1), ("fp32", 16, 4, 1), ("fp32", 16, 4, 1101),
    ("fp32", 14, 2, 1), ("fp32", 14, 4, 1), ("fp32", 100, 4, 1101),
    ("fp32", 30, 2, 1), ("fp32", 30, 4, 1), ("fp32", 250, 4, 1101),
    ("fp32", 100, 2, 1), ("fp32", 100, 4, 1), ("fp32", 400, 5, 201),
    ("fp32", 250, 2, 1), ("fp32", 400, 4, 1),
])
def test_every_group(method, what, dtype, V, depth, Bn):
    """Short rows: every number of lanes with every way of walking the trees."""
    wl = _workload(Bn, W.tree_nodes(2, depth), V, 2, depth, dtype, "probs" if what == "probs" else "logits")
    seqs = sorted({0, Bn // 2, Bn - 1})
    if what == "step":
        _check_step(method, wl, seqs)
    else:
        check_case(method, wl, seed=V, seqs=seqs, full_outputs=Bn < 999)


@pytest.mark.parametrize("method", ALL)
@pytest.mark.parametrize("V,dtype,Bn", [(9001, "bf16", 5), (33000, "bf16", 3), (9001, "bf16", 200), (50, "fp32", 33),
                                        (60, "bf16", 2015), (3000, "bf16", 5), (70001, "bf16", 3), (70001, "bf16", 150)])
def test_trees_given_by_a_table(method, V, dtype, Bn):
    wl = _workload(Bn, 9, V, 2, 5, dtype, "logits", first_child=[1, 3, -1, 5, -1, 7, -1, -1, -1])
    _check_step(method, wl, range(Bn) if Bn < 9 else [0, 1, Bn - 1])


@pytest.mark.parametrize("method,k", [("spechub", 2), ("rrs", 3), ("rrsw", 3)])
@pytest.mark.parametrize("dtype,V,off", [("bf16", 9001, 3), ("bf16", 20000, 0), ("bf16", 40001, 1), ("fp32", 9000, 0),
                                        ("bf16", 60, 0), ("fp32", 999, 1), ("bf16", 3001, 5), ("bf16", 170001, 1)])
def test_rows_with_little_to_draw_from(method, k, dtype, V, off):
    """One token with all the draft mass, as many as there are drafts, none, tokens at the type's lowest value, a NaN, a
    +inf, target rows with a single token: what the two calls give, flags and records included."""
    Bn, N = 12, W.tree_nodes(k, 2)
    wl = _workload(Bn, N, V, k, 2, dtype, "logits", off)
    low = torch.finfo(wl.draft.dtype).min
    d, t = wl.draft, wl.target
    d[0], d[1], d[2], d[3] = -torch.inf, -torch.inf, -torch.inf, low
    d[0, :, V - 3] = 1.0
    d[1, :, 5:5 + k] = 2.0
    d[3, :, ::97] = 3.0
    d[4, :, 0] = torch.nan
    d[5, :, V - 1] = torch.nan
    d[6, :, 7] = torch.inf
    t[7] = -torch.inf
    t[7, :, 11] = 0.0
    t[8] = low
    t[8, :, V // 2] = 0.0
    d[9], t[9] = -torch.inf, -torch.inf
    d[9, :, 3] = t[9, :, 4] = 0.0
    d[10] = -torch.inf
    d[10, :, 0] = 0.0
    pb = B.Problem.from_workload(wl)
    u_d, u_v = uniforms(wl, 3)
    plan = B.StepPlan(method, pb, u_d, u_v)
    names = ("outcome", "token", "flags", "accept_depth", "emitted")
    _poison(plan)
    plan.draft()
    plan._verify_walk(B._stream())
    torch.cuda.synchronize()
    want = {n: plan.out[n].clone() for n in names}
    drafted = (plan.tokens.clone(), plan.draft_flags.clone(), plan.hub.clone())
    records = plan.pb.draft_stats.clone()
    _poison(plan)
    out = plan.run()
    torch.cuda.synchronize()
    for got, w in zip((plan.tokens, plan.draft_flags, plan.hub), drafted):
        assert torch.equal(got, w)
    for n in names:
        assert torch.equal(out[n], want[n]), n
    got = plan.pb.draft_stats
    assert torch.equal(got.view(torch.int32)[..., 2], records.view(torch.int32)[..., 2])
    # sums of V positive terms in another order
    assert torch.allclose(got[..., :2], records[..., :2], rtol=2e-6, atol=0.0, equal_nan=True)


def test_what_run_refuses():
    """run() reports what draft() or the verify call would refuse, by the name of that call."""
    wl = _workload(2, 3, 9000, 2, 2, "bf16", "logits")
    u_d, u_v = uniforms(wl, 1)
    for field, value, name in (("temp_draft", 0.0, "spechub_draft"), ("temp_target", 0.0, "spechub_verify"),
                               ("depth", 3, "spechub_draft")):
        plan = B.StepPlan("spechub", B.Problem.from_workload(wl), u_d, u_v)
        setattr(plan._cp, field, value)
        with pytest.raises(B.MdsdError, match=name):
            plan.run()
    no_records = B.StepPlan("spechub", B.Problem.from_workload(wl), u_d, u_v, hand_stats=False)
    with_records = B.StepPlan("spechub", B.Problem.from_workload(wl), u_d, u_v)
    for key, got in no_records.run().items():
        assert torch.equal(got, with_records.run()[key])


@pytest.mark.parametrize("method", ALL)
@pytest.mark.parametrize("V,dtype", [(60, "bf16"), (3000, "bf16"), (9001, "bf16"), (70001, "bf16"), (33000, "fp32")])
def test_trees_of_one_node_and_steps_without_a_walk(method, V, dtype):
    """A tree that is its root drafts nothing; the C calls may leave the walk out."""
    wl = _workload(5, 1, V, 2, 1, dtype, "logits")
    _check_step(method, wl, range(5))
    wl = _workload(5, 7, V, 2, 3, dtype, "logits")
    u_d, u_v = uniforms(wl, 2)
    plan = B.StepPlan(method, B.Problem.from_workload(wl), u_d, u_v)
    want = {n: t.clone() for n, t in plan.run().items()}
    _poison(plan)
    hub = [plan.hub.data_ptr()] if method == "spechub" else []
    args = [u_d.data_ptr(), u_v.data_ptr(), plan.tokens.data_ptr(), *hub, plan.draft_flags.data_ptr()]
    rc = getattr(B.lib(), method + "_step")(C.byref(plan._cp), *args, C.byref(plan._res), None, 0, B._stream())
    torch.cuda.synchronize()
    assert rc == 0
    for n in ("outcome", "token", "flags"):
        assert torch.equal(plan.out[n], want[n]), n
    assert (plan.out["accept_depth"] == -9).all() and (plan.out["emitted"] == -9).all()


def _both(method, wl, seed):
    """What run() leaves and what draft() and the verify call leave, as dicts of tensors."""
    u_d, u_v = uniforms(wl, seed)
    plan = B.StepPlan(method, B.Problem.from_workload(wl), u_d, u_v)
    sides = []
    for call in (plan.run, lambda: (plan.draft(), plan.verify_and_walk())):
        _poison(plan)
        call()
        torch.cuda.synchronize()
        records = plan.pb.draft_stats
        left = dict(plan.out, tokens=plan.tokens, draft_flags=plan.draft_flags, largest=records[..., 0], rest=records[..., 1],
                    record_hub=records.view(torch.int32)[..., 2])
        if method == "spechub":
            left["hub"] = plan.hub
        sides.append({n: t.clone() for n, t in left.items() if t is not None})
    return sides


@pytest.mark.parametrize("method,k", [("spechub", 2), ("rrs", 2), ("rrsw", 2), ("rrs", 3), ("rrsw", 4)])
@pytest.mark.parametrize("dtype,V,off,nodes", [
    ("bf16", 2100, 0, 900), ("bf16", 7001, 3, 900), ("bf16", 9001, 1, 900), ("bf16", 12000, 0, 3300), ("fp32", 7001, 2, 3300),
    ("bf16", 20001, 1, 300), ("bf16", 32000, 0, 380), ("bf16", 20001, 0, 3300), ("bf16", 50304, 0, 300), ("bf16", 42001, 1, 900),
    ("fp32", 20001, 1, 300), ("bf16", 70001, 1, 400), ("bf16", 128256, 0, 300), ("bf16", 152064, 0, 300), ("bf16", 131073, 3, 900),
])
def test_drafts_of_a_step(method, k, dtype, V, off, nodes):
    """Rows of more than 256 chunks: the tokens, flags and records of the draft call, bit for bit."""
    N = W.tree_nodes(k, 3)
    one, two = _both(method, _workload(max(1, nodes // N), N, V, k, 3, dtype, "logits", off, seed=V), 6)
    for n in ("tokens", "draft_flags", "largest", "rest", "record_hub", "hub"):
        if n in one:
            assert torch.equal(one[n], two[n]), n


@pytest.mark.parametrize("method,k,depth,dtype,V,Bn", [
    ("spechub", 2, 4, "bf16", 60, 1500), ("rrs", 2, 4, "bf16", 60, 1500), ("rrsw", 3, 3, "bf16", 60, 1700),  # 4 lanes, drafted with 8 or 16
    ("spechub", 2, 4, "fp32", 50, 900), ("rrsw", 2, 4, "fp32", 50, 900),                                     # 8 and 16
    ("spechub", 2, 4, "bf16", 1000, 400), ("rrs", 4, 3, "bf16", 1000, 400), ("rrsw", 2, 2, "bf16", 250, 1500),
    ("rrs", 2, 4, "fp32", 20000, 24), ("rrs", 3, 3, "fp32", 32000, 50),                                      # 1024 threads, drafted from memory
])
def test_steps_within_rounding(method, k, depth, dtype, V, Bn):
    """Where the sums of the draft call are formed in another order: what both leave is the same except where a uniform lies
    within rounding of a boundary."""
    N = W.tree_nodes(k, depth)
    one, two = _both(method, _workload(Bn, N, V, k, depth, dtype, "logits", seed=V), 8)
    # A row's V boundaries move by less than 2^-25 each (half an ulp of sums that are mostly far from the largest), so that of
    # `nodes` nodes with k + 1 draws and k tests fewer than 2 (2 k + 1) V 2^-25 find a uniform on the other side; each changes its tree
    # only.  (Counted at V = 32000: one in 2600 nodes, a 25th of that.)  One tree more, for the batches in which that is none.
    expected = 2.0 ** -24 * (2 * k + 1) * V * Bn * N
    other = torch.zeros(Bn, dtype=torch.bool, device=DEV)
    for n in ("outcome", "token", "flags", "tokens", "draft_flags", "accept_depth", "emitted"):
        other |= (one[n] != two[n]).view(Bn, -1).any(1)
    assert int(other.sum()) <= 1 + expected
    for n in ("largest", "record_hub", "hub"):
        if n in one:
            assert torch.equal(one[n], two[n]), n
    # sums of V positive terms in another order
    assert torch.allclose(one["rest"], two["rest"], rtol=2e-6, atol=0.0)


@pytest.mark.parametrize("method,V,k,depth,Bn", [
    ("rrs", 42001, 1, 5, 170),       # sixteen chunks per lane, 680 nodes with children: one launch would take 1.13 times as long
    ("rrsw", 65500, 2, 5, 42),       # ... 630, 1.10
    ("rrs", 70001, 1, 5, 170),       # longer rows on 1024 threads, 850 nodes: 1.30
    ("rrs", 100000, 1, 5, 140),      # ... 700 nodes: 1.14
    ("rrs", 100001, 3, 3, 131),      # ... 1703 nodes: 1.15
])
def test_one_call_is_not_slower_than_two(method, V, k, depth, Bn):
    """Where the nodes with children fill a little more than the chip holds of a step kernel."""
    wl = _workload(Bn, W.tree_nodes(k, depth), V, k, depth, "bf16", "logits")
    u_d, u_v = uniforms(wl, 4)
    plan = B.StepPlan(method, B.Problem.from_workload(wl), u_d, u_v)
    assert plan.walk_in_verify
    st = B._stream()

    def two():
        plan.draft(st)
        plan.verify_and_walk(st)

    def run():
        plan.run(st)

    best = {two: float("inf"), run: float("inf")}
    for _ in range(12):
        for call in best:
            begin, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            begin.record()
            for _ in range(40):
                call()
            end.record()
            end.synchronize()
            best[call] = min(best[call], begin.elapsed_time(end))
    # runs of one side differ by less than 2 %
    assert best[run] < 1.04 * best[two], (best[run], best[two])
