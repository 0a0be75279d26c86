"""Verify calls at the edges of their routes: rows of probabilities that are streamed with several chunks asked for
ahead, small trees with a wavefront per node, trees given by a table, and softmax shifts so large that they do not take
every whole number."""
import pytest
import torch

from paper_2411_05289_amd import binding as B
from paper_2411_05289_amd import workloads as W
from parity import DRAFT, VERIFY, check_case

pytestmark = pytest.mark.gpu
DEV = "cuda"
ALL = ["spechub", "rrs", "rrsw"]


def _workload(Bn, N, V, k, depth, dtype, kind, off=0, temps=(0.9, 1.2), first_child=None, seed=5):
    td = torch.float32 if dtype == "fp32" else torch.bfloat16
    t, d = W.llm_like_logits(Bn, N, V, logit_std=2.0, draft_noise_std=1.0, dtype=torch.float32, seed=seed, device=DEV)
    if kind == "probs":
        t, d = torch.softmax(t.double(), -1), torch.softmax(d.double(), -1)
        temps = (1.0, 1.0)
    rows = []
    for x in (t, d):
        buf = torch.zeros((Bn * N * V + off,), dtype=td, device=DEV)
        view = buf[off:].view(Bn, N, V)
        view.copy_(x)
        rows.append(view)
    if first_child is not None:
        first_child = torch.tensor(first_child, dtype=torch.int32, device=DEV)
    return W.Workload("routes", Bn, N, V, k, depth, dtype, kind, temps[0], temps[1], rows[0], rows[1],
                      first_child=first_child)


@pytest.mark.parametrize("method", ALL)
@pytest.mark.parametrize("dtype,V,off,Bn", [
    ("fp32", 4097, 0, 3),       # the shortest rows of eight wavefronts, in registers
    ("fp32", 8101, 3, 3),
    ("fp32", 5601, 1, 87),      # streamed: 261 nodes of more than 1400 chunks
    ("fp32", 9001, 0, 3),       # ... the shortest that always are
    ("fp32", 16384, 0, 3),      # eight slabs per wavefront, the last one full
    ("fp32", 16385, 0, 3),      # ... and one slab of one chunk more
    ("fp32", 18433, 3, 3),      # ... and one each, rows that begin inside a chunk
    ("fp32", 50001, 1, 3),
    ("bf16", 9001, 5, 3),       # in registers
    ("bf16", 9001, 5, 171),     # streamed: 513 nodes
    ("bf16", 14001, 3, 86),     # ... 258 nodes of longer rows
    ("bf16", 9001, 5, 260),     # in registers: more than 768 nodes
    ("bf16", 32768, 0, 3),
    ("bf16", 33281, 7, 3),
])
def test_streamed_probabilities(method, dtype, V, off, Bn):
    wl = _workload(Bn, 3, V, 2, 2, dtype, "probs", off)
    check_case(method, wl, seed=V, seqs=None if Bn < 9 else [0, 1, Bn - 1], full_outputs=Bn < 9)


@pytest.mark.parametrize("method,k", [("spechub", 2), ("rrs", 2), ("rrsw", 3), ("rrsw", 4), ("rrs", 7)])
@pytest.mark.parametrize("V,dtype,Bn", [(16, "fp32", 1), (50, "fp32", 17), (60, "bf16", 700), (200, "bf16", 401),
                                        (500, "bf16", 203), (450, "fp32", 101), (50, "fp32", 30001)])
def test_a_wavefront_per_node(method, k, V, dtype, Bn):
    """Trees of 3, 4, 5, 7 and 8 nodes; the last workgroup short of trees; large batches of small rows."""
    for depth in (2, 3) if k == 2 and Bn < 9999 else (2,):
        wl = _workload(Bn, W.tree_nodes(k, depth), V, k, depth, dtype, "logits")
        check_case(method, wl, seed=V, seqs=sorted({0, Bn // 2, Bn - 1}), full_outputs=Bn < 9999)


@pytest.mark.parametrize("method", ALL)
@pytest.mark.parametrize("V,dtype,Bn", [(50, "fp32", 33), (600, "bf16", 9), (3000, "bf16", 5), (9001, "bf16", 5),
                                        (70001, "bf16", 3)])
def test_tables_node_by_node(method, V, dtype, Bn):
    """Trees of seven nodes (a wavefront each where the rows are short) and nine."""
    for fc in ([1, 3, 5, -1, -1, -1, -1], [1, 3, -1, 5, -1, 7, -1, -1, -1]):
        wl = _workload(Bn, len(fc), V, 2, 5, dtype, "logits", first_child=fc)
        check_case(method, wl, seed=V, full_outputs=V < 9999)


@pytest.mark.parametrize("method", ALL)
@pytest.mark.parametrize("V,dtype,Bn", [(50, "fp32", 2003), (17, "fp32", 2001), (60, "bf16", 2015), (60, "bf16", 7300),
                                        (110, "fp32", 2003), (8000, "fp32", 1400), (30000, "bf16", 1500)])
def test_tables_of_large_batches(method, V, dtype, Bn):
    """Nine-node trees beyond the workgroups that walk them: a wavefront per node number of sixteen trees, the last ones short
    of trees; node by node; tree by tree where the rows are 400 and 800 MB."""
    wl = _workload(Bn, 9, V, 2, 5, dtype, "logits", first_child=[1, 3, -1, 5, -1, 7, -1, -1, -1])
    check_case(method, wl, seed=V, seqs=[0, 1, 15, 16, Bn // 2, Bn - 2, Bn - 1], full_outputs=V < 999)


@pytest.mark.parametrize("method", ALL)
@pytest.mark.parametrize("records", [True, False])
@pytest.mark.parametrize("step,shift", [(8.0, 2.0 ** 20), (8.0, -2.0 ** 23), (8.0, 2.0 ** 26), (8.0, 15e6 * 8), (8.0, -16e6 * 8),
                                        (16.0, -15e6 * 16), (64.0, 15e6 * 64), (64.0, -16e6 * 64)])
def test_large_softmax_shifts(method, step, shift, records):
    """Logits that are whole multiples of a step, at T = 8, and the same logits (exactly, in fp32) far from 0, where the
    softmax shift takes large values, 1.9e5 to 1.2e7 and, from 15e6 steps on, 2^24.4 to 2^27.5, where it does not take every
    whole number: the same outcomes, tokens and residual masses."""
    wl = _workload(4, 3, 9000, 2, 2, "fp32", "logits")
    u = torch.rand((4, 3, 3), generator=torch.Generator(device=DEV).manual_seed(1), device=DEV)
    results = []
    for by in (0.0, shift):
        t, d = (torch.round(x) * step + by for x in (wl.target, wl.draft))
        assert torch.equal(t - by, torch.round(wl.target) * step)
        pb = B.Problem(t, d, B.LOGITS, 2, 2, 8.0, 8.0)
        if records:
            pb = pb.with_draft_stats()
        drafted = DRAFT[method](pb, u[..., :2].contiguous())
        results.append((drafted["tokens"][:, 1:], VERIFY[method](pb, drafted["tokens"], u, resid_mass=True)))
    (tokens, want), (tokens_far, got) = results
    assert torch.equal(tokens, tokens_far)
    for name in ("outcome", "token", "flags"):
        assert torch.equal(want[name], got[name]), name
    # the parity bar's bound for residual masses
    assert ((want["resid_mass"] - got["resid_mass"]).abs() <= 1e-5 * want["resid_mass"] + 5e-7).all()


@pytest.mark.parametrize("method", ALL)
@pytest.mark.parametrize("dtype,V,off,Bn", [
    ("bf16", 9000, 0, 3), ("bf16", 9001, 3, 3),                 # 512 threads per node, four chunks per lane
    ("bf16", 32000, 0, 3), ("bf16", 32001, 5, 3),               # ... eight; 1024 threads where unaligned
    ("fp32", 32000, 0, 3), ("fp32", 32001, 1, 3),               # ... sixteen; 1024 threads
    ("bf16", 50304, 0, 3), ("bf16", 70001, 1, 3),               # 1024 threads, resident and streamed
    ("bf16", 32000, 0, 768), ("bf16", 32001, 0, 768),           # 256 threads
])
def test_target_rows_far_from_zero(method, dtype, V, off, Bn):
    """Softmax shifts of 2^24 and more, which do not take every whole number, up to the bound of a usable reference, 2^31:
    target rows of one mask value throughout are uniform, and a temperature near 0 leaves the largest element."""
    for fill, T in ((-3e8, 1.0), (-1e9, 1.0), (-1e9, 0.7), (2e7, 1.0)):
        wl = _workload(Bn, 3, V, 2, 2, dtype, "logits", off, temps=(T, 1.0))
        wl.target[::2] = fill
        check_case(method, wl, seed=V, seqs=[0, 1, Bn - 1], full_outputs=Bn < 9)
    if dtype == "fp32":  # largest logits of 5 to 9: shifts of 2^29.4 and more
        check_case(method, _workload(Bn, 3, V, 2, 2, dtype, "logits", off, temps=(1e-8, 1.0)), seed=V)


@pytest.mark.parametrize("method", ALL)
@pytest.mark.parametrize("dtype,V", [("bf16", 9000), ("bf16", 32000), ("bf16", 32001), ("fp32", 32000), ("bf16", 50304)])
def test_acceptance_of_flat_rows(method, dtype, V):
    """The probability that the first acceptance test holds a token's p(x) to be, on flat target rows (the exponents
    of their weights relative to the largest are small, relative to their sum they are not): the root's first test is u q(x) <
    p(x) with q(x) = 1/2 exactly, so the uniforms between which it changes give p(x), here for 64 of the likelier tokens."""
    X, steps = 64, 48
    gen = torch.Generator(device=DEV).manual_seed(V)
    td = torch.float32 if dtype == "fp32" else torch.bfloat16
    target = (0.5 * torch.randn((X, 3, V), generator=gen, device=DEV)).to(td)
    p = torch.softmax(target[:, 0].double(), -1)
    likely = p[:, 1:].topk(200, -1).indices + 1
    x = likely[torch.arange(X, device=DEV), torch.randint(200, (X,), generator=gen, device=DEV)]
    # the draft's mass lies on token 0, the hub, and on x in equal parts
    draft = torch.full((X, 3, V), -torch.inf, dtype=td, device=DEV)
    draft[..., 0] = 0.0
    draft.scatter_(2, x[:, None, None].expand(X, 3, 1), 0.0)
    tokens = torch.full((X, 3), -1, dtype=torch.int32, device=DEV)
    tokens[:, 1], tokens[:, 2] = x, 0
    pb = B.Problem(target, draft, B.LOGITS, 2, 2, 1.0, 1.0).with_draft_stats()
    DRAFT[method](pb, torch.rand((X, 3, 2), generator=gen, device=DEV))
    exact = 2 * p[torch.arange(X, device=DEV), x]
    accepted = torch.zeros(X, dtype=torch.int64, device=DEV)
    offsets = (torch.arange(steps, device=DEV) - steps // 2 + 0.5) * 4e-8
    for off in offsets:
        u = torch.full((X, 3, 3), 0.5, device=DEV)
        u[:, 0, 0] = (exact * (1 + off)).float()
        accepted += VERIFY[method](pb, tokens, u)["outcome"][:, 0] == 0
    assert ((accepted > 0) & (accepted < steps)).all()
    error = (accepted - steps // 2).double() * 4e-8
    # In units of 2^-24 = 6e-8, root mean squares: the exponent, of up to 4 in magnitude, is rounded by 1.4 at most, 0.8, the
    # exponential by 0.6, the reciprocal of the sum and the product by 0.6 each, u and its product by 0.6, the grid of
    # offsets by 0.2: 1.5, or 0.9e-7; and as much again for the sum itself.  (Measured: 0.7e-7 to 1.0e-7.)
    assert error.square().mean().sqrt() < 1.3e-7, error.square().mean().sqrt()
