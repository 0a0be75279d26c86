"""Draft calls at the edges of their kernels: how many wavefronts share a node and its draws, how a row's largest
element is found, and where rows begin and end; draws, in draft and verify calls, at the edges of tokens without weight."""
import numpy as np
import pytest
import torch

from paper_2411_05289_amd import binding as B
from paper_2411_05289_amd import workloads as W
from parity import DRAFT, METHODS, _np, check_case, oracle_kwargs, uniforms
import oracle

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("method,k", [("spechub", 2), ("rrs", 2), ("rrs", 8), ("rrsw", 3), ("rrsw", 8)])
@pytest.mark.parametrize("dtype,V", [("bf16", 2100), ("bf16", 4089), ("bf16", 4097), ("bf16", 8186), ("bf16", 16369),
                                     ("bf16", 32737), ("bf16", 32768), ("bf16", 66000), ("fp32", 4091), ("fp32", 16380),
                                     ("fp32", 33000)])
def test_draws_of_every_wave(method, k, dtype, V):
    """Two, four, eight and sixteen wavefronts per node, up to eight draws: more draws than wavefronts, as many, fewer;
    rows in registers and streamed, the last slab full and nearly empty.  Tokens, hub and flags are the oracle's
    except where a uniform lies within 1e-6 of a boundary; the records to fp32 rounding."""
    wl = W.config(3 if dtype == "bf16" else 2, device=DEV, B=3, V=V, k=k, depth=2, seed=V + k)
    pb = B.Problem.from_workload(wl).with_draft_stats()
    u_d, _ = uniforms(wl, V)
    g = DRAFT[method](pb, u_d)
    rows = W.rows_as_numpy(wl.draft)
    o = oracle.batch_draft(METHODS[method], rows, _np(u_d), temp_draft=wl.temp_draft, nthreads=8, **oracle_kwargs(wl))
    sure = o["margin"][:, 0] > 1e-6
    assert sure.any()
    assert (_np(g["tokens"])[sure] == o["tokens"][sure]).all()
    assert (_np(g["flags"]) == o["flags"]).all()
    x = wl.draft[:, 0].double()
    w = torch.exp((x - x.amax(-1, keepdim=True)) / wl.temp_draft)
    mass = w.sum(-1)
    if method == "spechub":
        assert (_np(g["hub"]) == o["hub"]).all()
        mass = mass - 1.0        # the hub's weight is 1
    rec = pb.draft_stats[:, 0]
    assert torch.equal(rec[:, 0].double(), x.amax(-1))
    # a sum of V positive terms, each within 1e-6 (exponent and exp), added in trees and short chains
    assert ((rec[:, 1].double() - mass).abs() <= 2e-6 * mass).all()


@pytest.mark.parametrize("V,off", [(4104, 0), (4101, 3), (9001, 5), (32760, 0), (32741, 1)])
def test_largest_element_of_bf16_rows(V, off):
    """Rows whose largest element is positive, rows of negative numbers only (log-probabilities), rows with -0 or with
    most tokens at -inf, and rows with NaNs of either sign among their numbers: the record's largest element and
    the hub (its lowest index) are those of the numbers."""
    gen = torch.Generator(device=DEV).manual_seed(V)
    N = 3
    buf = torch.zeros(6 * N * V + 16, dtype=torch.bfloat16, device=DEV)
    rows = buf[off:off + 6 * N * V].view(6, N, V)
    x = torch.randn((6, N, V), generator=gen, device=DEV) * 3
    x[1] -= 100.0
    x[2] = torch.where(x[2] > -3, -0.0, x[2] - 5)          # all negative or -0
    x[3] = torch.where(torch.rand((N, V), generator=gen, device=DEV) < 0.999, -torch.inf, x[3] - 50)
    x[3, :, V - 1] = -60.0
    nan = torch.rand((2, N, V), generator=gen, device=DEV) < 0.01
    x[4][nan[0]] = torch.nan
    x[5] -= 100.0
    rows.copy_(x)
    bits = rows[5].view(torch.int16)
    bits[nan[1]] = -2                                       # 0xfffe: a negative NaN
    pb = B.Problem(None, rows, B.LOGITS, 2, 2).with_draft_stats()
    g = B.spechub_draft(pb, torch.rand((6, N, 2), generator=gen, device=DEV))
    numbers = torch.nan_to_num(rows.float(), nan=-torch.inf)
    want = numbers.amax(-1)
    assert torch.equal(pb.draft_stats[:, 0, 0], want[:, 0])
    first = torch.where(numbers == want[..., None], torch.arange(V, device=DEV), V).amin(-1)
    assert torch.equal(g["hub"][:, 0].long(), first[:, 0])


def _rounded_boundaries(count, seed):
    """Vectors of 64 weights, half of them 0, with a uniform u for which u * total lies between the running sums in
    front of and behind a weight of 0: the sums are formed as a wavefront forms them, lanes 1, 2, 4 and 8 below in rows of
    16, then row by row, and may differ by a rounding there."""
    f = np.float32

    def running(v):
        v = v.copy()
        for k in (1, 2, 4, 8):
            below = np.zeros((4, 16), f)
            below[:, k:] = v.reshape(4, 16)[:, :16 - k]
            v = v + below.reshape(64)
        v[16:32] += v[15]
        v[48:] += v[47]
        v[32:] += v[31]
        return v

    rng = np.random.default_rng(seed)
    weights, us = [], []
    while len(us) < count:
        v = np.where(rng.random(64) < 0.5, rng.random(64) / 32, 0.0).astype(f)
        v[[0, 63]] = f(0.03125)
        r = running(v)
        for n in np.nonzero((v[1:] == 0) & (r[1:] > r[:-1]))[0]:
            near = f(r[n] / r[63])
            for u in (near, np.nextafter(near, f(1)), np.nextafter(near, f(0))):
                if r[n] <= u * r[63] < r[n + 1] and len(us) < count:
                    weights.append(v)
                    us.append(u)
                    break
    return np.stack(weights), np.array(us, f)


@pytest.mark.parametrize("method", ["spechub", "rrs", "rrsw"])
@pytest.mark.parametrize("V,stride", [(16384, 256), (16384, 4), (4864, 4), (40000, 256)])
def test_draws_at_rounded_boundaries(method, V, stride):
    """Rows with one token in every second slab or lane, and uniforms at which the running sums exceed the threshold at a
    slab or lane without weight: draft draws, leaves and residuals (draft mass on tokens that the target lacks, so that the
    residual is the target's row) give a token with weight next to the threshold, and no flag."""
    Bn = 64
    weights, us = _rounded_boundaries(Bn, V + stride)
    row = np.zeros((Bn, V), np.float32)
    row[:, :64 * stride:stride] = weights
    rows = torch.from_numpy(row).to(DEV)[:, None].expand(Bn, 3, V).contiguous()
    u = torch.from_numpy(us).to(DEV)
    other = torch.zeros_like(rows)
    other[..., 1:3] = 0.5           # the hub and one token more, without weight in `rows`

    def check(token):
        token = _np(token)
        assert (token >= 0).all() and (row[np.arange(Bn), token] > 0).all()
        c = row.astype(np.float64).cumsum(-1)
        t = us.astype(np.float64) * c[:, -1]
        at, w = c[np.arange(Bn), token], row[np.arange(Bn), token]
        assert (np.maximum(at - w - t, t - at) <= 1e-6).all()

    # verify: the root's tokens are rejected, its token and those of the leaves drawn from `rows`
    tokens = torch.full((Bn, 3), -1, dtype=torch.int32, device=DEV)
    tokens[:, 1], tokens[:, 2] = 2, 1
    pb = B.Problem(rows, other, B.PROBS, 2, 2)
    u_v = torch.full((Bn, 3, 3), 0.5, device=DEV)
    u_v[..., 2] = u[:, None]
    g = getattr(B, method + "_verify")(pb, tokens, u_v)
    assert (g["outcome"] == -1).all()
    for n in (1, 2):
        check(g["token"][:, n])
    check(g["token"][:, 0])
    assert (g["flags"][:, 1:] == 0).all()
    if method != "rrsw":            # (RRSw: both drafts rejected, the draft's mass is exhausted)
        assert (g["flags"][:, 0] == 0).all()
    # draft: the first draw
    u_d = torch.full((Bn, 3, 2), 0.25, device=DEV)
    u_d[:, 0, 0] = u
    d = DRAFT[method](B.Problem(None, rows, B.PROBS, 2, 2), u_d)
    check(d["tokens"][:, 1])
    assert (d["flags"] == 0).all()


@pytest.mark.parametrize("method,k", [("spechub", 2), ("rrs", 2), ("rrs", 4), ("rrsw", 2), ("rrsw", 4)])
@pytest.mark.parametrize("dtype,V,off,Bn", [
    ("bf16", 9001, 3, 1536), ("bf16", 12000, 0, 1601), ("bf16", 16369, 1, 1601), ("fp32", 7001, 2, 1601), ("fp32", 8000, 0, 1601),
    ("bf16", 20001, 1, 1920), ("bf16", 32000, 0, 1921), ("fp32", 12000, 0, 1921), ("fp32", 16373, 3, 1921),
])
def test_drafts_of_large_batches(method, k, dtype, V, off, Bn):
    """256 threads per node where the nodes with children do not fit the chip at once: the oracle's tokens, hub and flags except
    where a uniform lies within 1e-6 of a boundary, and bit for bit what the same rows draft in a small batch."""
    N = W.tree_nodes(k, 2)
    buf = torch.zeros(Bn * N * V + 16, dtype=torch.float32 if dtype == "fp32" else torch.bfloat16, device=DEV)
    rows = buf[off:off + Bn * N * V].view(Bn, N, V)
    rows.normal_(0.0, 2.0, generator=torch.Generator(device=DEV).manual_seed(V))
    wl = W.Workload("large", Bn, N, V, k, 2, dtype, "logits", 1.0, 0.9, rows, rows)
    u_d, _ = uniforms(wl, V)
    pb = B.Problem.from_workload(wl).with_draft_stats()
    g = DRAFT[method](pb, u_d)
    for part in (slice(0, 4), slice(Bn - 4, Bn)):
        small = B.Problem(rows[part], rows[part], B.LOGITS, k, 2, 1.0, 0.9).with_draft_stats()
        s = DRAFT[method](small, u_d[part].contiguous())
        for name, t in s.items():
            if t is not None:
                assert torch.equal(t, g[name][part]), name
        assert torch.equal(small.draft_stats.view(torch.int32), pb.draft_stats[part].view(torch.int32))
    seqs = [0, Bn // 2, Bn - 1]
    o = oracle.batch_draft(METHODS[method], W.rows_as_numpy(rows[seqs]), _np(u_d[seqs]), temp_draft=0.9, nthreads=8,
                           **oracle_kwargs(wl))
    sure = o["margin"][:, 0] > 1e-6
    assert sure.any()
    assert (_np(g["tokens"][seqs])[sure] == o["tokens"][sure]).all()
    assert (_np(g["flags"][seqs]) == o["flags"]).all()
    if method == "spechub":
        assert (_np(g["hub"][seqs]) == o["hub"]).all()
