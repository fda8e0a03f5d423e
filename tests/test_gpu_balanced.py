"""Verify attention over the even division of the batch's key tiles: batches
that the automatic plan takes there, at the sizes where it can go wrong.

The plan is the automatic one (no split, row group or packing asked for), so
each case first checks that it is the even division."""

import numpy as np
import pytest
import torch

from paper_2606_04446_amd import workload as wl
from tests.gpu_cases import Case, TOL, d2sd, max_abs

pytestmark = pytest.mark.gpu


def even_case(lay, host_offsets=True, **kw):
    case = Case(lay, **kw)
    assert d2sd().cascade_division(case._args(host_offsets=host_offsets))[0], "not the even division"
    return case


def check(lay, stages=(0,), host_offsets=True, reqs=None):
    case = even_case(lay, host_offsets, poison_slack=True)
    for stage in stages:
        o, l = case.attention(stage=stage, host_offsets=host_offsets)
        torch.cuda.synchronize()
        assert torch.isfinite(o.float()).all()
        for b in range(lay.batch) if reqs is None else reqs:
            s, e = int(case.node_indptr[b]), int(case.node_indptr[b + 1])
            ow, lw = case.oracle_attention(b, ("cascade", "prefix", "tree")[stage])
            lg = l[s:e].cpu().numpy()
            fin = np.isfinite(lw)
            assert np.array_equal(fin, np.isfinite(lg))
            err = max(max_abs(o[s:e].double().cpu().numpy(), ow), max_abs(lg[fin], lw[fin]) if fin.any() else 0.0)
            assert err <= TOL[case.dtype], (stage, b, err)


def even_layout(B, p_rows, ctx, hq, hkv, dtype, seed):
    """The requests, and for bf16 as many more of 8192 tokens as the even
    division asks for (20 key tiles and 80 pairs of tiles per CU)."""
    p_rows, ctx = list(p_rows), list(ctx)
    extra = list(range(2, B, 3))
    nodes = sum(B + sum(B - x for x in r) for r in p_rows)
    while dtype == "bf16" and (len(ctx) * hkv * max(ctx) < 20 * 32 * 256 or hq * nodes * max(ctx) < 80 * 32 * 32 * 256):
        p_rows.append(extra)
        ctx.append(8192)
        nodes += B + sum(B - x for x in extra)
    return wl.custom_layout(B, p_rows, ctx, hq=hq, hkv=hkv, dtype=dtype, seed=seed)


def rows_for(rng, B, batch, k):
    return [sorted(rng.choice(np.arange(1, B), int(rng.integers(0, k + 1)), replace=False).tolist()) for _ in range(batch)]


# 1 to 14, 16, 24 and 31 query tiles per stream: one to three row groups, every
# wave count around the two key groups' limit (fp32), groups of 3, 4, 5 and 8 heads
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("B,p,hq,hkv", [(8, [], 8, 2), (16, [], 8, 2), (16, [4], 8, 2), (16, [1, 5], 12, 4), (16, [4], 40, 8),
                                        (16, [2, 9], 8, 2), (16, [1, 3], 8, 2), (16, [1, 5, 9, 13], 32, 8),
                                        (16, [1, 2, 3, 4, 5, 6], 8, 2), (16, [1, 2, 3, 4, 5, 6, 7], 8, 2),
                                        (24, [1, 2, 3, 4], 8, 2), (32, [1, 2, 3], 8, 2), (32, [1, 2], 8, 1),
                                        (32, [1, 2, 3], 8, 1)])
def test_query_tiles(B, p, hq, hkv, dtype):
    check(even_layout(B, [p], [1100], hq=hq, hkv=hkv, dtype=dtype, seed=B + len(p)), reqs=range(1))


# ends of key tiles, pages and ring fills; contexts shorter than the tree; empty ones
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("ctx", [[1024], [1025, 0, 1, 31], [1055, 32, 33, 63, 64, 65], [2047, 255, 256, 257, 511],
                                 [1040, 1039, 1041, 16, 15, 17, 0, 0]])
def test_ragged_contexts(ctx, dtype):
    rng = np.random.default_rng(len(ctx))
    check(even_layout(16, rows_for(rng, 16, len(ctx), 5), ctx, hq=8, hkv=2, dtype=dtype, seed=7), stages=(0, 1, 2),
          host_offsets=False, reqs=range(len(ctx)))


def test_many_requests_and_shares_of_many_streams():
    """One long context beside a hundred short ones (a workgroup takes many
    streams; more requests than lanes of the scheduling wave), and the largest
    batch the shape takes."""
    rng = np.random.default_rng(5)
    ctx = [6000] + [int(x) for x in rng.integers(0, 90, 100)]
    check(wl.custom_layout(16, rows_for(rng, 16, 101, 2), ctx, hq=4, hkv=1, seed=8), reqs=range(0, 101, 7))
    ctx = [1300] + [int(x) for x in rng.integers(0, 40, 255)]
    check(wl.custom_layout(8, rows_for(rng, 8, 256, 1), ctx, hq=8, hkv=1, seed=9), reqs=range(0, 256, 17))


def test_large_grid_of_the_four_wave_shape():
    """100 requests of 1 to 8 query tiles that one split would fill the chip
    with: shares of several streams, most of them whole, ragged contexts."""
    rng = np.random.default_rng(6)
    ctx = [1700] + [int(x) for x in rng.integers(1, 1700, 99)]
    p = [[2, 5, 9, 13]] + rows_for(rng, 16, 99, 4)
    p = [r if sum(16 - x for x in r) <= 48 else r[2:] for r in p]      # at most 64 nodes with the block
    lay = wl.custom_layout(16, p, ctx, hq=32, hkv=8, seed=10)
    lay_nodes = [16 + sum(16 - x for x in r) for r in p]
    assert 33 <= max(lay_nodes) <= 64 and sum(-(-4 * n // 128) for n in lay_nodes) * 8 >= 768
    check(lay, reqs=range(0, 100, 9))


def test_page_list_longer_than_one_staging():
    """256 streams of 40,000 tokens: a workgroup's piece is longer than the
    32,768 tokens whose page ids it stages at a time. The logical pages share
    500 physical ones."""
    lay = wl.custom_layout(8, [[]] * 16, [40000] * 16, hq=16, hkv=16, seed=3)
    lay.page_table = np.random.default_rng(3).integers(0, 500, lay.page_table.shape).astype(np.int32)
    lay.num_pages = 500
    case = even_case(lay)
    o, l = case.attention(host_offsets=True)
    torch.cuda.synchronize()
    for b in (0, 15):
        s, e = int(case.node_indptr[b]), int(case.node_indptr[b + 1])
        ow, lw = case.oracle_attention(b)
        assert max_abs(o[s:e].double().cpu().numpy(), ow) <= TOL["bf16"] and max_abs(l[s:e].cpu().numpy(), lw) <= TOL["bf16"]


@pytest.mark.parametrize("scale", [30.0, 1000.0])
def test_large_scores(scale):
    """Scores far above the first tile's reference: the reference moves in the
    middle of a stream, by more than the exponent range at the larger scale."""
    lay = even_layout(16, [[3, 9], [1]], [1500, 1100], hq=8, hkv=2, dtype="bf16", seed=11)
    case = even_case(lay)
    case.x["q"].mul_(scale)
    o, l = case.attention(host_offsets=True)
    torch.cuda.synchronize()
    for b in range(2):
        s, e = int(case.node_indptr[b]), int(case.node_indptr[b + 1])
        ow, lw = case.oracle_attention(b)
        # products of bf16 inputs are exact, their fp32 sums good to 1e-6 of a score of up to ~20 scale
        tol = 2e-2 + 2e-5 * scale
        assert max_abs(o[s:e].double().cpu().numpy(), ow) <= 2 * tol
        assert max_abs(l[s:e].cpu().numpy(), lw) <= tol


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_dominant_first_key_has_weight_one(dtype):
    """A key of the first tile that holds nearly all the weight of every row has
    probability 1, which bf16 holds exactly: lse is its score to the accuracy of
    fp32 sums (1e-6 of a score of about 28), not of a bf16 probability (2e-3)."""
    case = even_case(even_layout(16, [[3, 9], [1], []], [1500, 1100, 700], hq=8, hkv=2, dtype=dtype, seed=13))
    u = torch.zeros(128, device="cuda")
    u[::2] = 0.125                                             # a unit vector, exact in bf16
    case.x["q"] += 8 * u
    for b in range(3):
        case.x["k_cache"][int(case.layout.page_table[b, 0]), :, 3] = 40 * u
    o, l = case.attention(host_offsets=True)
    torch.cuda.synchronize()
    for b in range(3):
        s, e = int(case.node_indptr[b]), int(case.node_indptr[b + 1])
        ow, lw = case.oracle_attention(b)
        assert max_abs(l[s:e].cpu().numpy(), lw) <= 1e-4
        assert max_abs(o[s:e].double().cpu().numpy(), ow) <= TOL[dtype]


def test_partial_states_cost_no_accuracy():
    """Two roundings to bf16 (the probabilities and the result) have a relative
    error of 1.65e-3 each in the 2-norm, 2.34e-3 together; a third one, of the
    pieces' outputs, would make it 2.86e-3 however many pieces there are."""
    case = even_case(even_layout(16, [[2, 5, 8, 11]] * 4, [4096, 3000, 2000, 1500], hq=32, hkv=8, dtype="bf16", seed=14))
    o, _ = case.attention(host_offsets=True)
    torch.cuda.synchronize()
    err = ref = 0.0
    for b in range(4):
        s, e = int(case.node_indptr[b]), int(case.node_indptr[b + 1])
        ow, _ = case.oracle_attention(b)
        err += float(((o[s:e].double().cpu().numpy() - ow) ** 2).sum())
        ref += float((ow ** 2).sum())
    assert (err / ref) ** 0.5 <= 2.6e-3


def test_two_streams_with_their_own_workspaces():
    """Two calls in flight on two streams give what each gives alone."""
    lays = [even_layout(16, [[3, 9], [1]], [3000, 1100], hq=8, hkv=2, dtype="bf16", seed=s) for s in (21, 22)]
    cases = [even_case(x) for x in lays]
    alone = [c.attention(host_offsets=True) for c in cases]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in cases]
    for _ in range(5):
        got = []
        for c, st in zip(cases, streams):
            with torch.cuda.stream(st):
                got.append(c.attention(host_offsets=True))
        torch.cuda.synchronize()
        for g, a in zip(got, alone):
            assert torch.equal(g[0], a[0]) and torch.equal(g[1], a[1])
