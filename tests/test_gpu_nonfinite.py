"""Infinite V entries: softmax weights are positive, so a visible key whose V
holds an infinity makes that dim of every row that sees it infinite, and
touches nothing else."""

import numpy as np
import pytest
import torch

from paper_2606_04446_amd import workload as wl
from tests.gpu_cases import Case, d2sd
from tests.test_gpu_balanced import even_layout

pytestmark = pytest.mark.gpu


def check(lay, keys, **kw):
    """keys: {request: context key}; every row of the request sees its key, in
    one dim of one KV head. All other outputs and lse equal a run without it."""
    case = Case(lay)
    o, l = (t.clone() for t in case.attention(**kw))
    G = lay.spec.hq // lay.spec.hkv
    dims = {}
    for b, key in keys.items():
        h, d = b % lay.spec.hkv, (37 * b + 5) % 128
        case.x["v_cache"][int(lay.page_table[b, key // 16]), h, key % 16, d] = float("inf") if b % 2 else float("-inf")
        dims[b] = h, d
    oi, li = case.attention(**kw)
    torch.cuda.synchronize()
    assert torch.isfinite(o.float()).all() and torch.equal(l, li)
    for b, (h, d) in dims.items():
        s, e = int(case.node_indptr[b]), int(case.node_indptr[b + 1])
        got = oi[s:e, h * G:(h + 1) * G, d].float()
        assert (got == (float("inf") if b % 2 else float("-inf"))).all(), (b, got)
        oi[s:e, h * G:(h + 1) * G, d] = o[s:e, h * G:(h + 1) * G, d]
    assert torch.equal(o, oi)


# splits of a context that fill a round of the merge and that do not, in one and in four groups
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("kv_split", [64, 128, 192, 320, 512])
def test_infinite_value_in_the_last_split(kv_split, dtype):
    ctx = [1000, 650, 520, 330]
    lay = wl.custom_layout(16, [[3, 7], [1], [], [2, 5, 9, 15]], ctx, hq=8, hkv=2, dtype=dtype, seed=11)
    check(lay, {b: c - 1 for b, c in enumerate(ctx)}, kv_split=kv_split)


# the even division: keys of a partial last tile, of which the first also fills the copy's rows past the valid ones
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("at", ["first of the last tile", "last"])
def test_infinite_value_beside_padded_keys(at, dtype):
    ctx = [3000, 1001, 2060, 331, 33]
    lay = even_layout(16, [[3, 7], [1], [], [2, 5, 9, 15], [4]], ctx, hq=8, hkv=2, dtype=dtype, seed=12)
    assert d2sd().cascade_division(Case(lay)._args())[0]
    check(lay, {b: c - 1 if at == "last" else (c - 1) // 32 * 32 for b, c in enumerate(ctx)})
