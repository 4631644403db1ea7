"""GPU parity where the kernels' tilings can go wrong: matrices with fewer row
groups than XCDs, ragged groups, column counts that leave a wave without a
step, projections split over 2 to 8 workgroups, one to eight token tiles; and
the float32 path with sizes that rule out its 16-byte loads.  Every node's
logits against the oracle within the tolerances of gpu_cases (bf16 2e-2 + 1e-2
|o|, float32 1e-4 + 1e-4 |o|)."""
import dataclasses

import numpy as np
import pytest
import torch

import paper_2405_18628_amd as ppd
from gpu_cases import check_logits, check_pred, gpu_step, make_case, oracle_step, tree_for, workspace
from synth.configs import ModelShape, Workload
from test_plans_cpu import SPLIT_CASES

pytestmark = pytest.mark.gpu


def _case(dtype, hidden, heads, kv, d, ffn, vocab, L, cap=None, layers=2):
    sh = ModelShape(f"edge-{dtype}-{hidden}-{ffn}", layers, hidden, heads, kv, d, ffn, vocab, dtype)
    return make_case(Workload("edge", sh, L, "total:16", 5, "normal", 50), capacity=cap)


def _check(case, spec):
    tree = tree_for(case, spec=spec)
    ws = workspace(case, tree.T)
    res, ref = gpu_step(case, tree, ws), oracle_step(case, tree)
    assert ppd.ppd_device_status(ws) == 0
    check_logits(res["logits"], ref["logits"], case.shape.dtype, f"T={tree.T}")
    check_pred(res["pred"], ref["logits"], case.shape.dtype)


@pytest.mark.parametrize("shape", [
    (128, 1, 1, 64, 7),        # 4 gate/up groups and 1 LM-head group for 8 XCDs
    (640, 5, 1, 448, 333),     # 10 and 7 chunks of columns, ragged groups
    (384, 8, 2, 1152, 1000),   # 18 chunks of columns, ragged groups
    (2048, 16, 16, 5632, 500),  # the 1.4B widths: output / down whole or in 4 slices, LM head in 8
])
@pytest.mark.parametrize("specs", [("chain:1", "total:33", "total:80"), ("total:16", "total:50", "total:128")])
def test_bf16_tilings(shape, specs):
    hidden, heads, kv, ffn, vocab = shape
    case = _case("bf16", hidden, heads, kv, 128, ffn, vocab, 70, layers=1 if hidden > 1000 else 2)
    for spec in specs:
        _check(case, spec)


@pytest.mark.parametrize("shape,T,plans", SPLIT_CASES)
def test_bf16_split_tiles(shape, T, plans):
    """GEMMs of every kind in 2, 4 and 8 K slices (that they are is checked
    beside SPLIT_CASES)."""
    hidden, heads, kv, ffn, vocab = shape
    case = _case("bf16", hidden, heads, kv, 128, ffn, vocab, 70, layers=1)
    _check(case, f"total:{T}")


@pytest.mark.parametrize("hidden,heads,kv,d,ffn,vocab,L,cap,spec", [
    (256, 4, 4, 64, 688, 1000, 128, 256, "total:25"),  # 16-byte loads everywhere
    (66, 3, 1, 22, 77, 101, 37, 61, "total:17"),       # none: rows of 66 and 77, head 22, capacity 61
    (40, 2, 2, 20, 36, 37, 5, 9, "chain:1"),           # one node and its chain
    (128, 1, 1, 128, 64, 16, 300, 431, "total:128"),   # the widest head, eight token tiles
    (60, 2, 1, 30, 44, 50, 0, 8, "total:7"),           # no prefix; head rows unaligned, matrix rows aligned
    (132, 2, 1, 126, 70, 60, 150, 255, "total:20"),     # wide heads without 16-byte rows, capacity odd
    (132, 2, 1, 102, 70, 60, 150, 256, "total:33"),     # and values with them
])
def test_f32_sizes(hidden, heads, kv, d, ffn, vocab, L, cap, spec):
    _check(_case("f32", hidden, heads, kv, d, ffn, vocab, L, cap), spec)


def test_f32_overflowed_node_stays_invisible():
    """A node whose embedding is infinite changes no node that does not see it
    (bit for bit), in the float32 path."""
    case = _case("f32", 256, 4, 4, 64, 688, 1000, 40)
    tree = tree_for(case, spec="total:25")
    ws = workspace(case, tree.T)
    clean = gpu_step(case, tree, ws)["logits"]
    last = tree.T - 1  # the last node of the last prompt chain: nothing sees it
    assert last not in tree.parent
    tree.ids[last] = 999
    assert not (np.delete(tree.ids, last) == 999).any()
    case.W["tok_emb"][999].fill_(float("inf"))
    torch.cuda.synchronize()
    got = gpu_step(case, tree, ws)["logits"]
    assert np.array_equal(got[:last], clean[:last])
    assert not np.isfinite(got[last]).all()


@pytest.mark.parametrize("hidden,heads,kv,d,L", [
    (256, 4, 4, 64, 37),   # keys 37 .. 61: three blocks, prefix and tree keys mixed
    (66, 3, 1, 22, 37),    # heads that are no multiple of 16, no 16-byte rows
    (132, 2, 1, 126, 44),
])
def test_f32_overflowed_node_among_visible_keys(hidden, heads, kv, d, L):
    """The same for leaves whose keys share their 16-key block with keys that the
    other nodes see: the block's sums are then formed key by key, which changes
    their order only (float32 tolerance)."""
    case = _case("f32", hidden, heads, kv, d, 77, 1000, L)
    tree = tree_for(case, spec="total:25")
    ws = workspace(case, tree.T)
    clean = gpu_step(case, tree, ws)["logits"]
    leaves = [i for i in range(tree.T) if i not in tree.parent]
    ids = tree.ids.copy()
    case.W["tok_emb"][999].fill_(float("inf"))
    torch.cuda.synchronize()
    tried = 0
    for leaf in leaves[:-1]:
        block = [k for k in range((L + leaf) // 16 * 16, (L + leaf) // 16 * 16 + 16) if k < L + tree.T]
        if len(block) < 4:
            continue
        tried += 1
        tree.ids[:] = ids
        tree.ids[leaf] = 999
        got = gpu_step(case, tree, ws)["logits"]
        rest = np.delete(np.arange(tree.T), leaf)
        check_logits(got[rest], clean[rest], "f32", f"leaf {leaf}")
        assert not np.isfinite(got[leaf]).all()
    assert tried >= 3


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("f32", 64), ("f32", 22)])
@pytest.mark.parametrize("n", [0, 1, 2, 3, 7, 8, 9, 40])  # up to eight rows in registers, more through LDS
def test_compaction_lengths(dtype, d, n):
    """cache[L + k] <- cache[L + path[k]] for every path length, bit for bit,
    with the path longer than its count and its last row at the capacity."""
    layers, nkv, L, T = 2, 3, 24, 64
    cap = L + T
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    gen = torch.Generator(device="cuda").manual_seed(n)
    k = torch.randn((layers, nkv, cap, d), generator=gen, device="cuda").to(dt)
    v = torch.randn((layers, nkv, d, cap), generator=gen, device="cuda").to(dt)
    rows = [0] + sorted(np.random.RandomState(n).permutation(np.arange(1, T))[:max(0, n - 1)].tolist())
    rows = rows[:n]
    if n > 1:
        rows[-1] = T - 1
    path = torch.full((T,), -1, dtype=torch.int32, device="cuda")
    path[:n] = torch.tensor(rows, dtype=torch.int32)
    kw, vw = k.clone(), v.clone()
    kw[:, :, L:L + n] = k[:, :, [L + r for r in rows]]
    vw[:, :, :, L:L + n] = v[:, :, :, [L + r for r in rows]]
    sh = ModelShape("compact", layers, 128, nkv, nkv, d, 64, 16, dtype)
    case = make_case(Workload("compact", sh, 8, "total:16", 5, "normal", 50))
    ppd.ppd_kv_compact(case.model, ppd.KVCache(k, v), L, path, torch.tensor([n], dtype=torch.int32, device="cuda"))
    assert torch.equal(k, kw) and torch.equal(v, vw)


@pytest.mark.parametrize("T", [1, 2, 7, 8, 9, 15])  # the padding lanes' mask ends at eight tokens
def test_bf16_few_tokens(T):
    case = _case("bf16", 640, 5, 1, 128, 448, 333, 70)
    tree = tree_for(case, spec="total:16")
    # a prefix of a topological order is a tree
    tree = dataclasses.replace(tree, parent=tree.parent[:T], ids=tree.ids[:T],
                               n_candidates=min(T, tree.n_candidates))
    ws = workspace(case, T)
    res, ref = gpu_step(case, tree, ws), oracle_step(case, tree)
    assert ppd.ppd_device_status(ws) == 0
    check_logits(res["logits"], ref["logits"], "bf16", f"T={T}")
    check_pred(res["pred"], ref["logits"], "bf16")
