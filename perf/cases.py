"""The work that a user has this library do, as cases with inputs, one timed
pass each, and a 64-bit reference.

Two kinds of case, both through the package's public entry points:

  step   one decode step: verify (or the batched / static-workspace verify),
         accept, compact, as a decode loop enqueues them.  Returns the logits
         of every tree node, the greedy tokens, the accepted path and the
         whole KV cache (the step writes the tree's rows into it and commits
         the accepted ones).
  tail   what follows a forward pass whose logits are at hand: accept,
         compact over all layers, the next tree's ids.

Models are random but predict confidently, as trained ones do: the LM head
row of a token's successor is aligned with the token's embedding, the output
and down projections are scaled with the depth (so the residual stream keeps
the embedding), prompt embeddings lie near token embeddings, and about half of
the guesses in a tree are right, so that some are accepted.  Keys and values
of the prefix are N(0, 1).
"""
from __future__ import annotations

import math
import random
from types import SimpleNamespace

import numpy as np
import torch

import paper_2405_18628_amd as ppd

N_PROMPT = 3
EPS, BASE = 1e-6, 10000.0

# hidden, heads, kv heads, ffn of the model shapes used below
W_1B4 = dict(hidden=2048, heads=16, kv_heads=16, ffn=5632)
W_7B = dict(hidden=4096, heads=32, kv_heads=32, ffn=11008)
W_13B = dict(hidden=5120, heads=40, kv_heads=40, ffn=13824)
W_GQA = dict(hidden=4096, heads=32, kv_heads=8, ffn=11008)  # 7B width, grouped-query heads


def _step(name, width, layers, T, L, batch=1, vocab=32000, dtype="bf16", static=False):
    c = dict(kind="step", dtype=dtype, layers=layers, head_dim=128 if dtype == "bf16" else 64,
             vocab=vocab, T=T, L=L, batch=batch, static=static, **width)
    return dict(c, name=name) if name else c


def _tail(name, layers, kv_heads, T, L, vocab, accepted, n_ept):
    c = dict(kind="tail", dtype="bf16", layers=layers, kv_heads=kv_heads, head_dim=128, vocab=vocab,
             T=T, L=L, accepted=accepted, n_ept=n_ept)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the small launches after every forward pass of the 7B shape: five
        # guesses accepted, the cache of 32 layers compacted, the next
        # 64-node tree filled
        _tail("tail_7b", 32, 32, 64, 2048, 32000, 5, 1),
        # the fp32 path, a whole tiny decoder: launches and latency count
        _step("tiny_f32", dict(hidden=256, heads=4, kv_heads=4, ffn=688), 2, 25, 128, vocab=1000,
              dtype="f32"),
        # edge-size model, small tree, short context, the entry point that
        # needs no caller workspace
        _step("edge_static_T16", W_1B4, 4, 16, 200, static=True),
        # vanilla decoding: the root alone (what speculative decoding is
        # compared with, and the first step of every generation)
        _step("7b_vanilla_T1", W_7B, 4, 1, 2048),
        # the tree size that the hardware-aware sizing picks at 7B
        _step("7b_T32", W_7B, 4, 32, 2048),
        # four users' sequences of different lengths in one step
        _step("7b_batch4_T16", W_7B, 4, 16, 2048, batch=4),
        # grouped-query heads, a ragged tree, an odd prefix and an odd
        # vocabulary (added special tokens)
        _step("gqa_ragged_T41", W_GQA, 4, 41, 777, vocab=32001),
        # long context: the cache read outweighs the weights of a layer
        _step("7b_32k_T64", W_7B, 2, 64, 32768),
        # the largest tree on the widest model
        _step("13b_T128", W_13B, 2, 128, 4096),
        # a mid-size tree that is no multiple of a power of two
        _step("13b_T88", W_13B, 3, 88, 4000),
        # whole models: the 1.4B shape with its 80-node tree, and the 7B shape
        # with 64 nodes over a 2048-token prefix (the benchmark's step)
        _step("1.4b_full_T80", W_1B4, 24, 80, 1024),
        _step("7b_full_T64", W_7B, 32, 64, 2048),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    u = rng.random()
    if u < 0.1:
        return _tail(None, rng.randint(4, 32), rng.choice([8, 16, 32, 40]), rng.randint(16, 128),
                     _log_int(rng, 16, 8192), rng.choice([32000, rng.randint(1000, 50000)]),
                     rng.randint(0, 3), rng.choice([1, 1, 2]))
    if u < 0.2:
        heads = rng.choice([2, 4, 6])
        return _step(None, dict(hidden=heads * 64, heads=heads, kv_heads=rng.choice([heads, heads // 2]),
                                ffn=rng.randint(200, 1400)), rng.randint(1, 4),
                     _log_int(rng, 1, 64), _log_int(rng, 1, 512), vocab=rng.randint(300, 4000),
                     dtype="f32")
    if rng.random() < 0.25:
        kv = rng.choice([2, 4, 8])
        width = dict(hidden=128 * rng.randint(8, 40), heads=kv * rng.choice([1, 2, 4]), kv_heads=kv,
                     ffn=64 * rng.randint(20, 220))
    else:
        width = rng.choice([W_1B4, W_7B, W_13B, W_GQA])
    batch = rng.choice([1, 1, 1, rng.randint(2, 8)])
    return _step(None, width, rng.randint(1, 4), _log_int(rng, 1, 128 // batch),
                 _log_int(rng, 1, 32768 if batch == 1 else 4096), batch=batch,
                 vocab=rng.choice([32000, rng.randint(1000, 50000)]),
                 static=batch == 1 and rng.random() < 0.15)


# ---------------------------------------------------------------------------
# inputs, from the seed alone


def _lengths(case):
    """Cached tokens of each sequence of the step."""
    B, L = case["batch"], case["L"]
    return [L - j * L // (2 * B) for j in range(B)]


def _capacity(L):
    return (L + 128 + 63) // 64 * 64


def _tree(rng, T, vocab, succ, root, n_ept=1):
    """T nodes: a root, guesses below it (about a quarter of the nodes) and
    chains of prompt tokens under them; guesses follow succ about half of the
    time."""
    n = max(1, -(-T // (1 + N_PROMPT * n_ept)))
    parent, ids, depth, kids = [-1], [root], [0], [set()]
    while len(parent) < n:
        p = rng.choice([i for i in range(len(parent)) if depth[i] < 5 and len(kids[i]) < 4])
        t = int(succ[ids[p]])
        if t in kids[p] or rng.random() < 0.5:
            t = rng.choice([x for x in (rng.randrange(vocab) for _ in range(8)) if x not in kids[p]])
        kids[p].add(t)
        parent.append(p)
        ids.append(t)
        depth.append(depth[p] + 1)
        kids.append(set())
    for c in range(n):
        for g in range(n_ept):
            prev = c
            for j in range(N_PROMPT):
                if len(parent) == T:
                    break
                parent.append(prev)
                ids.append(vocab + j * n_ept + g)
                prev = len(parent) - 1
    return parent, ids


def _cache(case, L, gen):
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    n, h, d, cap = case["layers"], case["kv_heads"], case["head_dim"], _capacity(L)
    k = torch.zeros((n, h, cap, d), dtype=dt, device="cuda")
    v = torch.zeros((n, h, d, cap), dtype=dt, device="cuda")
    for l in range(n):
        k[l, :, :L] = torch.randn((h, L, d), generator=gen, device="cuda", dtype=dt)
        v[l, :, :, :L] = torch.randn((h, d, L), generator=gen, device="cuda", dtype=dt)
    return k, v


def _inputs(case, seed):
    """Weights, caches and trees of a step."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    rng = random.Random(seed)
    H, F, V, d = case["hidden"], case["ffn"], case["vocab"], case["head_dim"]
    nq, rows = case["heads"] * d, (case["heads"] + 2 * case["kv_heads"]) * d
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32

    def normal(shape, std):
        return torch.randn(shape, generator=gen, device="cuda", dtype=dt).mul_(std)

    def gain():
        return (1 + 0.1 * torch.randn(H, generator=gen, device="cuda")).to(dt)

    emb = torch.randn((V, H), generator=gen, device="cuda")
    succ = torch.randperm(V, generator=gen, device="cuda")
    head = torch.empty((V, H), device="cuda")
    head[succ] = 0.8 * emb + 0.6 * torch.randn((V, H), generator=gen, device="cuda")
    near = torch.randint(V, (N_PROMPT,), generator=gen, device="cuda")
    prompt = 0.8 * emb[near] + 0.6 * torch.randn((N_PROMPT, H), generator=gen, device="cuda")
    out_std = 0.02 / math.sqrt(2 * 32)
    W = dict(tok_emb=emb.to(dt), prompt_emb=prompt.to(dt), final_norm=gain(),
             lm_head=(0.02 * head).to(dt), layers=[])
    for _ in range(case["layers"]):
        W["layers"].append(dict(attn_norm=gain(), w_qkv=normal((rows, H), 0.02),
                                w_o=normal((H, nq), out_std), mlp_norm=gain(),
                                w_gate_up=normal((2 * F, H), 0.02), w_down=normal((H, F), out_std)))
    succ = succ.cpu().numpy()
    seqs = []
    for L in _lengths(case):
        parent, ids = _tree(rng, case["T"], V, succ, rng.randrange(V))
        k, v = _cache(case, L, gen)
        seqs.append(dict(L=L, parent=parent, ids=ids, k=k, v=v))
    return W, seqs


def _ints(v):
    return torch.tensor(v, dtype=torch.int32, device="cuda")


def _path_buffers(seq, T):
    seq["parent_d"] = _ints(seq["parent"])
    seq["path"] = torch.full((T,), -1, dtype=torch.int32, device="cuda")
    seq["n_path"] = torch.zeros(1, dtype=torch.int32, device="cuda")
    seq["next_tok"] = torch.zeros(1, dtype=torch.int32, device="cuda")
    seq["kv"] = ppd.KVCache(seq["k"], seq["v"])


def prepare(case, seed):
    if case["kind"] == "tail":
        return _prepare_tail(case, seed)
    W, seqs = _inputs(case, seed)
    T, V, B = case["T"], case["vocab"], case["batch"]
    shape = SimpleNamespace(n_layers=case["layers"], hidden=case["hidden"], n_heads=case["heads"],
                            n_kv_heads=case["kv_heads"], head_dim=case["head_dim"], ffn=case["ffn"],
                            vocab=V, n_prompt=N_PROMPT, rms_eps=EPS, rope_base=BASE,
                            dtype=case["dtype"])
    model = ppd.Model(shape, W)
    depth, mask = zip(*(ppd.ppd_build_tree_mask(s["parent"]) for s in seqs))
    s = SimpleNamespace(case=case, model=model, seqs=seqs, Ls=[q["L"] for q in seqs], Ts=[T] * B)
    s.ids = _ints(sum((q["ids"] for q in seqs), []))
    s.depth = torch.from_numpy(np.concatenate(depth)).cuda()
    s.mask = torch.from_numpy(np.concatenate(mask).view(np.int64)).cuda()
    s.logits = torch.zeros((B * T, V), device="cuda")
    s.pred = torch.zeros(B * T, dtype=torch.int32, device="cuda")
    n_ws = 256 if case["static"] else ppd.ppd_workspace_bytes(model, B * T, _capacity(max(s.Ls)))
    s.ws = torch.empty(n_ws, dtype=torch.uint8, device="cuda")
    ppd.ppd_workspace_init(s.ws)
    for q in seqs:
        _path_buffers(q, T)
    return s


def _prepare_tail(case, seed):
    """Outputs of a forward pass as a step leaves them: logits, greedy tokens
    that accept a chain of guesses, and the tree's rows in the cache."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    rng = random.Random(seed)
    T, V, G = case["T"], case["vocab"], case["n_ept"]
    succ = np.random.RandomState(seed % (1 << 32)).permutation(V)
    parent, ids = _tree(rng, T, V, succ, rng.randrange(V), G)
    logits = torch.randn((T, V), generator=gen, device="cuda")
    pred = [int(succ[t]) if t < V else rng.randrange(V) for t in ids]
    node = 0  # a chain of guesses made right
    for _ in range(case["accepted"]):
        kids = [i for i in range(T) if parent[i] == node and ids[i] < V]
        if not kids:
            break
        pred[node] = ids[kids[0]]
        node = kids[0]
    k, v = _cache(case, case["L"] + T, gen)
    seq = dict(L=case["L"], parent=parent, ids=ids, k=k, v=v)
    # the model description that compaction is given: sizes and set pointers
    one = torch.zeros(256, dtype=torch.bfloat16, device="cuda")
    s = SimpleNamespace(case=case, seqs=[seq], Ls=[case["L"]], Ts=[T], logits=logits)
    s.pred, s.ids = _ints(pred), _ints(ids)
    s.ws = torch.empty(256, dtype=torch.uint8, device="cuda")
    ppd.ppd_workspace_init(s.ws)
    shape = SimpleNamespace(n_layers=case["layers"], hidden=128, n_heads=case["kv_heads"],
                            n_kv_heads=case["kv_heads"], head_dim=128, ffn=64, vocab=V,
                            n_prompt=N_PROMPT * G, rms_eps=EPS, rope_base=BASE, dtype="bf16")
    z = lambda r, c: torch.zeros((r, c), dtype=torch.bfloat16, device="cuda")  # noqa: E731
    nq = case["kv_heads"] * 128
    lay = dict(attn_norm=one[:128], w_qkv=z(3 * nq, 128), w_o=z(128, nq), mlp_norm=one[:128],
               w_gate_up=z(128, 128), w_down=z(128, 64))
    s.model = ppd.Model(shape, dict(tok_emb=z(V, 128), prompt_emb=z(N_PROMPT * G, 128),
                                    final_norm=one[:128], lm_head=z(V, 128),
                                    layers=[lay] * case["layers"]))
    # the next tree: rank paths of a sparse tree, prompt chains under each node
    n = max(1, T // (1 + N_PROMPT * G))
    tp, tk, td, kids = [-1], [0], [0], [0]
    while len(tp) < n:
        p = rng.choice([i for i in range(len(tp)) if td[i] < 3 and kids[i] < 6])
        tp.append(p)
        tk.append(kids[p])
        td.append(td[p] + 1)
        kids.append(0)
        kids[p] += 1
    for c in range(n):
        for g in range(G):
            prev = c
            for j in range(N_PROMPT):
                if len(tp) < 128:
                    tp.append(prev)
                    tk.append(-1 - (j * G + g))
                    prev = len(tp) - 1
    s.tpl_parent, s.tpl_kind = np.asarray(tp, np.int32), np.asarray(tk, np.int32)
    s.next_ids = torch.full((len(tp),), -1, dtype=torch.int32, device="cuda")
    _path_buffers(seq, T)
    return s


def run(s):
    c = s.case
    T, V = c["T"], c["vocab"]
    if c["kind"] == "step":
        kvs = [q["kv"] for q in s.seqs]
        if c["static"]:
            ppd.ppd_verify_step_static(s.model, kvs[0], c["L"], T, s.ids, s.depth, s.mask, s.logits,
                                       s.pred)
        elif len(kvs) > 1:
            ppd.ppd_verify_batch(s.model, kvs, s.Ls, s.Ts, s.ids, s.depth, s.mask, s.ws, s.logits,
                                 s.pred)
        else:
            ppd.ppd_verify_step(s.model, kvs[0], c["L"], T, s.ids, s.depth, s.mask, s.ws, s.logits,
                                s.pred)
    for j, q in enumerate(s.seqs):
        ids, pred = s.ids[j * T:(j + 1) * T], s.pred[j * T:(j + 1) * T]
        ppd.ppd_accept(T, q["parent_d"], ids, pred, V, q["path"], q["n_path"], q["next_tok"], s.ws)
        ppd.ppd_kv_compact(s.model, q["kv"], q["L"], q["path"], q["n_path"])
    out = dict(path=[q["path"] for q in s.seqs], n_path=[q["n_path"] for q in s.seqs],
               next_tok=[q["next_tok"] for q in s.seqs], k=[q["k"] for q in s.seqs],
               v=[q["v"] for q in s.seqs])
    if c["kind"] == "tail":
        q = s.seqs[0]
        ppd.ppd_next_tree(T, q["parent_d"], s.ids, V, N_PROMPT, s.logits, q["path"], q["n_path"],
                          q["next_tok"], s.tpl_parent, s.tpl_kind, s.next_ids, s.ws,
                          n_ept=c["n_ept"])
        out["next_ids"] = s.next_ids
    else:
        out["logits"], out["pred"] = s.logits, s.pred
    return out


# ---------------------------------------------------------------------------


def work(case):
    T, V, d = case["T"], case["vocab"], case["head_dim"]
    if case["kind"] == "tail":
        # three logits rows per EPT group, the accepted rows read and written
        rows = (1 + case["accepted"]) * case["layers"] * case["kv_heads"] * d * 2 * 2
        return dict(bytes=3 * case["n_ept"] * V * 4 + 2 * rows, flops=0)
    e = 2 if case["dtype"] == "bf16" else 4
    H, F, n, B = case["hidden"], case["ffn"], case["layers"], case["batch"]
    nq, nkv = case["heads"] * d, case["kv_heads"] * d
    mats = n * ((nq + 2 * nkv) * H + H * nq + 3 * F * H) + V * H
    Ls, tok = _lengths(case), B * T
    cache = n * 2 * nkv * e * (sum(Ls) + tok)
    attn = n * sum(4 * T * (L + (T + 1) / 2) * nq for L in Ls)
    return dict(bytes=e * mats + e * (2 * n + 1) * H + e * tok * H + cache + 4 * tok * V,
                flops=2 * tok * mats + attn)


def tolerance(case):
    if case["kind"] == "tail":
        return "exact"
    if case["dtype"] == "f32":
        # 3e-7 from the 64-bit result at the listed case; four times that,
        # and room for the longer sums of the drawn ones
        return dict(rel=4e-6)
    # the same nodes under another partition of the sums: logits within
    # 2e-6 .. 9e-6, stored keys and values within 5e-5 .. 1.4e-4 of the tree's
    # rows, since some round to the neighbouring bf16 value (2^-7 of it at
    # most: 0.0078 was seen); four times the largest, and two such steps
    return dict(rel=6e-4, max=2e-2)


def _rotate(x, pos):
    """RoPE of x [T, heads, d], rotate-half pairing, at positions pos [T]."""
    d = x.shape[-1]
    inv = BASE ** (-2.0 * torch.arange(d // 2, device=x.device, dtype=torch.float64) / d)
    a = pos.double()[:, None, None] * inv
    c, s = a.cos(), a.sin()
    lo, hi = x[..., :d // 2], x[..., d // 2:]
    return torch.cat((lo * c - hi * s, hi * c + lo * s), -1)


def _norm(x, gain):
    return x * gain.double() / (x.square().mean(-1, keepdim=True) + EPS).sqrt()


def _exact_sequence(case, W, q):
    """One sequence's step in 64 bits; keys and values are rounded only where
    attention reads them back from a bf16 cache."""
    T, L, V, d, nh, nkv = (case["T"], q["L"], case["vocab"], case["head_dim"], case["heads"],
                           case["kv_heads"])
    parent, ids = q["parent"], q["ids"]
    depth, see = [0] * T, torch.zeros((T, T), dtype=torch.bool)
    for i in range(T):
        if i:
            depth[i] = depth[parent[i]] + 1
            see[i] = see[parent[i]]
        see[i, i] = True
    visible = torch.cat((torch.ones((T, L), dtype=torch.bool), see), 1).cuda()
    pos = L + torch.tensor(depth, device="cuda")
    store = (lambda t: t.bfloat16().double()) if case["dtype"] == "bf16" else (lambda t: t)
    table = torch.cat((W["tok_emb"], W["prompt_emb"]))
    x = table[torch.tensor(ids, device="cuda")].double()
    K, Vv = q["k"].double(), q["v"].double()
    for l, w in enumerate(W["layers"]):
        qkv = _norm(x, w["attn_norm"]) @ w["w_qkv"].double().t()
        qq, kk, vv = (t.reshape(T, -1, d) for t in qkv.split([nh * d, nkv * d, nkv * d], 1))
        qq, kk = _rotate(qq, pos), _rotate(kk, pos)
        K[l, :, L:L + T] = kk.transpose(0, 1)
        Vv[l, :, :, L:L + T] = vv.permute(1, 2, 0)
        o = torch.empty((T, nh, d), dtype=torch.float64, device="cuda")
        for h in range(nh):
            g = h // (nh // nkv)
            keys = torch.cat((K[l, g, :L], store(kk[:, g])))
            vals = torch.cat((Vv[l, g, :, :L].t(), store(vv[:, g])))
            s = (qq[:, h] @ keys.t()) / math.sqrt(d)
            o[:, h] = s.masked_fill(~visible, -math.inf).softmax(-1) @ vals
        x = x + o.reshape(T, nh * d) @ w["w_o"].double().t()
        g, u = (_norm(x, w["mlp_norm"]) @ w["w_gate_up"].double().t()).chunk(2, -1)
        x = x + (torch.nn.functional.silu(g) * u) @ w["w_down"].double().t()
    logits = _norm(x, W["final_norm"]) @ W["lm_head"].double().t()
    pred = logits.argmax(-1).tolist()
    ok, best = [True] * T, 0
    for i in range(1, T):
        ok[i] = ok[parent[i]] and ids[i] < V and ids[i] == pred[parent[i]]
        if ok[i] and depth[i] > depth[best]:
            best = i
    path = []
    while best >= 0:
        path.insert(0, L + best)
        best = parent[best]
    K[:, :, L:L + len(path)] = K[:, :, path]
    Vv[:, :, :, L:L + len(path)] = Vv[:, :, :, path]
    return logits, K, Vv


def exact(case, seed):
    if case["kind"] == "tail":
        return None  # whole numbers and moved bytes
    W, seqs = _inputs(case, seed)
    got = [_exact_sequence(case, W, q) for q in seqs]
    none = [None] * len(seqs)
    return dict(path=none, n_path=none, next_tok=none, k=[g[1] for g in got], v=[g[2] for g in got],
                logits=torch.cat([g[0] for g in got]), pred=None)
