"""Cases whose time the framework is measured by.

Each case is one pass through the public entry points as a decoding program
makes it: the tree attention of all layers of a verify step, the LM head, the
decoder layers around the attention, the commit (acceptance and compaction),
a whole float32 verify step, and one round of the decoding loop.  Passes over
layers are captured once into a HIP graph and replayed, as ``DecodeLoop`` and
``bench.py`` do; the others call the entry points directly.

Sizes are the repository's own workload and decoder shapes (``workload.py``,
``model_workload.py``) and generic ones; ``draw`` spreads trie sizes, prefix
lengths, head counts, widths, layouts and options over the same ranges.
Inputs are made on the GPU from the seed; values follow the workloads'
distributions (K, V, Q and hidden rows N(0, 1), weights N(0, 0.02^2)).
"""

import concurrent.futures as cf
import dataclasses
import math

import numpy as np
import torch

from paper_2608_00814_amd import model_workload as mw
from paper_2608_00814_amd import ooo
from paper_2608_00814_amd import workload as wl
from paper_2608_00814_amd.decode import DecodeLoop, SidecarHint
from paper_2608_00814_amd.model import ModelRunner
from paper_2608_00814_amd.step import VerifyRunner

EPS = 1.0e-6
THETA = 1.0e6
BF = torch.bfloat16


def listed():
    return [
        # One round of the decoding loop on the 2-layer parity decoder (head_dim 64): the smallest whole call, all
        # launches, host packing, hint lanes and the result's way back.
        {"name": "round_small", "kind": "round", "model": "small-model", "hint": True},
        # A whole float32 verify step (one layer, 25-node trie) launched call by call: the float32 option.
        {"name": "step_fp32", "kind": "step_fp32", "Hq": 4, "Hkv": 1, "D": 64, "N": 25, "P": 128, "H": 256, "V": 1024},
        # Tree attention of all 28 layers of a small target (Qwen3-0.6B shape): 32 nodes, short prefix.
        {"name": "attn_0.6b_32", "kind": "attn", "layers": 28, "Hq": 16, "Hkv": 8, "D": 128, "N": 32, "P": 1024,
         "dev": False},
        # ... of all 36 layers at the Qwen3-8B shape, the ordinary verify step.
        {"name": "attn_8b_64", "kind": "attn", "layers": 36, "Hq": 32, "Hkv": 8, "D": 128, "N": 64, "P": 4096,
         "dev": False},
        # ... of 4 layers late in a long decode (Llama-3.1-8B shape): the largest trie, a ragged prefix past 32k read
        # from device memory, as replayed rounds read it.
        {"name": "attn_long_256", "kind": "attn", "layers": 4, "Hq": 32, "Hkv": 8, "D": 128, "N": 256, "P": 36217,
         "dev": True},
        # LM head and greedy tokens: the ordinary 64-node trie, and the wide ones of the two larger workloads.
        {"name": "lmhead_8b_64", "kind": "lmhead", "N": 64, "H": 4096, "V": 151936, "packed": True, "logits": False},
        {"name": "lmhead_32b_128", "kind": "lmhead", "N": 128, "H": 5120, "V": 152064, "packed": True,
         "logits": False},
        {"name": "lmhead_llama_256", "kind": "lmhead", "N": 256, "H": 4096, "V": 128256, "packed": True,
         "logits": False},
        # Decoder layers over the trie (embedding rows, norms, projections, rotation, attention, MLP): plain decoding
        # (one node), the ordinary trie, and a wide trie of a larger target.
        {"name": "layers_8b_1", "kind": "layers", "layers": 2, "Hq": 32, "Hkv": 8, "D": 128, "H": 4096, "I": 12288,
         "N": 1, "P": 4096, "packed": True, "dev": True},
        {"name": "layers_8b_64", "kind": "layers", "layers": 2, "Hq": 32, "Hkv": 8, "D": 128, "H": 4096, "I": 12288,
         "N": 64, "P": 4096, "packed": True, "dev": True},
        {"name": "layers_32b_128", "kind": "layers", "layers": 1, "Hq": 40, "Hkv": 8, "D": 128, "H": 5120, "I": 27648,
         "N": 128, "P": 8192, "packed": True, "dev": False},
        # Acceptance and cache compaction of all layers of a verify step.
        {"name": "commit_8b_64", "kind": "commit", "layers": 36, "Hkv": 8, "D": 128, "N": 64, "P": 4096, "depth": 40,
         "accept": 23, "dev": False},
    ]


# ---------------------------------------------------------------- drawing


def _log(rng, lo, hi):
    """An integer between lo and hi, its logarithm spread evenly."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["attn", "attn", "attn", "lmhead", "lmhead", "layers", "layers", "layers", "commit", "step_fp32"])
    if kind == "step_fp32":
        D = rng.choice([64, 128])
        Hkv = rng.choice([1, 2, 4])
        return {"kind": kind, "Hq": Hkv * rng.choice([1, 2, 4]), "Hkv": Hkv, "D": D, "N": _log(rng, 1, 64),
                "P": _log(rng, 1, 1024), "H": 64 * _log(rng, 1, 16), "V": _log(rng, 500, 8000)}
    if kind == "commit":
        N = _log(rng, 2, 256)
        depth = rng.randint(1, min(64, N - 1))
        return {"kind": kind, "layers": _log(rng, 2, 36), "Hkv": rng.choice([2, 4, 8]), "D": rng.choice([64, 128]),
                "N": N, "P": _log(rng, 1, 8192), "depth": depth, "accept": rng.randint(0, depth),
                "dev": rng.random() < 0.5}
    if kind == "lmhead":
        H = 64 * rng.choice([4, 16, 16, 32, 64, 64, 80])
        V = _log(rng, 1000, 152064)
        N = _log(rng, 1, 256)
        return {"kind": kind, "N": N, "H": H, "V": V, "packed": rng.random() < 0.8,
                "logits": N * V < 4_000_000 and rng.random() < 0.3}
    N = _log(rng, 1, 256)
    Hq, Hkv = rng.choice([(16, 8), (32, 8), (32, 8), (40, 8), (4, 1), (8, 4), (8, 8), (14, 2)])
    D = rng.choice([64, 128, 128, 128])
    if kind == "attn":
        P = _log(rng, 16, 40000)
        cost = 4 * Hq * N * P * D + 2e2 * (4 * Hkv * P * D)
        return {"kind": kind, "layers": max(1, min(28, int(3e11 / cost))), "Hq": Hq, "Hkv": Hkv, "D": D, "N": N,
                "P": P, "dev": rng.random() < 0.5}
    while (Hq + 2 * Hkv) * D % 128:
        Hkv *= 2
        Hq *= 2
    H = 64 * rng.choice([8, 16, 16, 32, 40, 64, 64, 80])
    I = 128 * max(2, round(H * rng.choice([2.0, 2.75, 3.0, 3.5, 5.4]) / 128))
    return {"kind": kind, "layers": 1 if H > 4096 else 2, "Hq": Hq, "Hkv": Hkv, "D": D, "H": H, "I": I, "N": N,
            "P": _log(rng, 16, 8192), "packed": rng.random() < 0.85, "dev": rng.random() < 0.5}


# ----------------------------------------------------------------- inputs


def _gen(seed, stream):
    g = torch.Generator(device="cuda")
    g.manual_seed((int(seed) * 1000003 + stream) & 0x7FFFFFFFFFFF)
    return g


def _randn(shape, seed, stream, std=1.0, dtype=BF, mean=0.0):
    g = _gen(seed, stream)
    out = torch.empty(shape, dtype=dtype, device="cuda")
    flat = out.view(-1)
    step = 1 << 26
    for i in range(0, flat.numel(), step):
        n = min(step, flat.numel() - i)
        flat[i:i + n] = torch.randn(n, generator=g, device="cuda").mul_(std).add_(mean)
    return out


def _trie(N, depth, seed, vocab=100000):
    """A trie of exactly N nodes: a spine, then branches off it (drafts sharing a prefix), each with fresh tokens."""
    r = np.random.default_rng(int(seed) % (1 << 32))
    spine = [int(t) for t in r.integers(0, vocab, size=depth)]
    cands, fresh, made = [spine], vocab, 1 + len(spine)
    while made < N:
        at = int(r.integers(0, max(1, depth)))
        n = int(min(r.integers(1, 13), max(1, depth - at)))
        cands.append(spine[:at] + list(range(fresh, fresh + n)))
        fresh += n
        made += n
    offs = np.cumsum([0] + [len(c) for c in cands]).astype(np.int32)
    flat = np.array([t for c in cands for t in c], np.int32)
    t = ooo.pack_tree(int(r.integers(0, vocab)), flat, offs, N, depth)
    assert t["n_nodes"] == N, (t["n_nodes"], N)
    return t


def _trie_depth(N):
    return max(0, min(64, N - 1, 8 + N // 2))


def _mask(t):
    return torch.from_numpy(t["anc_mask"].view(np.int64).reshape(t["n_nodes"], -1).copy()).cuda()


def _graph(fn):
    """fn's launches as a replayable graph, captured as DecodeLoop captures a round."""
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        fn()
    return g


def _cap(c):
    return c["P"] + c["N"] + 7


def _attn_inputs(c, seed):
    L, N, Hq, Hkv, D = c["layers"], c["N"], c["Hq"], c["Hkv"], c["D"]
    q = _randn((L, N, Hq, D), seed, 1)
    k = _randn((L, Hkv, _cap(c), D), seed, 2)
    v = _randn((L, Hkv, _cap(c), D), seed, 3)
    return q, k, v, _trie(N, _trie_depth(N), seed)


def _bound(c):
    """Prefix bound of the launches: the prefix itself, or for replays the capacity a decode loop plans for."""
    return _cap(c) - c["N"] if c["dev"] else c["P"]


def _workspace(nbytes):
    return torch.zeros(max(nbytes, 256) // 4 + 1, dtype=torch.float32, device="cuda")


def _prefix_dev(c):
    return torch.tensor([c["P"]], dtype=torch.int32, device="cuda") if c["dev"] else None


def _prepare_attn(c, seed):
    q, k, v, t = _attn_inputs(c, seed)
    N, Hq, Hkv, D = c["N"], c["Hq"], c["Hkv"], c["D"]
    out = torch.zeros_like(q)
    ws = _workspace(ooo.tree_attn_workspace(N, Hq, Hkv, D, _bound(c), ooo.BF16))
    mask, pd = _mask(t), _prefix_dev(c)

    def step():
        for l in range(c["layers"]):
            ooo.tree_attn(q[l], k[l], v[l], _bound(c), N, mask, Hq, Hkv, 1.0 / math.sqrt(D), out[l], ws,
                          prefix_dev=pd)

    return {"kind": "attn", "graph": _graph(step), "out": out, "keep": (q, k, v, mask, pd, ws)}


def _prepare_lmhead(c, seed):
    x, w = _randn((c["N"], c["H"]), seed, 1), _randn((c["V"], c["H"]), seed, 2, 0.02)
    weight = ooo.lmhead_pack(w) if c["packed"] else w
    torch.cuda.synchronize()
    return {"kind": "lmhead", "x": x, "w": weight, "ids": torch.zeros(c["N"], dtype=torch.int32, device="cuda"),
            "max": torch.zeros(c["N"], dtype=torch.float32, device="cuda"),
            "logits": torch.empty(c["N"], c["V"], dtype=torch.float32, device="cuda") if c["logits"] else None,
            "ws": _workspace(ooo.lmhead_workspace(c["N"], c["H"], c["V"], ooo.BF16))}


EMB_ROWS = 4096  # rows of the embedding table (a pass reads one row a node)


def _layer_weights(c, seed, l):
    H, I, D, Hq, Hkv = c["H"], c["I"], c["D"], c["Hq"], c["Hkv"]
    r = lambda j, shape, std=0.02, mean=0.0: _randn(shape, seed, 100 + 16 * l + j, std, mean=mean)
    return {"in": r(0, (H,), 0.1, 1.0), "qkv": r(1, ((Hq + 2 * Hkv) * D, H)), "qn": r(2, (D,), 0.1, 1.0),
            "kn": r(3, (D,), 0.1, 1.0), "o": r(4, (H, Hq * D)), "post": r(5, (H,), 0.1, 1.0),
            "gu": r(6, (2 * I, H)), "down": r(7, (H, I))}


def _layers_inputs(c, seed):
    t = _trie(c["N"], _trie_depth(c["N"]), seed, EMB_ROWS // 2)
    tokens = torch.from_numpy((t["token"].astype(np.int64) % EMB_ROWS).astype(np.int32)).cuda()
    emb, fin = _randn((EMB_ROWS, c["H"]), seed, 4), _randn((c["H"],), seed, 5, 0.1, mean=1.0)
    k = _randn((c["layers"], c["Hkv"], _cap(c), c["D"]), seed, 2)
    v = _randn((c["layers"], c["Hkv"], _cap(c), c["D"]), seed, 3)
    return t, tokens, emb, fin, k, v


def _prepare_layers(c, seed):
    t, tokens, emb, fin, k, v = _layers_inputs(c, seed)
    N, H, I, D, Hq, Hkv = c["N"], c["H"], c["I"], c["D"], c["Hq"], c["Hkv"]
    ws = []
    for l in range(c["layers"]):
        w = _layer_weights(c, seed, l)
        ws.append({n: ooo.linear_pack(x) if c["packed"] and x.dim() == 2 else x for n, x in w.items()})
        torch.cuda.synchronize()
    depth = torch.from_numpy(t["depth"].astype(np.int32).copy()).cuda()
    new = lambda *shape, dt=BF: torch.zeros(shape, dtype=dt, device="cuda")
    h, x, xf = new(N, H, dt=torch.float32), new(N, H), new(N, H)
    q, o, act = new(N, Hq, D), new(N, Hq, D), new(N, I)
    lin = _workspace(max(ooo.linear_workspace(N, a, b)
                         for a, b in ((H, (Hq + 2 * Hkv) * D), (Hq * D, H), (H, 2 * I), (I, H))))
    aws = _workspace(ooo.tree_attn_workspace(N, Hq, Hkv, D, _bound(c), ooo.BF16))
    mask, pd, P = _mask(t), _prefix_dev(c), _bound(c)

    def step():
        ooo.embed_rows(emb, tokens, N, h)
        ooo.rmsnorm(h, ws[0]["in"], EPS, x)
        for l, w in enumerate(ws):
            last = l + 1 == len(ws)
            ooo.linear_qk_norm_rope(x, w["qkv"], w["qn"], w["kn"], EPS, depth, N, P, THETA, Hq, Hkv, q, k[l], v[l],
                                    lin, prefix_dev=pd)
            ooo.tree_attn(q, k[l], v[l], P, N, mask, Hq, Hkv, 1.0 / math.sqrt(D), o, aws, prefix_dev=pd)
            ooo.linear_add_rmsnorm(o.view(N, Hq * D), w["o"], h, w["post"], EPS, x, lin)
            ooo.linear(x, w["gu"], act, ooo.EPI_SWIGLU_BF16, lin)
            ooo.linear_add_rmsnorm(act, w["down"], h, fin if last else ws[l + 1]["in"], EPS, xf if last else x, lin)

    rows = slice(c["P"], c["P"] + N)  # the cache rows that the pass writes
    return {"kind": "layers", "graph": _graph(step),
            "out": {"residual": h, "final": xf, "k": k[:, :, rows], "v": v[:, :, rows]},
            "keep": (ws, emb, tokens, depth, mask, pd, lin, aws, x, q, o, act, fin)}


def _commit_inputs(c, seed):
    """A trie and greedy tokens that accept `accept` drafts along its first branch."""
    t = _trie(c["N"], c["depth"], seed)
    ids = np.full(c["N"], 7_000_000, np.int32)
    node = 0
    for _ in range(c["accept"]):
        child = next(i for i in range(c["N"]) if t["parent"][i] == node)
        ids[node] = t["token"][child]
        node = child
    k = _randn((c["layers"], c["Hkv"], _cap(c), c["D"]), seed, 2)
    v = _randn((c["layers"], c["Hkv"], _cap(c), c["D"]), seed, 3)
    return t, ids, k, v


def _prepare_commit(c, seed):
    t, ids, k, v = _commit_inputs(c, seed)
    i32 = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).cuda()
    return {"kind": "commit", "c": c, "token": i32(t["token"]), "parent": i32(t["parent"]), "depth": i32(t["depth"]),
            "mask": _mask(t), "ids": i32(ids), "k": k, "v": v, "pd": _prefix_dev(c), "bound": _bound(c),
            "path": torch.zeros(c["depth"] + 1, dtype=torch.int32, device="cuda"),
            "len": torch.zeros(1, dtype=torch.int32, device="cuda"),
            "bonus": torch.zeros(1, dtype=torch.int32, device="cuda")}


def _fp32_inputs(c, seed):
    f = torch.float32
    N = c["N"]
    q = _randn((N, c["Hq"], c["D"]), seed, 1, dtype=f)
    k = _randn((1, c["Hkv"], _cap(c), c["D"]), seed, 2, dtype=f)
    v = _randn((1, c["Hkv"], _cap(c), c["D"]), seed, 3, dtype=f)
    return q, k, v, _randn((N, c["H"]), seed, 4, dtype=f), _randn((c["V"], c["H"]), seed, 5, 0.02, dtype=f)


def _fp32_candidates(c, seed):
    t = _trie(c["N"], _trie_depth(c["N"]), seed, c["V"])
    cands = []
    for i in range(c["N"]):
        seq, j = [], i
        while j > 0:
            seq.append(int(t["token"][j]))
            j = int(t["parent"][j])
        cands.append(seq[::-1])
    offs = np.cumsum([0] + [len(s) for s in cands]).astype(np.int32)
    return int(t["token"][0]), np.array([x for s in cands for x in s], np.int32), offs


def _prepare_fp32(c, seed):
    q, k, v, x, w = _fp32_inputs(c, seed)
    vr = VerifyRunner(1, c["Hq"], c["Hkv"], c["D"], c["H"], c["V"], c["N"], _trie_depth(c["N"]), torch.float32,
                      max_prefix=c["P"])
    vr.set_weight(w)
    return {"kind": "step_fp32", "c": c, "vr": vr, "cand": _fp32_candidates(c, seed), "q": q, "k": k, "v": v, "x": x,
            "logits": torch.empty(c["N"], c["V"], dtype=torch.float32, device="cuda")}


def _round_model(c, seed):
    """Decoder weights whose greedy next token of t is perm(t) by a wide margin (embeddings times 16, LM-head rows the
    permuted embedding rows), so that tokens do not hang on the last bit of a logit."""
    cfg = mw.MODEL_CONFIGS[c["model"]]
    seed = int(seed) % (1 << 31)
    layers = [mw.layer_weights(cfg, seed, l) for l in range(cfg.n_layers)]
    emb = wl.to_bf16_bits(wl.bf16_to_f32(mw.embedding(cfg, seed)) * 16.0)
    perm = np.random.default_rng(seed).permutation(cfg.vocab)
    lm = np.empty_like(emb)
    lm[perm] = mw.embedding(cfg, seed)
    kv = [mw.prefix_kv(cfg, seed, l) for l in range(cfg.n_layers)]
    root = mw.random_tokens(cfg, seed, 1)[0]
    chain = [root]
    for _ in range(cfg.max_depth):
        chain.append(int(perm[chain[-1]]))
    r = np.random.default_rng(seed + 1)
    wrong = lambda n: [int(x) for x in r.integers(0, cfg.vocab - 1, size=n)]
    # two native candidates that follow the target for some tokens, and hint views, one of which does so for longer
    native = [chain[1:4] + wrong(6), chain[1:3] + wrong(5)]
    views = [wrong(40), wrong(3) + chain[:8] + wrong(9), wrong(40)]
    return cfg, layers, emb, mw.final_norm(cfg, seed), lm, kv, root, native, views


def _prepare_round(c, seed):
    cfg, layers, emb, fin, lm, kv, root, native, views = _round_model(c, seed)
    model = ModelRunner(cfg, layers, emb, fin, lm)
    dev = lambda arrs: torch.stack([torch.from_numpy(a.view(np.int16)).view(BF) for a in arrs]).cuda()
    k, v = dev([a for a, _ in kv]), dev([b for _, b in kv])
    hint = None
    if c["hint"]:
        done = cf.Future()
        done.set_result(views)
        hint = SidecarHint(done, cfg.vocab - 1)
    loop = DecodeLoop(model, k, v, cfg.prefix_len, root, lambda r, y: native, hint)
    loop.round()  # captures the round's graph, as the first round of a request does
    return {"kind": "round", "loop": loop, "cfg": cfg, "root": root, "k": k, "v": v}


def prepare(case, seed):
    return {"attn": _prepare_attn, "lmhead": _prepare_lmhead, "layers": _prepare_layers, "commit": _prepare_commit,
            "step_fp32": _prepare_fp32, "round": _prepare_round}[case["kind"]](case, seed)


# -------------------------------------------------------------------- run


def run(s):
    kind = s["kind"]
    if kind in ("attn", "layers"):
        s["graph"].replay()
        return s["out"]
    if kind == "lmhead":
        ooo.lmhead_argmax(s["x"], s["w"], s["ids"], s["max"], s["logits"], s["ws"])
        return {"ids": s["ids"], "max_logit": s["max"], "logits": s["logits"]}
    if kind == "commit":
        c = s["c"]
        ooo.accept(s["token"], s["parent"], s["depth"], s["mask"], s["ids"], c["N"], s["path"], s["len"], s["bonus"],
                   max_depth=c["depth"])
        ooo.kv_compact(s["k"], s["v"], s["bound"], c["N"], s["path"], s["len"], prefix_dev=s["pd"])
        return {"path": s["path"], "len": s["len"], "bonus": s["bonus"], "k": s["k"], "v": s["v"]}
    if kind == "step_fp32":
        vr, c = s["vr"], s["c"]
        vr.pack(*s["cand"], keep=False)
        vr.device_step([s["q"]], s["k"], s["v"], s["x"], c["P"], logits=s["logits"])
        return {"out": vr.out, "logits": s["logits"], "ids": vr.ids, "max_logit": vr.max_logit, "result": vr.res}
    # a new request on the same prefix: its first round
    loop, cfg = s["loop"], s["cfg"]
    loop.P, loop.committed, loop.rounds = cfg.prefix_len, [s["root"]], 0
    rec = loop.round()
    n, vr = rec.n_nodes, loop.model.vr
    return {"tokens": np.array(rec.committed, np.int64), "nodes": n, "final": loop.model.xf[:n],
            "ids": vr.ids[:n], "max_logit": vr.max_logit[:n], "k": s["k"], "v": s["v"]}


# ------------------------------------------------------------------- work


def work(case):
    c = case
    if c["kind"] == "attn":
        one = 2 * 2 * c["Hkv"] * (c["P"] + c["N"]) * c["D"] + 2 * 2 * c["N"] * c["Hq"] * c["D"]
        return {"bytes": c["layers"] * one, "flops": c["layers"] * 4.0 * c["Hq"] * c["N"] * (c["P"] + c["N"]) * c["D"]}
    if c["kind"] == "lmhead":
        b = 2.0 * c["V"] * c["H"] + 2 * c["N"] * c["H"] + 8 * c["N"] + (4.0 * c["N"] * c["V"] if c["logits"] else 0)
        return {"bytes": b, "flops": 2.0 * c["N"] * c["V"] * c["H"]}
    if c["kind"] == "layers":
        return _layers_work(c["layers"], c["Hq"], c["Hkv"], c["D"], c["H"], c["I"], c["N"], c["P"])
    if c["kind"] == "commit":
        moved = 2.0 * c["layers"] * c["Hkv"] * c["accept"] * c["D"] * 2
        return {"bytes": 2 * moved + c["N"] * (16 + 8 * ((c["N"] + 63) // 64)) + 4 * c["depth"], "flops": 0.0}
    if c["kind"] == "step_fp32":
        keys = c["P"] + c["N"]
        b = 4.0 * (2 * c["Hkv"] * keys * c["D"] + 2 * c["N"] * c["Hq"] * c["D"] + c["V"] * c["H"] + c["N"] * c["H"] +
                   c["N"] * c["V"])
        return {"bytes": b, "flops": 4.0 * c["Hq"] * c["N"] * keys * c["D"] + 2.0 * c["N"] * c["V"] * c["H"]}
    m, n = mw.MODEL_CONFIGS[c["model"]], 16
    w = _layers_work(m.n_layers, m.n_q_heads, m.n_kv_heads, m.head_dim, m.hidden, m.intermediate, n, m.prefix_len)
    return {"bytes": w["bytes"] + 2.0 * m.vocab * m.hidden, "flops": w["flops"] + 2.0 * n * m.vocab * m.hidden}


def _layers_work(L, Hq, Hkv, D, H, I, N, P):
    weights = (Hq + 2 * Hkv) * D * H + H * Hq * D + 3 * I * H
    kv = 2 * 2 * Hkv * (P + N) * D
    return {"bytes": L * (2.0 * weights + kv + 2 * 2 * Hkv * N * D) + 2 * N * H + 4 * N * H + 2 * N * H,
            "flops": L * (2.0 * N * weights + 4.0 * Hq * N * (P + N) * D)}


def tolerance(case):
    return {"attn": {"rel": 1e-2}, "lmhead": {"rel": 1e-5}, "layers": {"rel": 1e-2}, "commit": "exact",
            "step_fp32": {"rel": 1e-5}, "round": {"rel": 1e-2}}[case["kind"]]


# ------------------------------------------------------------------ exact


def _allowed(t, P):
    """[N][P + N] whether node i sees key j, from the parents."""
    N = t["n_nodes"]
    a = np.zeros((N, P + N), bool)
    a[:, :P] = True
    for i in range(N):
        j = i
        while j >= 0:
            a[i, P + j] = True
            j = int(t["parent"][j])
    return torch.from_numpy(a).cuda()


def _attn64(q, k, v, P, t):
    """q [N][Hq][D], k and v [Hkv][rows][D] -> [N][Hq][D] in float64."""
    N, Hq, D = q.shape
    G = Hq // k.shape[0]
    ok = _allowed(t, P)
    out = torch.empty(N, Hq, D, dtype=torch.float64, device="cuda")
    for g in range(k.shape[0]):
        kk, vv = k[g, :P + N].double(), v[g, :P + N].double()
        for hd in range(g * G, (g + 1) * G):
            s = (q[:, hd].double() @ kk.t()) / math.sqrt(D)
            s.masked_fill_(~ok, -math.inf)
            out[:, hd] = torch.softmax(s, dim=1) @ vv
    return out


def _norm64(x, w):
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + EPS) * w.double()


def _rope64(x, pos, theta):
    D = x.shape[-1]
    f = theta ** (-2.0 * torch.arange(D // 2, dtype=torch.float64, device="cuda") / D)
    a = (pos[:, None] * f)[:, None, :]
    x1, x2 = x[..., :D // 2], x[..., D // 2:]
    return torch.cat([x1 * a.cos() - x2 * a.sin(), x2 * a.cos() + x1 * a.sin()], -1)


def _mm64(x, w):
    """x w^T in float64, the weight widened a slice at a time."""
    step = max(1, (1 << 27) // w.shape[1])
    return torch.cat([x @ w[i:i + step].double().t() for i in range(0, w.shape[0], step)], 1)


def _layers64(h, layers, fin, k, v, P, t, Hq, Hkv, D, I, theta):
    N = h.shape[0]
    pos = P + torch.from_numpy(t["depth"].astype(np.float64)).cuda()
    ks, vs = [], []
    for l, w in enumerate(layers):
        qkv = _mm64(_norm64(h, w["in"]), w["qkv"]).view(N, Hq + 2 * Hkv, D)
        q = _rope64(_norm64(qkv[:, :Hq], w["qn"]), pos, theta)
        kn = _rope64(_norm64(qkv[:, Hq:Hq + Hkv], w["kn"]), pos, theta)
        vn = qkv[:, Hq + Hkv:]
        kk, vv = k[l, :, :P + N].double(), v[l, :, :P + N].double()
        kk[:, P:], vv[:, P:] = kn.transpose(0, 1), vn.transpose(0, 1)
        ks.append(kn.transpose(0, 1))
        vs.append(vn.transpose(0, 1))
        h = h + _mm64(_attn64(q, kk, vv, P, t).reshape(N, Hq * D), w["o"])
        gu = _mm64(_norm64(h, w["post"]), w["gu"])
        h = h + _mm64(torch.nn.functional.silu(gu[:, :I]) * gu[:, I:], w["down"])
    return h, _norm64(h, fin), torch.stack(ks), torch.stack(vs)


def exact(case, seed):
    c = case
    if c["kind"] == "attn":
        q, k, v, t = _attn_inputs(c, seed)
        return torch.stack([_attn64(q[l], k[l], v[l], c["P"], t) for l in range(c["layers"])])
    if c["kind"] == "lmhead":
        x, w = _randn((c["N"], c["H"]), seed, 1).double(), _randn((c["V"], c["H"]), seed, 2, 0.02)
        y = _mm64(x, w)
        return {"ids": None, "max_logit": y.max(1).values, "logits": y if c["logits"] else None}
    if c["kind"] == "layers":
        t, tokens, emb, fin, k, v = _layers_inputs(c, seed)
        ws = [_layer_weights(c, seed, l) for l in range(c["layers"])]
        h, x, ks, vs = _layers64(emb[tokens.long()].double(), ws, fin, k, v, c["P"], t, c["Hq"], c["Hkv"], c["D"],
                                 c["I"], THETA)
        return {"residual": h, "final": x, "k": ks, "v": vs}
    if c["kind"] == "commit":
        t, ids, k, v = _commit_inputs(c, seed)
        node, path = 0, [0]
        while True:
            child = next((i for i in range(c["N"]) if t["parent"][i] == node and t["token"][i] == ids[node]), None)
            if child is None:
                break
            path.append(child)
            node = child
        src = torch.tensor(path, device="cuda") + c["P"]
        for x in (k, v):
            x[:, :, c["P"]:c["P"] + len(path)] = x[:, :, src]
        return {"path": None, "len": None, "bonus": None, "k": k.double(), "v": v.double()}
    if c["kind"] == "step_fp32":
        q, k, v, x, w = _fp32_inputs(c, seed)
        root, flat, offs = _fp32_candidates(c, seed)
        t = ooo.pack_tree(root, flat, offs, c["N"], _trie_depth(c["N"]))
        y = _mm64(x.double(), w)
        return {"out": _attn64(q, k[0], v[0], c["P"], t)[None], "logits": y, "ids": None,
                "max_logit": y.max(1).values, "result": None}
    cfg, layers, emb, fin, lm, kv, root, native, views = _round_model(c, seed)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a).view(np.int16)).view(BF).cuda()
    lanes = native
    if c["hint"]:
        bank = np.array([x for w in views for x in list(w) + [cfg.vocab - 1]], np.int32)
        offs = np.cumsum([0] + [len(s) for s in native]).astype(np.int32)
        m = ooo.hint_merge(bank, cfg.vocab - 1, np.array([root], np.int32),
                           np.array([x for s in native for x in s], np.int32), offs, 8, max_len=cfg.max_depth)
        lanes = [m["tokens"][m["offsets"][i]:m["offsets"][i + 1]].tolist() for i in range(m["n_out"])]
    offs = np.cumsum([0] + [len(s) for s in lanes]).astype(np.int32)
    t = ooo.pack_tree(root, np.array([x for s in lanes for x in s], np.int32), offs, cfg.max_nodes, cfg.max_depth)
    ws = [{"in": dev(w["in_norm"]), "qkv": dev(w["w_qkv"]), "qn": dev(w["q_norm"]), "kn": dev(w["k_norm"]),
           "o": dev(w["w_o"]), "post": dev(w["post_norm"]),
           "gu": torch.cat([dev(w["w_gate"]), dev(w["w_up"])]), "down": dev(w["w_down"])} for w in layers]
    e = dev(emb)
    h = e[torch.from_numpy(t["token"].astype(np.int64)).cuda()].double()
    k, v = (torch.stack([dev(a[i]) for a in kv]) for i in range(2))
    _, x, _, _ = _layers64(h, ws, dev(fin), k, v, cfg.prefix_len, t, cfg.n_q_heads, cfg.n_kv_heads, cfg.head_dim,
                           cfg.intermediate, cfg.rope_theta)
    y = _mm64(x, dev(lm))
    return {"tokens": None, "nodes": None, "final": x, "ids": None, "max_logit": y.max(1).values, "k": None, "v": None}
