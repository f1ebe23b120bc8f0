"""The work that a serving program has this framework do, as cases that can be timed and compared.

Each case is one block of a decoder iteration called through the public entry points
(``paper_2505_05286_amd.hxf`` and ``device.Engine``), or one whole serving exchange of an engine.
The sizes are those of the model shapes and request streams in ``synth`` (iterations of 64 decode
rows, fork groups of 256 rows, mixed iterations of a 2048-token chunk plus 32 decodes, lone
requests); ``draw`` spreads further cases over the same ranges.
"""
import math
import random

import numpy as np
import torch

import synth
from paper_2505_05286_amd import hxf
from paper_2505_05286_amd.device import Engine

DEV = "cuda"
PAGE = 16
EPS, ROPE_BASE = 1e-5, 10000.0
MAX_POS = 9216


# ------------------------------------------------------------------ the cases
def listed():
    return [
        # a decode iteration's attention input: norm, QKV projection, RoPE and KV write of 64 sequences
        {"name": "qkv_decode_8b", "kind": "qkv", "model": "llama8b", "decode": 64, "prompt": 0},
        # the same of a mixed iteration: a 2048-token prompt chunk and 32 decodes
        {"name": "qkv_mixed_8b", "kind": "qkv", "model": "llama8b", "decode": 32, "prompt": 2048},
        # decode attention over 64 contexts around 3000 tokens
        {"name": "attn_decode_8b", "kind": "decode", "model": "llama8b", "seqs": 64, "median": 3000, "lengths": 1},
        # 8 candidate requests of each of 32 queries, forked from a 4000-token prompt, decoding together
        {"name": "attn_forks_8b", "kind": "forks", "model": "llama8b", "parents": 32, "forks": 8, "prefix": 4000,
         "tail": 130, "lengths": 2},
        # prompt attention: the last chunk of a long prompt and the first of the next one
        {"name": "attn_prompt_8b", "kind": "prefill", "model": "llama8b", "pos_a": 6144, "n_a": 1531, "pos_b": 0,
         "n_b": 517},
        # a lone request's decode step through one MLP: the lowest latency the weights allow
        {"name": "mlp_lone_8b", "kind": "mlp", "model": "llama8b", "rows": 1, "packed": False},
        # the MLP of a 64-sequence decode iteration, its hidden activations kept in the packed layout
        {"name": "mlp_decode_8b", "kind": "mlp", "model": "llama8b", "rows": 64, "packed": True},
        # fork groups decoding together on the 32B shape; an odd number of rows
        {"name": "mlp_forks_32b", "kind": "mlp", "model": "qwen32b", "rows": 251, "packed": True},
        # the MLP of a mixed iteration on the 70B shape, the largest call
        {"name": "mlp_mixed_70b", "kind": "mlp", "model": "llama70b", "rows": 2080, "packed": True},
        # final norm, LM head and greedy choice of 64 decoding sequences
        {"name": "head_decode_8b", "kind": "head", "model": "llama8b", "rows": 64},
        # whole engine exchange, small model: four prompts prefilled in chunks and decoded together (launch-bound)
        {"name": "serve_tiny", "kind": "serve", "model": "tiny", "layers": 2, "prompt": 160, "others": 3, "new": 8,
         "forks": 0, "chunk": 128},
        # whole engine exchange, three 8B layers: a prompt and a bystander in mixed iterations, then 8 forks decoding
        {"name": "serve_8b", "kind": "serve", "model": "llama8b", "layers": 3, "prompt": 1611, "others": 1, "new": 8,
         "forks": 8, "chunk": 2048},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["qkv", "decode", "forks", "prefill", "mlp", "mlp", "mlp", "head", "serve"])
    model = rng.choice(["llama8b", "llama8b", "qwen32b", "llama70b"])
    if kind == "qkv":
        c = {"decode": _log_int(rng, 1, 256), "prompt": rng.choice([0, 1]) * _log_int(rng, 16, 2048)}
        return {"kind": kind, "model": rng.choice([model, "tiny"]), **c}
    if kind == "decode":
        return {"kind": kind, "model": rng.choice([model, "tiny"]), "seqs": _log_int(rng, 1, 128),
                "median": _log_int(rng, 100, 6000), "lengths": rng.randrange(1 << 30)}
    if kind == "forks":
        return {"kind": kind, "model": model, "parents": _log_int(rng, 1, 32), "forks": rng.randint(2, 8),
                "prefix": _log_int(rng, 300, 4096), "tail": _log_int(rng, 4, 256), "lengths": rng.randrange(1 << 30)}
    if kind == "prefill":
        n_a = _log_int(rng, 16, 2048)
        n_b = min(_log_int(rng, 1, 1024), 2049 - n_a)
        return {"kind": kind, "model": model, "pos_a": rng.choice([0, rng.randint(1, 6144)]), "n_a": n_a, "pos_b": 0,
                "n_b": max(n_b, 0)}
    if kind == "mlp":
        return {"kind": kind, "model": model, "rows": _log_int(rng, 1, 2080), "packed": rng.random() < 0.7}
    if kind == "head":
        return {"kind": kind, "model": model, "rows": _log_int(rng, 1, 256)}
    if rng.random() < 0.6:
        return {"kind": "serve", "model": "tiny", "layers": 2, "prompt": rng.randint(20, 240),
                "others": rng.randint(0, 5), "new": rng.randint(2, 12), "forks": rng.choice([0, 0, 3]), "chunk": 128}
    return {"kind": "serve", "model": "llama8b", "layers": 3, "prompt": _log_int(rng, 200, 1200),
            "others": rng.randint(0, 2), "new": rng.randint(2, 8), "forks": rng.randint(2, 8), "chunk": 2048}


# ------------------------------------------------------------------ inputs
def _shape(case):
    return synth.model_shape(case["model"], case.get("layers"))


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed * 7919 + 17)
    return g


def _normal(g, shape, scale, dtype=torch.bfloat16):
    """N(0, scale) values, drawn in slices so that no large fp32 copy is held."""
    out = torch.empty(shape, dtype=dtype, device=DEV)
    flat = out.view(-1)
    step = 1 << 28
    for a in range(0, flat.numel(), step):
        part = flat[a:a + step]
        part.copy_(torch.randn(part.numel(), generator=g, device=DEV).mul_(scale))
    return out


def _gain(g, d):
    return (1.0 + 0.5 * (2.0 * torch.rand(d, generator=g, device=DEV) - 1.0)).to(torch.bfloat16)


def _packed(w):
    n, k = w.shape
    out = torch.empty(hxf.packed_weight_bytes(n, k) // 2, dtype=torch.bfloat16, device=DEV)
    hxf.op_pack_weight(w.data_ptr(), n, k, out.data_ptr(), _stream())
    return out


def _weight(g, n, k):
    """A projection matrix in the library's packed layout."""
    return _packed(_normal(g, (n, k), synth.weights.WEIGHT_STD))


def _stream():
    return torch.cuda.current_stream().cuda_stream


def _ws(nbytes):
    return torch.empty(max(int(nbytes), 256), dtype=torch.uint8, device=DEV)


def _i32(a):
    return torch.tensor(np.asarray(a, np.int32), device=DEV)


def _hidden(g, rows, d):
    return _normal(g, (rows, d), 1.0, torch.float32)


def _contexts(case):
    """(shared prefix pages per sequence group, contexts): context lengths belong to the case."""
    r = random.Random(case["lengths"])
    if case["kind"] == "forks":
        return [case["prefix"] + r.randint(1, case["tail"]) for _ in range(case["parents"] * case["forks"])]
    return [min(8192, max(16, int(round(r.lognormvariate(math.log(case["median"]), 0.5)))))
            for _ in range(case["seqs"])]


def _tables(case, ctx, g):
    """Block tables over a shuffled pool; the forks of one parent share its full pages."""
    seqs = []
    n = 0
    if case["kind"] == "forks":
        shared = case["prefix"] // PAGE
        for p in range(case["parents"]):
            common = list(range(n, n + shared))
            n += shared
            for f in range(case["forks"]):
                own = -(-ctx[p * case["forks"] + f] // PAGE) - shared
                seqs.append(common + list(range(n, n + own)))
                n += own
    else:
        for c in ctx:
            pages = -(-c // PAGE)
            seqs.append(list(range(n, n + pages)))
            n += pages
    perm = torch.randperm(n, generator=g, device=DEV).cpu().numpy()
    bt = np.zeros((len(seqs), max(len(s) for s in seqs)), np.int32)
    for i, s in enumerate(seqs):
        bt[i, :len(s)] = perm[s]
    return bt, n


def _pools(g, n_blocks, sh):
    n = n_blocks * sh.n_kv_heads * PAGE * sh.head_dim
    return _normal(g, (n,), 1.0), _normal(g, (n,), 1.0)


def _chunks(case):
    return [(case[p], case[n]) for p, n in (("pos_a", "n_a"), ("pos_b", "n_b")) if case[n] > 0]


class _Model:
    """Weights of a decoder in HBM, as device.Engine reads them."""

    def __init__(self, sh, g, keep):
        d, f, v = sh.d_model, sh.ffn_dim, sh.vocab
        self.shape, self.device = sh, DEV
        self.plain = {} if keep else None   # row-major copies, for the 64-bit forward only

        def mat(name, n, k):
            w = _normal(g, (n, k), synth.weights.WEIGHT_STD)
            if keep:
                self.plain[name] = w
            return _packed(w)
        self.embed = _normal(g, (v, d), synth.weights.WEIGHT_STD)
        self.norm = _gain(g, d)
        self.lm_head = mat("lm_head", v, d)
        self.layers = []
        for l in range(sh.n_layers):
            self.layers.append({
                "attn_norm": _gain(g, d), "ffn_norm": _gain(g, d), "wqkv": mat((l, "wqkv"), sh.qkv_dim, d),
                "wo": mat((l, "wo"), d, sh.q_dim), "w_gate": mat((l, "w_gate"), f, d), "w_up": mat((l, "w_up"), f, d),
                "w_down": mat((l, "w_down"), d, f)})

    def layer_ptrs(self):
        return [{k: t.data_ptr() for k, t in L.items()} for L in self.layers]


def _requests(case, seed):
    """The exchange's requests: (prompt ids, forced ids) of the parent and the others, forced ids of the forks."""
    sh = _shape(case)
    r = np.random.default_rng(seed + 101)

    def ids(n):
        return r.integers(0, sh.vocab, n).astype(np.int32)
    first = [(ids(case["prompt"]), ids(case["new"]))]
    first += [(ids(max(8, case["prompt"] * (k + 1) // (case["others"] + 1) + 3 * k)), ids(case["new"]))
              for k in range(case["others"])]
    return first, [ids(case["new"]) for _ in range(case["forks"])]


def _serve_state(case, seed, keep=False):
    sh = _shape(case)
    model = _Model(sh, _gen(seed), keep)
    first, forks = _requests(case, seed)
    longest = max(len(p) for p, _ in first) + 2 * case["new"] + 16
    total = sum(len(p) + case["new"] + 16 for p, _ in first) + len(forks) * (case["new"] + 48)
    return model, first, forks, longest, -(-total // PAGE) + len(first) + 2 * len(forks) + 8


def prepare(case, seed):
    g = _gen(seed)
    sh = _shape(case)
    d, hq, hkv, dh = sh.d_model, sh.n_q_heads, sh.n_kv_heads, sh.head_dim
    kind = case["kind"]
    s = {"case": case, "sh": sh}
    if kind == "serve":
        model, first, forks, longest, blocks = _serve_state(case, seed)
        cost, it = (200_000_000, 50_000, 10, 150_000_000), (500_000_000, 1000, 20, 1)
        eng = Engine(model, max_context=longest, n_blocks=blocks, max_seqs=16, chunk_tokens=case["chunk"],
                     cost_ps=cost, iter_ps=it)
        s.update(engine=eng, first=first, forks=forks, now=0)
        return s
    if kind == "qkv":
        rows = case["decode"] + case["prompt"]
        pages = case["decode"] + -(-case["prompt"] // PAGE)
        perm = torch.randperm(pages, generator=g, device=DEV).cpu().numpy()
        r = np.random.default_rng(seed)
        pos = np.concatenate([np.arange(case["prompt"]), r.integers(0, MAX_POS, case["decode"])]).astype(np.int32)
        slot = [perm[i // PAGE] * PAGE + i % PAGE for i in range(case["prompt"])]
        slot += [perm[pages - 1 - i] * PAGE + pos[case["prompt"] + i] % PAGE for i in range(case["decode"])]
        rope = torch.empty(MAX_POS * dh, dtype=torch.float32, device=DEV)
        hxf.op_rope_table(rope.data_ptr(), MAX_POS, dh, ROPE_BASE, _stream())
        ws = hxf.op_gemm_workspace_bytes(rows, sh.qkv_dim, d)
        n = pages * hkv * PAGE * dh
        s.update(rows=rows, x=_hidden(g, rows, d), gain=_gain(g, d), w=_weight(g, sh.qkv_dim, d), pos=_i32(pos),
                 slot=_i32(slot), rope=rope, ws=_ws(ws), ws_n=ws, pages=pages,
                 h=torch.empty(rows, d, dtype=torch.bfloat16, device=DEV),
                 qkv=torch.empty(rows, sh.qkv_dim, dtype=torch.bfloat16, device=DEV),
                 k=torch.zeros(n, dtype=torch.bfloat16, device=DEV), v=torch.zeros(n, dtype=torch.bfloat16, device=DEV))
    elif kind in ("decode", "forks"):
        ctx = _contexts(case)
        bt, blocks = _tables(case, ctx, g)
        b = len(ctx)
        k, v = _pools(g, blocks, sh)
        ws = hxf.op_decode_attention_workspace_bytes(b, hq, hkv, dh, ctx, bt, bt.shape[1])
        s.update(ctx=np.asarray(ctx, np.int32), bt_host=bt, bt=_i32(bt), blocks=blocks, k=k, v=v, ws=_ws(ws), ws_n=ws,
                 q=_normal(g, (b, hq, dh), 1.0), out=torch.empty(b, hq, dh, dtype=torch.bfloat16, device=DEV))
    elif kind == "prefill":
        chunks = _chunks(case)
        ctx = [p + n for p, n in chunks]
        bt, blocks = _tables(case, ctx, g)
        rows = sum(n for _, n in chunks)
        k, v = _pools(g, blocks, sh)
        ns = np.asarray([n for _, n in chunks], np.int32)
        ws = hxf.op_prefill_attention_workspace_bytes(len(chunks), hq, hkv, ns)
        s.update(pos0=np.asarray([p for p, _ in chunks], np.int32), n=ns,
                 row0=np.asarray(np.cumsum(ns) - ns, np.int32), bt=_i32(bt), bt_host=bt, blocks=blocks, k=k, v=v,
                 ws=_ws(ws), ws_n=ws, q=_normal(g, (rows, hq, dh), 1.0),
                 out=torch.empty(rows, hq, dh, dtype=torch.bfloat16, device=DEV))
    elif kind == "mlp":
        rows, f = case["rows"], sh.ffn_dim
        ws = max(hxf.op_gemm_workspace_bytes(rows, 2 * f, d), hxf.op_gemm_workspace_bytes(rows, d, f))
        s.update(rows=rows, x=_hidden(g, rows, d), gain=_gain(g, d), gate=_weight(g, f, d), up=_weight(g, f, d),
                 down=_weight(g, d, f), ws=_ws(ws), ws_n=ws,
                 h=torch.empty(rows, d, dtype=torch.bfloat16, device=DEV),
                 act=torch.empty(-(-rows // PAGE) * PAGE * f, dtype=torch.bfloat16, device=DEV))
    else:
        rows = case["rows"]
        ws = hxf.op_gemm_workspace_bytes(rows, sh.vocab, d)
        s.update(rows=rows, x=_hidden(g, rows, d), gain=_gain(g, d), w=_weight(g, sh.vocab, d), ws=_ws(ws), ws_n=ws,
                 h=torch.empty(rows, d, dtype=torch.bfloat16, device=DEV),
                 logits=torch.empty(rows, sh.vocab, dtype=torch.float32, device=DEV),
                 ids=torch.empty(rows, dtype=torch.int32, device=DEV))
    return s


# ------------------------------------------------------------------ one pass
def _serve(s):
    """Submit, step until idle, fork the retained prompt, step until idle; the logits of every
    request's last token."""
    inst = s["engine"].inst
    retain = len(s["forks"]) > 0
    logits = {}
    now = s["now"]

    def until_idle():
        nonlocal now
        while True:
            status, info = inst.step(now)
            if status == hxf.IDLE:
                return
            now += info["t_iter_us"]
            if info["n_finished"]:
                for c in inst.drain(64):
                    logits[c["id"]] = inst.last_logits(c["id"])
    ids = [inst.submit(now, k, 0, now, 10 ** 9, p, len(f), retain=retain and k == 0, forced=f)
           for k, (p, f) in enumerate(s["first"])]
    until_idle()
    if retain:
        parent = ids[0]
        ids += [inst.submit(now, 0, 1, now, 10 ** 9, np.zeros(0, np.int32), len(f), parent=parent, forced=f)
                for f in s["forks"]]
        until_idle()
        inst.release(parent)
    s["now"] = now
    return {"logits": [logits[i] for i in ids]}


def run(s):
    kind, sh, st = s["case"]["kind"], s["sh"], _stream()
    d, f, hq, hkv, dh = sh.d_model, sh.ffn_dim, sh.n_q_heads, sh.n_kv_heads, sh.head_dim
    if kind == "serve":
        return _serve(s)
    if kind == "qkv":
        t = s["rows"]
        hxf.op_rmsnorm(s["x"].data_ptr(), 0, s["gain"].data_ptr(), s["h"].data_ptr(), t, d, EPS, st)
        hxf.op_gemm(s["h"].data_ptr(), d, s["w"].data_ptr(), 0, s["qkv"].data_ptr(), sh.qkv_dim, t, sh.qkv_dim, d,
                    hxf.EPI_BF16, s["ws"].data_ptr(), s["ws_n"], st)
        hxf.op_rope_kv_write(s["qkv"].data_ptr(), s["pos"].data_ptr(), s["slot"].data_ptr(), s["rope"].data_ptr(),
                             s["k"].data_ptr(), s["v"].data_ptr(), s["pages"], t, hq, hkv, dh, st)
        return {"q": s["qkv"][:, :sh.q_dim], "k": s["k"], "v": s["v"]}
    if kind in ("decode", "forks"):
        b = len(s["ctx"])
        hxf.op_decode_attention(s["q"].data_ptr(), s["k"].data_ptr(), s["v"].data_ptr(), s["blocks"],
                                s["bt"].data_ptr(), s["bt"].shape[1], s["ctx"], s["out"].data_ptr(), b, hq, hkv, dh,
                                s["ws"].data_ptr(), s["ws_n"], st, bt_host=s["bt_host"])
        return {"out": s["out"]}
    if kind == "prefill":
        hxf.op_prefill_attention(s["q"].data_ptr(), s["k"].data_ptr(), s["v"].data_ptr(), s["blocks"],
                                 s["bt"].data_ptr(), s["bt"].shape[1], s["row0"], s["pos0"], s["n"],
                                 s["out"].data_ptr(), len(s["n"]), hq, hkv, dh, s["ws"].data_ptr(), s["ws_n"], st)
        return {"out": s["out"]}
    t = s["rows"]
    hxf.op_rmsnorm(s["x"].data_ptr(), 0, s["gain"].data_ptr(), s["h"].data_ptr(), t, d, EPS, st)
    if kind == "mlp":
        out, inp = (hxf.GEMM_C_PACKED, hxf.GEMM_A_PACKED) if s["case"]["packed"] else (0, 0)
        hxf.op_gemm(s["h"].data_ptr(), d, s["gate"].data_ptr(), s["up"].data_ptr(), s["act"].data_ptr(), f, t, 2 * f,
                    d, hxf.EPI_SWIGLU | out, s["ws"].data_ptr(), s["ws_n"], st)
        hxf.op_gemm(s["act"].data_ptr(), f, s["down"].data_ptr(), 0, s["x"].data_ptr(), d, t, d, f,
                    hxf.EPI_RESID | inp, s["ws"].data_ptr(), s["ws_n"], st)
        return {"x": s["x"]}
    hxf.op_gemm(s["h"].data_ptr(), d, s["w"].data_ptr(), 0, s["logits"].data_ptr(), sh.vocab, t, sh.vocab, d,
                hxf.EPI_F32, s["ws"].data_ptr(), s["ws_n"], st)
    hxf.op_argmax(s["logits"].data_ptr(), s["ids"].data_ptr(), t, sh.vocab, st)
    return {"logits": s["logits"], "ids": s["ids"]}


# ------------------------------------------------------------------ what a pass cannot do without
def work(case):
    sh = _shape(case)
    d, f, hq, hkv, dh, v = sh.d_model, sh.ffn_dim, sh.n_q_heads, sh.n_kv_heads, sh.head_dim, sh.vocab
    kind = case["kind"]
    kv_token = hkv * dh * 2 * 2
    if kind == "qkv":
        t = case["decode"] + case["prompt"]
        return {"bytes": 2 * d * sh.qkv_dim + t * (4 * d + 2 * sh.qkv_dim + 4 * dh), "flops": 2 * t * d * sh.qkv_dim}
    if kind in ("decode", "forks"):
        ctx = _contexts(case)
        tokens = sum(ctx)
        if kind == "forks":
            shared = case["prefix"] // PAGE * PAGE
            tokens -= case["parents"] * (case["forks"] - 1) * shared
        return {"bytes": tokens * kv_token + len(ctx) * hq * dh * 4, "flops": 4 * dh * hq * sum(ctx)}
    if kind == "prefill":
        pairs = sum(n * p + n * (n + 1) // 2 for p, n in _chunks(case))
        rows = sum(n for _, n in _chunks(case))
        return {"bytes": sum(p + n for p, n in _chunks(case)) * kv_token + rows * hq * dh * 4,
                "flops": 4 * dh * hq * pairs}
    if kind == "mlp":
        return {"bytes": 6 * d * f + case["rows"] * d * 8, "flops": 6 * case["rows"] * d * f}
    if kind == "head":
        return {"bytes": 2 * v * d + case["rows"] * (4 * d + 4 * v), "flops": 2 * case["rows"] * v * d}
    first, forks = _requests(case, 0)
    chunks = -(-sum(len(p) for p, _ in first) // case["chunk"])
    layers = sh.n_layers * sh.params_per_layer()
    steps = chunks + case["new"] - 1 + (case["new"] if forks else 0)   # each reads every weight once
    tokens = sum(len(p) + case["new"] - 1 for p, _ in first) + len(forks) * case["new"]
    rows = (len(first) + len(forks)) * case["new"]
    return {"bytes": steps * 2 * (layers + v * d), "flops": 2 * tokens * layers + 2 * rows * v * d}


def tolerance(case):
    # About four times the measured distance to the 64-bit result: bf16 outputs of one projection (2.9e-3 after
    # norm, projection and rotation) or one attention (2.2e-3), the MLP's bf16 hidden activations (2.9e-3), logits
    # that see only the normed row's rounding (1.7e-3), and a whole model's logits, which see the roundings of
    # all its layers (5e-3 for the two small layers, 1.8e-2 for the three large ones).
    return {
        "qkv": {"rel": 1.2e-2},
        "decode": {"rel": 9e-3},
        "forks": {"rel": 9e-3},
        "prefill": {"rel": 8e-3},
        "mlp": {"rel": 1.2e-2},
        "head": {"rel": 7e-3, "differ": 0.01},
        "serve": {"rel": 2e-2 if case["model"] == "tiny" else 3e-2},
    }[case["kind"]]


# ------------------------------------------------------------------ the same in 64 bits
def _norm64(x, gain):
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + EPS) * gain.double()


def _unpack64(w, n, k):
    """A packed matrix (16 x 32 tiles, [k%32 / 8][row][k%8] inside) back in rows, in 64 bits."""
    kt = -(-k // 32)
    t = w.view(-(-n // 16), kt, 4, 16, 8).permute(0, 3, 1, 2, 4).reshape(-1, kt * 32)
    return t[:n, :k].double()


def _matmul64(a, w, n, k, step=4096):
    """a . w^T for a packed w, a slice of its rows at a time."""
    kt = -(-k // 32)
    return torch.cat([a @ _unpack64(w[r // 16 * kt * 512:], min(step, n - r), k).T if r + step >= n else
                      a @ _unpack64(w[r // 16 * kt * 512:(r + step) // 16 * kt * 512], step, k).T
                      for r in range(0, n, step)], 1)


def _rope64(x, pos):
    half = x.shape[-1] // 2
    theta = ROPE_BASE ** (-2.0 * torch.arange(half, dtype=torch.float64, device=DEV) / x.shape[-1])
    a = pos.double()[:, None, None] * theta
    u, v = x[..., :half], x[..., half:]
    return torch.cat([u * a.cos() - v * a.sin(), v * a.cos() + u * a.sin()], -1)


# position of token t inside a V page row
_V_POS = [(t & 3) | ((t >> 1) & 4) | ((t << 1) & 8) for t in range(PAGE)]


def _gather64(s, i, n):
    """K and V [n, Hkv, dh] of sequence i, read from the paged pools."""
    sh = s["sh"]
    pages = torch.tensor(s["bt_host"][i, :-(-n // PAGE)].astype(np.int64), device=DEV)
    k = s["k"].view(sh.n_kv_heads, s["blocks"], sh.head_dim // 8, PAGE, 8)[:, pages]
    k = k.permute(1, 3, 0, 2, 4).reshape(-1, sh.n_kv_heads, sh.head_dim)
    v = s["v"].view(sh.n_kv_heads, s["blocks"], sh.head_dim, PAGE)[:, pages][..., _V_POS]
    v = v.permute(1, 3, 0, 2).reshape(-1, sh.n_kv_heads, sh.head_dim)
    return k[:n].double(), v[:n].double()


def _attend64(q, k, v, pos0):
    """Causal attention of q [n, Hq, dh] at positions pos0.. over k, v [c, Hkv, dh], a kv-head at a time."""
    n, hq, dh = q.shape
    grp = hq // k.shape[1]
    hidden = torch.arange(len(k), device=DEV)[None, :] > torch.arange(pos0, pos0 + n, device=DEV)[:, None]
    out = torch.empty_like(q)
    for h in range(hq):
        sc = (q[:, h] @ k[:, h // grp].T) / math.sqrt(dh)
        out[:, h] = torch.softmax(sc.masked_fill_(hidden, -math.inf), -1) @ v[:, h // grp]
    return out


def _last_logits64(m, ids):
    """Logits after the last of the token ids, by the plain decoder."""
    sh = m.shape
    hq, hkv, dh = sh.n_q_heads, sh.n_kv_heads, sh.head_dim
    pos = torch.arange(len(ids), device=DEV)
    x = m.embed[torch.tensor(np.asarray(ids, np.int64), device=DEV)].double()
    for l, L in enumerate(m.layers):
        w = {k: m.plain[(l, k)] for k in ("wqkv", "wo", "w_gate", "w_up", "w_down")}
        qkv = _norm64(x, L["attn_norm"]) @ w["wqkv"].double().T
        q, k, v = (t.reshape(len(ids), -1, dh) for t in qkv.split([hq * dh, hkv * dh, hkv * dh], 1))
        x = x + _attend64(_rope64(q, pos), _rope64(k, pos), v, 0).reshape(len(ids), -1) @ w["wo"].double().T
        h = _norm64(x, L["ffn_norm"])
        x = x + (torch.nn.functional.silu(h @ w["w_gate"].double().T) * (h @ w["w_up"].double().T)) @ \
            w["w_down"].double().T
    return (_norm64(x[-1:], m.norm) @ m.plain["lm_head"].double().T)[0]


def exact(case, seed):
    sh = _shape(case)
    d, f, hq, hkv, dh = sh.d_model, sh.ffn_dim, sh.n_q_heads, sh.n_kv_heads, sh.head_dim
    kind = case["kind"]
    if kind == "serve":
        model, first, forks, _, _ = _serve_state(case, seed, keep=True)
        # the last generated token is not fed back; a fork goes on from all of its parent's tokens
        seqs = [np.concatenate([p, t[:-1]]) for p, t in first]
        stem = np.concatenate(first[0])
        seqs += [np.concatenate([stem, t[:-1]]) for t in forks]
        return {"logits": [_last_logits64(model, q) for q in seqs]}
    s = prepare(case, seed)
    if kind == "qkv":
        y = _matmul64(_norm64(s["x"].double(), s["gain"]), s["w"], sh.qkv_dim, d)
        q, k, v = (t.reshape(s["rows"], -1, dh) for t in y.split([hq * dh, hkv * dh, hkv * dh], 1))
        q, k = _rope64(q, s["pos"]), _rope64(k, s["pos"])
        page, off = s["slot"].long() // PAGE, s["slot"].long() % PAGE
        kp = torch.zeros(s["pages"], PAGE, hkv, dh, dtype=torch.float64, device=DEV)
        vp = torch.zeros_like(kp)
        kp[page, off], vp[page, torch.tensor(_V_POS, device=DEV)[off]] = k, v
        kp = kp.view(-1, PAGE, hkv, dh // 8, 8).permute(2, 0, 3, 1, 4)
        return {"q": q.reshape(s["rows"], -1), "k": kp.reshape(-1), "v": vp.permute(2, 0, 3, 1).reshape(-1)}
    if kind in ("decode", "forks"):
        return {"out": torch.cat([_attend64(s["q"][i:i + 1].double(), *_gather64(s, i, int(c)), int(c) - 1)
                                  for i, c in enumerate(s["ctx"])])}
    if kind == "prefill":
        out = []
        for i, (p, n) in enumerate(_chunks(case)):
            r = int(s["row0"][i])
            out.append(_attend64(s["q"][r:r + n].double(), *_gather64(s, i, p + n), p))
        return {"out": torch.cat(out)}
    x = s["x"].double()
    h = _norm64(x, s["gain"])
    if kind == "mlp":
        act = torch.nn.functional.silu(_matmul64(h, s["gate"], f, d)) * _matmul64(h, s["up"], f, d)
        return {"x": x + _matmul64(act, s["down"], d, f)}
    logits = _matmul64(h, s["w"], sh.vocab, d)
    return {"logits": logits, "ids": None}
