"""The calls that a program built on this library makes, as cases to be timed and compared.

A case is one call of a public entry point on inputs that are already on the GPU: a verify step (duo_verify, both
selection rules), one round of the deferred form (duo_verify_deferred), a prompt chunk (duo_prefill_chunk), or the
speculative sampler alone (duo_spec_sample, duo_spec_sample_noalloc, duo_deferred_sample).  `model` names one of the
repository's shapes, `layers` how many decoder layers of it are resident: a step is the same few kernels per layer, so
a stack of a few layers between embedding and LM head shows the layer, and one case runs the 7B shape whole.

Weights, prefix cache and drafts are drawn from the seed: weights N(0, 0.02), gains 1 + N(0, 0.02), cached keys and
values N(0, 1.28^2), draft distributions softmax(N(0, 1)) with tokens drawn from them, which a random-weight target
(logits ~ N(0, 1.28^2)) accepts about half of the time.  The matrices of a large stack repeat from a few that are drawn;
every layer's copy on the GPU is its own.
"""
import dataclasses
import math

import numpy as np
import torch

from paper_2503_00784_amd import binding as B
from paper_2503_00784_amd import inputs

DEVICE = "cuda:0"
SHAPES = {"tiny": inputs.TINY, "mid": inputs.MID, "7b": inputs.LLAMA2_7B, "8b": inputs.LLAMA3_8B, "13b": inputs.WIDE13}
DISTINCT_LAYERS = 2
KV_STD = 1.28

STEP = {"kind": "step", "dtype": "bf16", "root": True, "mode": "longest", "temperature": 1.0, "top_p": 0.0}
PREFILL = {"kind": "prefill", "dtype": "bf16"}
DEFERRED = {"kind": "deferred", "dtype": "bf16", "root": True, "temperature": 1.0, "top_p": 0.0}
SAMPLE = {"kind": "sample", "entry": "noalloc", "root": True, "mode": "longest", "temperature": 1.0, "top_p": 0.0}


def listed():
    return [
        # the smallest whole step: a 68M-class model, where launches and latency are what counts
        {"name": "tiny_step", **STEP, "model": "tiny", "layers": 2, "P": 128, "n": 1, "k": 8, "root": False},
        # the whole 7B step right after a prompt: one sequence of eight tokens, every weight streamed once
        {"name": "7b_whole_step", **STEP, "model": "7b", "layers": 32, "P": 512, "n": 1, "k": 8, "root": False},
        # the chained step of a single short draft with a nucleus-restricted target (5 rows)
        {"name": "7b_step_top_p", **STEP, "model": "7b", "layers": 8, "P": 901, "n": 1, "k": 4, "temperature": 0.7, "top_p": 0.9},
        # a chained step of four sequences: the previously emitted token makes it 33 rows
        {"name": "7b_step_4x8", **STEP, "model": "7b", "layers": 8, "P": 2048, "n": 4, "k": 8},
        # the benchmark's largest 7B step: 64 rows on a 4096-token prefix
        {"name": "7b_step_8x8", **STEP, "model": "7b", "layers": 8, "P": 4096, "n": 8, "k": 8, "root": False},
        # grouped queries, a 128k vocabulary, a long prefix, the paper's own (distribution-preserving) selection rule, 65 rows
        {"name": "8b_step_4x16_paper", **STEP, "model": "8b", "layers": 8, "P": 8192, "n": 4, "k": 16, "mode": "paper"},
        # one round of the paper's pipelined loop in its own precision: 15 unverified tokens + root, four new sequences
        {"name": "7b_deferred_fp16", **DEFERRED, "model": "7b", "layers": 8, "P": 1339, "k": 15, "s": 4, "dtype": "fp16"},
        # a full prompt chunk (time to first token), the second of a prompt
        {"name": "7b_prefill_1024", **PREFILL, "model": "7b", "layers": 8, "P": 1024, "m": 1024},
        # a short ragged prompt in fp16, grouped queries, from an empty cache
        {"name": "8b_prefill_333_fp16", **PREFILL, "model": "8b", "layers": 8, "P": 0, "m": 333, "dtype": "fp16"},
        # the sampler on a program's own logits, results left on the device
        {"name": "sample_32k", **SAMPLE, "vocab": 32000, "n": 1, "k": 8},
        {"name": "sample_128k_paper", **SAMPLE, "vocab": 128256, "n": 4, "k": 16, "mode": "paper", "root": False},
        # nucleus sampling over a large vocabulary (the call that returns its results to the host)
        {"name": "sample_128k_top_p", **SAMPLE, "vocab": 128256, "n": 4, "k": 8, "entry": "workspace", "temperature": 0.8, "top_p": 0.95},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choices(["step", "prefill", "deferred", "sample"], [5, 2, 1, 2])[0]
    temperature = rng.choice([1.0, 1.0, 0.8, 0.6])
    top_p = rng.choice([0.0, 0.0, 0.0, 0.9, 0.95])
    root = rng.random() < 0.6
    mode = rng.choice(["longest", "paper"])
    n = rng.choice([1, 1, 2, 3, 4, 6, 8])
    k = rng.randint(1, min(24, 79 // n))
    if kind == "sample":
        vocab = rng.choice([32000, 128256, 4099, _log_int(rng, 1000, 131072)])
        entry = rng.choice(["workspace"] if top_p else ["noalloc", "noalloc", "workspace"])
        return {**SAMPLE, "vocab": vocab, "n": n, "k": k, "root": root, "mode": mode, "temperature": temperature, "top_p": top_p,
                "entry": entry}
    model = rng.choices(["tiny", "mid", "7b", "8b", "13b"], [2, 1, 4, 4, 1])[0]
    layers = min(SHAPES[model].n_layers, 4)
    dtype = rng.choice(["bf16", "bf16", "fp16"])
    P = _log_int(rng, 16, 8192 if model in ("7b", "8b") else 1024)
    base = {"model": model, "layers": layers, "dtype": dtype, "P": P}
    if kind == "prefill":
        return {**PREFILL, **base, "P": rng.choice([0, P]), "m": _log_int(rng, 5, 1024)}
    if kind == "deferred":
        return {**DEFERRED, **base, "k": rng.randint(0 if root else 1, 32), "s": rng.randint(0, 6), "root": root, "temperature": temperature,
                "top_p": top_p}
    return {**STEP, **base, "n": n, "k": k, "root": root, "mode": mode, "temperature": temperature, "top_p": top_p}


# --------------------------------------------------------------------------- inputs
def _gen(seed, *stream):
    g = torch.Generator(device=DEVICE)
    key = int(seed) & 0x7FFFFFFF
    for s in stream:
        key = (key * 1000003 + int(s) + 12345) & 0x7FFFFFFFFFFF
    g.manual_seed(key)
    return g


def _shape(case):
    return dataclasses.replace(SHAPES[case["model"]], n_layers=case["layers"])


def _type(case):
    return torch.float16 if case["dtype"] == "fp16" else torch.bfloat16


def _normal(dims, std, mean, dtype, g):
    return (torch.randn(dims, generator=g, device=DEVICE) * std + mean).to(dtype)


def _weights(case, seed):
    """Parameters as 16-bit tensors on the GPU, row-major [out][in]; per-layer entries are lists of the distinct layers."""
    s, t = _shape(case), _type(case)
    d, f = s.d_model, s.d_ff
    dims = {"wq": (s.q_dim, d), "wk": (s.kv_dim, d), "wv": (s.kv_dim, d), "wo": (d, s.q_dim), "w_gate": (f, d), "w_up": (f, d),
            "w_down": (d, f), "g_attn": (d,), "g_ffn": (d,)}
    w = {name: [_normal(dim, 0.02, 1.0 if name.startswith("g_") else 0.0, t, _gen(seed, 1, l, i)) for l in range(min(DISTINCT_LAYERS, s.n_layers))]
         for i, (name, dim) in enumerate(dims.items())}
    w["embed"] = _normal((s.vocab, d), 0.02, 0.0, t, _gen(seed, 2))
    w["lm_head"] = _normal((s.vocab, d), 0.02, 0.0, t, _gen(seed, 3))
    w["g_final"] = _normal((d,), 0.02, 1.0, t, _gen(seed, 4))
    return w


def _cache_rows(case, seed, max_seq):
    """Prefix keys and values [2][layers][kv heads][max_seq][head_dim] in the 16-bit type, zero from slot P on."""
    s, P = _shape(case), case["P"]
    kv = torch.zeros((2, s.n_layers, s.n_kv_heads, max_seq, s.head_dim), dtype=_type(case), device=DEVICE)
    for i in range(2):
        for l in range(s.n_layers):
            kv[i, l, :, :P] = _normal((s.n_kv_heads, P, s.head_dim), KV_STD, 0.0, _type(case), _gen(seed, 5, i, l))
    return kv


def _rows(case):
    if case["kind"] == "prefill":
        return case["m"]
    return int(case["root"]) + case.get("n", 1) * case["k"]


def _max_seq(case):
    return (case["P"] + _rows(case) + 31) // 32 * 32


def _drafts(vocab, lead, seed, stream, like=None):
    """Draft distributions fp32 [*lead][vocab] and a token drawn from each, int32 [*lead]."""
    rows = int(np.prod(lead))
    if rows == 0:
        return torch.zeros((*lead, vocab), device=DEVICE), torch.zeros(lead, dtype=torch.int32, device=DEVICE)
    g = _gen(seed, 6, stream)
    z = torch.randn((rows, vocab), generator=g, device=DEVICE)
    if like is not None:  # a draft model that agrees with the target's logits in part
        z = 0.8 * like.reshape(rows, vocab) + 0.6 * z
    q = torch.softmax(z.double(), -1).float()
    u = torch.rand((rows, 1), generator=g, device=DEVICE, dtype=torch.float64)
    c = torch.cumsum(q.double(), -1)
    tok = torch.searchsorted(c, u * c[:, -1:], right=True).clamp_(max=vocab - 1)
    return q.reshape(*lead, vocab).contiguous(), tok.to(torch.int32).reshape(lead).contiguous()


def _uniforms(lead, seed, stream):
    return torch.rand(lead, generator=_gen(seed, 7, stream), device=DEVICE)


def _host(t):
    """A 16-bit tensor as the host array that the binding takes: numpy float16, or bf16 bit patterns."""
    return t.cpu().numpy() if t.dtype == torch.float16 else t.view(torch.int16).cpu().numpy().view(np.uint16)


def _root_token(case, seed):
    return (int(seed) * 7919 + 11) % SHAPES[case["model"]].vocab if case.get("root") else -1


def _root_logits(case, seed):
    return torch.randn(SHAPES[case["model"]].vocab, generator=_gen(seed, 8), device=DEVICE) * KV_STD


def _prompt(case, seed):
    return torch.randint(0, SHAPES[case["model"]].vocab, (case["m"],), generator=_gen(seed, 9), device=DEVICE).cpu().tolist()


def _sample_inputs(case, seed):
    V, n, k, R = case["vocab"], case["n"], case["k"], int(case["root"])
    rows = torch.randn((R + n * k, V), generator=_gen(seed, 10), device=DEVICE) * 2.0
    root = torch.randn(V, generator=_gen(seed, 11), device=DEVICE) * 2.0
    first = rows[0] if R else root
    judge = torch.stack([first if j == 0 else rows[R + i * k + j - 1] for i in range(n) for j in range(k)])
    q, tok = _drafts(V, (n, k), seed, 0, like=judge)
    return rows, root, q, tok, _uniforms((n, k + 1), seed, 0)


def prepare(case, seed):
    if case["kind"] == "sample":
        rows, root, q, tok, u = _sample_inputs(case, seed)
        return {"case": case, "args": (rows, root, tok, q, u), "sampler": B.NoAllocSampler() if case["entry"] == "noalloc" else None}
    s, max_seq = _shape(case), _max_seq(case)
    w = _weights(case, seed)
    host = {name: [_host(t) for t in v] if isinstance(v, list) else _host(v) for name, v in w.items()}
    del w
    for name, v in host.items():
        if isinstance(v, list):
            host[name] = [v[l % len(v)] for l in range(s.n_layers)]
    eng = B.VerifyEngine(s, host, max_seq, max_prefill_rows=max(_rows(case), B.DUO_MAX_ROWS) if case["kind"] == "prefill" else B.DUO_MAX_ROWS)
    kv = _cache_rows(case, seed, max_seq)
    root_logits = _root_logits(case, seed)
    eng.load_cache(_host(kv[0]), _host(kv[1]), case["P"], root_logits.cpu().numpy())
    state = {"case": case, "engine": eng}
    if case["kind"] == "prefill":
        state["tokens"] = _prompt(case, seed)
        return state
    state["root"] = _root_token(case, seed)
    state["logits"] = torch.zeros((_rows(case), s.vocab), dtype=torch.float32, device=DEVICE)
    if case["kind"] == "deferred":
        state["suffix"] = _drafts(s.vocab, (case["k"],), seed, 0)
        state["first"] = _drafts(s.vocab, (case["s"],), seed, 1)
        state["u"], state["u_first"] = _uniforms((case["k"] + 1,), seed, 0), _uniforms((case["s"],), seed, 1)
    else:
        state["draft"] = _drafts(s.vocab, (case["n"], case["k"]), seed, 0)
        state["u"] = _uniforms((case["n"], case["k"] + 1), seed, 0)
    return state


# --------------------------------------------------------------------------- one pass
def _written_blocks(eng, P, dtype):
    """The 32-slot blocks of the cache from the one that holds slot P on, as they lie in memory."""
    L, H, _ = eng.k.shape
    D = eng.shape.head_dim
    return [c.view(dtype).view(L, H, eng.max_seq // 32, 32 * D)[:, :, P // 32:] for c in (eng.k, eng.vT)]


def run(state):
    case = state["case"]
    if case["kind"] == "sample":
        rows, root, tok, q, u = state["args"]
        opts = dict(temperature=case["temperature"], select_mode=int(case["mode"] == "paper"), has_root=case["root"], prefix_len=100)
        if case["entry"] == "workspace":
            return B.spec_sample(rows, root, tok, q, u, top_p=case["top_p"], **opts)
        sampler = state["sampler"]
        code = sampler.run(rows, root, tok, q, u, **opts)
        return [code, sampler.accept_len[:case["n"]], sampler.next_token[:case["n"]], sampler.commit, sampler.status]
    eng = state["engine"]
    eng.set_prefix_len(case["P"])  # the pass before advanced it
    if case["kind"] == "prefill":
        eng.prefill(state["tokens"], chunk=case["m"])
        k, v = _written_blocks(eng, case["P"], _type(case))
        return {"root_logits": eng.root_logits, "k": k, "v": v, "prefix_len": eng.prefix_len, "status": eng.status}
    opts = dict(temperature=case["temperature"], root_token=state["root"], logits_out=state["logits"], top_p=case["top_p"])
    if case["kind"] == "deferred":
        (q, tok), (fq, ftok) = state["suffix"], state["first"]
        new = (ftok, fq, state["u_first"]) if case["s"] else (None, None, None)
        eng.verify_deferred(tok if case["k"] else None, q if case["k"] else None, state["u"], *new, **opts)
        n = 1
    else:
        (q, tok), n = state["draft"], case["n"]
        eng.verify(tok, q, state["u"], select_mode=int(case["mode"] == "paper"), **opts)
    # The emitted token is left to the sampling cases: a draw close to a step of a 32000-entry distribution function
    # moves with the last bits of a logit.  The accepted lengths decide which keys and values are committed.
    k, v = _written_blocks(eng, case["P"], _type(case))
    return {"logits": state["logits"], "k": k, "v": v, "accept_len": eng.accept_len[:n], "prefix_len": eng.prefix_len, "status": eng.status}


# --------------------------------------------------------------------------- what a pass cannot do without
def work(case):
    if case["kind"] == "sample":
        V, n, k = case["vocab"], case["n"], case["k"]
        # every judging row once for its normaliser and the draft row behind one correction token
        rows = 1 + n * k if case["mode"] == "longest" else n + k
        return {"bytes": 4.0 * V * (rows + n), "flops": 0.0}
    s, M, P = _shape(case), _rows(case), case["P"]
    last_only = case["kind"] == "prefill"
    kv_token = s.kv_bytes_per_token()
    nbytes = s.weight_bytes() + P * kv_token + M * kv_token + 4 * s.vocab * (1 if last_only else M)
    body = (s.weight_bytes() // 2 - s.vocab * s.d_model)
    causal = M / 2.0 if last_only else (M if M < 2 else case["k"] / 2.0)
    flops = 2.0 * M * body + 2.0 * (1 if last_only else M) * s.vocab * s.d_model + 4.0 * M * (P + causal) * s.q_dim * s.n_layers
    return {"bytes": float(nbytes), "flops": flops}


def tolerance(case):
    if case["kind"] == "sample":
        return "exact"
    # Seen against 64 bits: logits 9e-6 .. 1.3e-4 (activations carry 16 mantissa bits or more through up to 32 layers),
    # caches 2e-5 .. 6e-4 (16-bit values, of which a few round the other way: an ulp, 0.8 % of a value in bf16).
    return {"rel": 2.5e-3, "max": 0.03}


# --------------------------------------------------------------------------- the same pass in 64 bits
def _rotate(x, pos, theta):
    """Half-split rotary embedding of x [rows][heads][D] at positions pos [rows]."""
    D = x.shape[-1]
    ang = pos.double()[:, None] * theta ** (-2.0 * torch.arange(D // 2, device=x.device, dtype=torch.float64) / D)
    c, s = ang.cos()[:, None], ang.sin()[:, None]
    a, b = x[..., : D // 2], x[..., D // 2:]
    return torch.cat([a * c - b * s, b * c + a * s], -1)


def _to_tiles(rows, kind):
    """[L][H][S][D] -> the cache's tile order (include/duo_verify.h), [L][H][S / 32][32 * D]."""
    L, H, S, D = rows.shape
    if kind == "k":
        x = rows.reshape(L, H, S // 32, 4, 2, 4, D // 32, 4, 8).permute(0, 1, 2, 4, 6, 7, 3, 5, 8)
    else:
        x = rows.reshape(L, H, S // 32, 4, 8, D // 16, 16).permute(0, 1, 2, 5, 3, 6, 4)
    return x.reshape(L, H, S // 32, 32 * D)


def exact(case, seed):
    if case["kind"] == "sample":
        return None
    s, P, M = _shape(case), case["P"], _rows(case)
    max_seq, dev = _max_seq(case), DEVICE
    w = _weights(case, seed)
    kv = _cache_rows(case, seed, max_seq)
    if case["kind"] == "prefill":
        tokens = torch.tensor(_prompt(case, seed), device=dev)
        R, n, k = 0, 1, M
    else:
        R, n, k = int(case["root"]), case.get("n", 1), case["k"]
        lead = (k,) if case["kind"] == "deferred" else (n, k)
        tokens = _drafts(s.vocab, lead, seed, 0)[1].reshape(-1).long()
        if R:
            tokens = torch.cat([torch.tensor([_root_token(case, seed)], device=dev), tokens])
    m = torch.arange(M, device=dev)
    kk = max(k, 1)
    pos = torch.where(m < R, P, P + R + (m - R) % kk)
    seq = torch.where(m < R, -1, (m - R) // kk)
    mine = (seq[:, None] == seq[None, :]) | (seq[None, :] < 0)  # row i may see row j: same sequence, or the root
    visible = torch.cat([torch.ones((M, P), dtype=torch.bool, device=dev), mine & (m[None, :] <= m[:, None])], 1)
    x = w["embed"][tokens].double()
    group = s.n_q_heads // s.n_kv_heads

    def normed(x, g):
        return x / torch.sqrt(x.square().mean(-1, keepdim=True) + s.rms_eps) * g.double()

    for l in range(s.n_layers):
        lw = {name: w[name][l % len(w[name])] for name in ("wq", "wk", "wv", "wo", "w_gate", "w_up", "w_down", "g_attn", "g_ffn")}
        h = normed(x, lw["g_attn"])
        q = _rotate((h @ lw["wq"].double().T).reshape(M, s.n_q_heads, s.head_dim), pos, s.rope_theta)
        kn = _rotate((h @ lw["wk"].double().T).reshape(M, s.n_kv_heads, s.head_dim), pos, s.rope_theta)
        vn = (h @ lw["wv"].double().T).reshape(M, s.n_kv_heads, s.head_dim)
        kv[0, l, :, P:P + M] = kn.transpose(0, 1).to(kv.dtype)  # the cache holds 16-bit values
        kv[1, l, :, P:P + M] = vn.transpose(0, 1).to(kv.dtype)
        o = torch.empty((M, s.n_q_heads, s.head_dim), dtype=torch.float64, device=dev)
        for hk in range(s.n_kv_heads):
            K, V = kv[0, l, hk, :P + M].double(), kv[1, l, hk, :P + M].double()
            for hq in range(hk * group, (hk + 1) * group):
                sc = (q[:, hq] @ K.T.contiguous()) / math.sqrt(s.head_dim)
                o[:, hq] = torch.softmax(sc.masked_fill(~visible, -math.inf), -1) @ V
        x = x + o.reshape(M, -1) @ lw["wo"].double().T
        h = normed(x, lw["g_ffn"])
        gate = h @ lw["w_gate"].double().T
        x = x + (gate * torch.sigmoid(gate) * (h @ lw["w_up"].double().T)) @ lw["w_down"].double().T
    if case["kind"] == "prefill":
        x = x[-1:]
    logits = normed(x, w["g_final"]) @ w["lm_head"].double().T
    if n > 1:  # what is committed is moved next to the prefix: the caches depend on the accepted lengths
        kt = vt = None
    else:
        kt, vt = (_to_tiles(kv[i].double(), kind)[:, :, P // 32:] for i, kind in ((0, "k"), (1, "v")))
    if case["kind"] == "prefill":
        return {"root_logits": logits[0], "k": kt, "v": vt}
    return {"logits": logits, "k": kt, "v": vt}
