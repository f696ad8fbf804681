"""Performance cases of the decode framework: whole requests (prefill, then
draft/verify steps), prefill alone and single GEMMs, each through the public
entry points (Session and the chimera_gemm_static call) at the model widths,
trees and prompt lengths of this repository's workloads.

A case of kind "request" is what a serving program does for a batch of
prompts: chimera_prefill, then a number of speculative (or plain greedy)
steps.  A request starts with a prefill, so the same state can serve one
request after another.  Models are the published widths at a stated number of
layers with random-init weights; acceptance is forced with probability
``accept`` through the documented forcing tables, as the benchmark does it.

A case of kind "gemm" is one product through chimera_gemm_static, the
allocation-free entry point for serving loops.
"""
import dataclasses
import math

import numpy as np
import torch

import synth
from paper_2402_15758_amd import Session
from paper_2402_15758_amd import binding as B

MODELS = {
    "tiny": synth.TINY,              # fp32, d 256
    "small": synth.small_config(),   # bf16, d 256, heads of 128
    "7b": synth.LLAMA7B,
    "13b": synth.LLAMA13B,
}
STD = 0.02


def _request(name, model, layers, batch, lo, hi, steps, tree, **opt):
    c = {"name": name, "kind": "request", "model": model, "layers": layers, "batch": batch, "lo": lo, "hi": hi,
         "steps": steps, "tree": tree, "accept": 0.0, "branch": False, "typical": False, "cache": 0,
         "pipelined": True, "stream": True}
    c.update(opt)
    return c


def listed():
    return [
        # one small product from a serving loop: launches and latency
        {"name": "gemm_f32_m5", "kind": "gemm", "dtype": "f32", "M": 5, "N": 1024, "K": 1024},
        # a batch of 256 rows against a bf16 matrix, near the call's largest
        {"name": "gemm_bf16_m256", "kind": "gemm", "dtype": "bf16", "M": 256, "N": 4096, "K": 1280},
        # the smallest model in use (smoke and fp32 checks): one call per step
        _request("tiny_f32_t8", "tiny", 2, 1, 32, 32, 24, "T8", pipelined=False),
        # a small bf16 model sampling with typical acceptance, ragged batch
        _request("small_b3_typical", "small", 2, 3, 61, 600, 16, "T32", typical=True),
        # a short chat turn: time to the first speculative tokens
        _request("7b_short_prompt", "7b", 8, 1, 17, 17, 1, "T64", pipelined=False),
        # the headline workload at full depth: 512-token prompt, T64, p = 0.7
        _request("7b_p512_t64", "7b", 32, 1, 512, 512, 60, "T64", accept=0.7, stream=False),
        # a long document: 4096-token prompt and an answer over it
        _request("7b_p4096_t64", "7b", 8, 1, 4096, 4096, 32, "T64", accept=0.7),
        # prompt ingestion only, ragged batch
        _request("7b_prefill_b4", "7b", 4, 4, 300, 1911, 0, "T64"),
        # throughput serving: eight ragged sequences with the 32-node tree
        _request("7b_b8_t32", "7b", 8, 8, 256, 2048, 48, "T32", accept=0.65),
        # the same batch size on chat-length prompts with the 8-node tree
        _request("7b_b8_t8", "7b", 8, 8, 40, 333, 48, "T8", accept=0.65),
        # the wider model, branch-conditioned drafting and the trigram cache
        _request("13b_p1024_branch", "13b", 6, 1, 1024, 1024, 32, "T64", accept=0.8, branch=True, cache=16384),
        # plain greedy decoding, the baseline every speedup is quoted against
        _request("7b_greedy_p130", "7b", 16, 1, 130, 130, 48, "none", pipelined=False),
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    if rng.random() < 0.2:
        dtype = rng.choice(["f32", "bf16"])
        while True:
            M, N, K = _logint(rng, 1, 256), 64 * _logint(rng, 4, 128), 32 * _logint(rng, 8, 128)
            es = 2 if dtype == "bf16" else 4
            # operands and at most 8 split-K partials inside the 32 MiB scratch
            if N * K * es + 256 * K * es + 8 * M * N * 4 < 30 << 20:
                return {"kind": "gemm", "dtype": dtype, "M": M, "N": N, "K": K}
    model = rng.choice(["tiny", "small", "7b", "7b", "7b", "13b"])
    layers = rng.randint(1, 3) if model in ("tiny", "small") else rng.randint(2, 8)
    batch = rng.choice([1, 1, 2, 3, 5, 8])
    hi = _logint(rng, 4, 1000 if model in ("tiny", "small") else (3000 if batch == 1 else 1500))
    lo = max(1, int(hi * rng.uniform(0.2, 1.0)))
    tree = rng.choice(["none", "T8", "T32", "T64"]) if model != "tiny" else rng.choice(["none", "T8"])
    steps = rng.choice([0, 1, 5, 16, 33])
    spec = tree != "none"
    c = _request("", model, layers, batch, lo, hi, steps, tree, accept=round(rng.uniform(0.3, 0.9), 2) if spec else 0.0,
                 branch=spec and rng.random() < 0.3, typical=rng.random() < 0.2,
                 cache=rng.choice([0, 0, 4096]) if spec else 0, pipelined=rng.random() < 0.6,
                 stream=rng.random() < 0.7)
    del c["name"]
    if c["typical"]:
        c["accept"] = 0.0  # forcing follows the greedy stream
    return c


# ---------------------------------------------------------------------------
def _cfg(c):
    return dataclasses.replace(MODELS[c["model"]], n_layers=c["layers"])


def _tree(c):
    return () if c["tree"] == "none" else synth.TREES[c["tree"]]


def _lens(c):
    """Prompt lengths of the batch: lo .. hi, spread unevenly."""
    n = c["batch"]
    if n == 1:
        return [c["hi"]]
    return [int(c["lo"] + (c["hi"] - c["lo"]) * ((5 * i + 3) % n) / (n - 1)) for i in range(n)]


def _prompts(c, seed):
    rng = np.random.default_rng(seed)
    return [rng.integers(0, _cfg(c).vocab, size=n).astype(np.int32) for n in _lens(c)]


def _weights(c, seed):
    """Random-init weights, made on the GPU from one generator."""
    cfg = _cfg(c)
    dt = torch.float32 if cfg.dtype == "f32" else torch.bfloat16
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    out = {}
    for name, shape, group in synth.tensor_specs(cfg):
        if group == "gain":
            out[name] = torch.ones(shape, dtype=torch.float32, device="cuda")
        else:
            out[name] = torch.empty(shape, dtype=dt, device="cuda").normal_(0.0, STD, generator=g)
    return out


def _prepare_request(c, seed):
    cfg, tree, prompts = _cfg(c), _tree(c), _prompts(c, seed)
    depth = max((len(r) for r in tree), default=0)
    max_len = max(_lens(c)) + (c["steps"] + 1) * (depth + 1) + len(tree) + 64
    stream = torch.cuda.Stream() if c["stream"] else torch.cuda.current_stream()
    with torch.cuda.stream(stream):
        sess = Session(cfg, _weights(c, seed), tree, max_batch=c["batch"], max_len=max_len)
        if c["branch"]:
            sess.set_drafting(True)
        if c["typical"]:
            sess.set_decoding(True, temperature=1.0, eps=0.09, delta=0.3, seed=seed & 0xFFFFFFFF)
        if c["cache"]:
            sess.trigram_cache(c["cache"])
        # paged K/V of the target: [layer][page][K|V][head][slot][head_dim] at
        # the start of the KV arena, zeroed so that unwritten slots compare
        shape = (cfg.n_layers, sess.n_pages, 2, cfg.n_heads, sess.page_size, cfg.head_dim)
        dt = torch.float32 if cfg.dtype == "f32" else torch.bfloat16
        nbytes = math.prod(shape) * (4 if dt is torch.float32 else 2)
        pool = sess.kv_arena[:nbytes].view(dt).view(shape)
        pool.zero_()
        if c["accept"] > 0:
            # the greedy stream of the same prompts is the forcing reference
            want = (c["steps"] + 1) * (depth + 1)
            greedy = Session(cfg, None, (), max_batch=c["batch"], max_len=max_len, share_model=sess)
            streams = [[int(t)] for t in greedy.prefill(prompts)]
            while len(streams[0]) < want:
                toks, _, _ = greedy.steps(min(64, want - len(streams[0])))
                for b, s in enumerate(streams):
                    s += [int(t) for t in toks[:, b, 0]]
            greedy.close()
            rng = np.random.default_rng(seed + 1)
            ref = np.full((c["batch"], max_len + 8), -1, dtype=np.int32)
            for b, s in enumerate(streams):
                n0 = len(prompts[b])
                m = min(len(s), max_len + 8 - n0)
                ref[b, n0:n0 + m] = s[:m]
            ok = (rng.random(ref.shape) < c["accept"]).astype(np.uint8)
            sess.set_forcing(torch.from_numpy(ref).cuda(), torch.from_numpy(ok).cuda())
    torch.cuda.synchronize()
    ps = sess.page_size
    per = math.ceil((max_len + 64) / ps)
    # whole pages of each prompt; without steps also its last, partial one
    kv = [pool[:, b * per:b * per + (n // ps if c["steps"] else -(-n // ps))] for b, n in enumerate(_lens(c))]
    return {"case": c, "sess": sess, "prompts": prompts, "stream": stream, "kv": kv}


def _run_request(s):
    c, sess = s["case"], s["sess"]
    with torch.cuda.stream(s["stream"]):
        out = {"first": sess.prefill(s["prompts"]), "kv": s["kv"]}
        if c["steps"]:
            if c["pipelined"]:
                out["tokens"], out["n"], out["path"] = sess.steps(c["steps"])
            else:
                out["tokens"], out["n"], out["path"] = map(np.stack, zip(*(sess.step() for _ in range(c["steps"]))))
            # the last step's logits of every tree node
            out["logits"] = sess.debug(B.DBG_VERIFY_LOGITS)
    return out


def prepare(case, seed):
    if case["kind"] == "request":
        return _prepare_request(case, seed)
    dt = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    x = torch.empty((case["M"], case["K"]), dtype=dt, device="cuda").normal_(generator=g)
    w = torch.empty((case["K"], case["N"]), dtype=dt, device="cuda").normal_(0.0, STD, generator=g)
    y = torch.zeros((case["M"], case["N"]), dtype=torch.float32, device="cuda")
    return {"case": case, "x": x, "w": w, "y": y}


def run(state):
    c = state["case"]
    if c["kind"] == "request":
        return _run_request(state)
    x, w, y = state["x"], state["w"], state["y"]
    B.chimera_gemm_static(B.CHIMERA_F32 if c["dtype"] == "f32" else B.CHIMERA_BF16, x.data_ptr(), w.data_ptr(),
                          c["M"], c["N"], c["K"], y.data_ptr(), torch.cuda.current_stream().cuda_stream)
    return y


# ---------------------------------------------------------------------------
def work(case):
    if case["kind"] == "gemm":
        M, N, K = case["M"], case["N"], case["K"]
        es = 4 if case["dtype"] == "f32" else 2
        return {"bytes": (M * K + K * N) * es + M * N * 4, "flops": 2 * M * N * K}
    cfg, tree = _cfg(case), _tree(case)
    es = 4 if cfg.dtype == "f32" else 2
    d, F, V, hd, L = cfg.d_model, cfg.d_ffn, cfg.vocab, cfg.n_heads * cfg.head_dim, cfg.n_layers
    layer = 4 * d * hd + 3 * d * F
    lens, steps = _lens(case), case["steps"]
    depth = max((len(r) for r in tree), default=0)
    nodes, batch, tok = len(tree) + 1, case["batch"], sum(lens)
    # prefill: the target stack on every prompt token, the LM head on the last
    # one, the draft's trigram encoder and its K/V projection of both streams
    fl = 2.0 * tok * (L * layer + 4 * d * d + 4 * d * hd) + 2.0 * batch * d * V
    fl += sum(2.0 * L * hd * n * n for n in lens)
    by = float(es) * (L * layer + d * V + 4 * d * d + 2 * d * hd + tok * (d + 2 * L * hd + 4 * hd))
    if depth == 0:  # no draft is ever used
        fl -= 2.0 * tok * (4 * d * d + 4 * d * hd)
        by -= float(es) * (4 * d * d + 2 * d * hd + tok * 4 * hd)
    # a step: every draft level streams the trigram encoder, the encoder block
    # and its head; the verify pass streams the target and reads the context
    level = 4 * d * d + layer + 2 * d * d + d * V
    by += steps * float(es) * (depth * level + L * layer + d * V + 2 * hd * (L + 2 * depth) * tok)
    fl += steps * 2.0 * batch * (depth * level + nodes * (L * layer + d * V))
    fl += steps * 4.0 * hd * (L * nodes + 2 * depth) * tok
    return {"bytes": by, "flops": fl}


def tolerance(case):
    if case["kind"] == "gemm":
        # 32-bit sums of exact products (bf16) or of fp32 ones
        return {"rel": 1e-5}
    if _cfg(case).dtype == "f32":
        return {"rel": 2e-5, "differ": 0.0}
    # bf16 storage points flip between two summation orders and the flips
    # travel through the layers
    return {"rel": 0.015 if case["layers"] <= 8 else 0.03, "differ": 0.01}


# ---------------------------------------------------------------------------
def _rope(x, pos, base, hd):
    """Rotate-half rotary embedding of x [n, H, hd] at positions pos."""
    i = torch.arange(hd // 2, dtype=torch.float64, device=x.device)
    a = pos.double()[:, None] * base ** (-2.0 * i / hd)
    c, s = a.cos()[:, None], a.sin()[:, None]
    x1, x2 = x[..., :hd // 2], x[..., hd // 2:]
    return torch.cat([x1 * c - x2 * s, x2 * c + x1 * s], -1)


def _exact_kv(cfg, w, prompt):
    """K and V [layer][2][n][H][hd] of a prompt, in 64 bits throughout."""
    n, H, hd = len(prompt), cfg.n_heads, cfg.head_dim
    t = torch.from_numpy(prompt.astype(np.int64)).cuda()
    pos = torch.arange(n, device="cuda")
    x = w["tok_embed"][t].double()

    def norm(v):
        return v * torch.rsqrt(v.square().mean(-1, keepdim=True) + cfg.rms_eps)

    out = []
    for l in range(cfg.n_layers):
        p = f"layers.{l}."
        h = norm(x)
        q, k, v = ((h @ w[p + m].double()).view(n, H, hd) for m in ("wq", "wk", "wv"))
        q, k = _rope(q, pos, cfg.rope_base, hd), _rope(k, pos, cfg.rope_base, hd)
        out.append(torch.stack([k, v]))
        if l + 1 == cfg.n_layers:
            break
        o = torch.empty_like(v)
        for j in range(H):
            kj = k[:, j].t().contiguous()
            for r0 in range(0, n, 1024):
                r = slice(r0, min(n, r0 + 1024))
                s = (q[r, j].contiguous() @ kj) / math.sqrt(hd)
                s = s.masked_fill(pos[None, :] > pos[r, None], -math.inf)
                o[r, j] = torch.softmax(s, -1) @ v[:, j].contiguous()
        x = x + o.reshape(n, H * hd) @ w[p + "wo"].double()
        h = norm(x)
        g = h @ w[p + "w_gate"].double()
        x = x + (g / (1 + torch.exp(-g)) * (h @ w[p + "w_up"].double())) @ w[p + "w_down"].double()
    return torch.stack(out)


def exact(case, seed):
    if case["kind"] == "gemm":
        s = prepare(case, seed)
        return s["x"].double() @ s["w"].double()
    cfg, w = _cfg(case), _weights(case, seed)
    ps, kv = 16, []
    for p in _prompts(case, seed):
        k = _exact_kv(cfg, w, p)  # [L][2][n][H][hd]
        n = len(p)
        pages = n // ps if case["steps"] else -(-n // ps)
        full = torch.zeros((cfg.n_layers, 2, pages * ps, cfg.n_heads, cfg.head_dim), dtype=torch.float64, device="cuda")
        m = min(n, pages * ps)
        full[:, :, :m] = k[:, :, :m]
        full = full.view(cfg.n_layers, 2, pages, ps, cfg.n_heads, cfg.head_dim)
        kv.append(full.permute(0, 2, 1, 4, 3, 5).contiguous())
    out = {"first": None, "kv": kv}
    if case["steps"]:
        out.update(tokens=None, n=None, path=None, logits=None)
    return out
