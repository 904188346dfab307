"""Measured workloads of the library: whole generations, prompts alone, and the sampling arithmetic alone, each
through the public Python entry points (DelContext, controllers.generate, del_spec_sample_static).

Shapes are those of synthdata/configs.py, some with fewer layers (every layer of a shape does the same work, so a
stack of 4 or 8 of them shows a layer's time); weights are random, built so that a token's successor is predicted with
a clear margin at every layer (a trained model is about that sure of most tokens): the emitted ids, the acceptance
counts and with them the work of a pass are then the same for every correct implementation, and the logits, hidden
rows and statistics returned beside them carry its rounding.

  listed()  the named cases            draw(rng)  another case of the same ranges
  prepare   context with weights loaded, prompt, uniform numbers       run  one call, all outputs
  work      bytes and flops the call cannot do without                 exact  the same call in 64-bit torch
"""
import math

import numpy as np
import torch

from paper_2504_05598_amd import binding, controllers
from paper_2504_05598_amd.binding import DelContext
from synthdata.configs import ModelConfig

PEAK = 16.0      # logit of a token's successor in front of heads whose other logits have standard deviation NOISE
NOISE = 1.28
BRANCH = 0.15    # size of what a layer's branches add to a residual of size 1


# ---- shapes -----------------------------------------------------------------------------------------------------------
# (d_model, query heads, kv heads, head dim, feed-forward width, vocabulary, tied head, dtype, rotary base)
SHAPES = {
    "tiny": (256, 4, 4, 64, 688, 4096, False, "fp32", 1e4),
    "mini_gqa": (512, 8, 2, 64, 1384, 8008, True, "bf16", 5e5),
    "1b": (2048, 32, 8, 64, 8192, 128256, True, "bf16", 5e5),
    "7b": (4096, 32, 32, 128, 11008, 32000, False, "bf16", 1e4),
    "13b": (5120, 40, 40, 128, 13824, 32000, False, "bf16", 1e4),
    "70b": (8192, 64, 8, 128, 28672, 32000, False, "bf16", 1e4),
}


def _model(shape, layers):
    d, nq, nkv, hd, f, v, tied, dtype, theta = shape
    return {"layers": layers, "d": d, "nq": nq, "nkv": nkv, "hd": hd, "f": f, "vocab": v, "tied": tied, "dtype": dtype,
            "theta": theta}


def _generate(name, shape, layers, prompt, tokens, control, E, gamma, d_max):
    c = {"kind": "generate", **_model(shape, layers), "prompt": prompt, "tokens": tokens, "control": control, "E": E,
         "gamma": gamma, "d_max": d_max}
    return {"name": name, **c} if name else c


def _prefill(name, shape, layers, prompt):
    c = {"kind": "prefill", **_model(shape, layers), "prompt": prompt, "d_max": 8}
    return {"name": name, **c} if name else c


def _sampling(name, vocab, gamma, temperature, top_p):
    c = {"kind": "sampling", "vocab": vocab, "gamma": gamma, "temperature": temperature, "top_p": top_p}
    return {"name": name, **c} if name else c


def listed():
    return [
        # the sampling arithmetic on logits in device memory, as a serving loop with its own model calls it per round
        _sampling("sampling_v32000", 32000, 4, 0.6, 0.95),
        # the 32-bit path on the smallest decoder: launches and latency
        _generate("tiny_fp32", SHAPES["tiny"], 4, 32, 64, "ls", 2, 4, 4),
        # a reduced 16-bit decoder with grouped heads, a tied head and ragged sizes everywhere
        _generate("mini_gqa_greedy", SHAPES["mini_gqa"], 6, 45, 48, "ls", 3, 5, 6),
        # a small chat model, whole: tied head over a large vocabulary
        _generate("1b_greedy", SHAPES["1b"], 16, 512, 48, "ls", 5, 4, 8),
        # the headline: the 7B shape, whole, 1024-token prompt, early-exit drafting and verification
        _generate("7b_greedy", SHAPES["7b"], 32, 1024, 64, "ls", 12, 4, 8),
        # auto-regressive decoding, the baseline every user compares with: one row per step
        _generate("7b_vanilla", SHAPES["7b"], 8, 128, 48, "vanilla", 1, 0, 8),
        # speculative sampling, temperature 0.6 and top_p 0.95
        _generate("7b_sampling", SHAPES["7b"], 8, 256, 48, "sample", 3, 4, 8),
        # draft-exiting: the host decides after every draft step; a long context
        _generate("13b_dynamic", SHAPES["13b"], 6, 1999, 48, "dynamic", 3, 8, 10),
        # the largest layers, grouped heads, the longest speculation
        _generate("70b_greedy", SHAPES["70b"], 4, 1024, 52, "ls", 2, 12, 12),
        # a short question alone (time to the first token), ragged
        _prefill("1b_prefill_93", SHAPES["1b"], 16, 93),
        # an ordinary prompt alone
        _prefill("7b_prefill_1024", SHAPES["7b"], 8, 1024),
        # a prompt that fills the shape's context, ragged: attention weighs most
        _prefill("13b_prefill_4001", SHAPES["13b"], 4, 4001),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """Another case: the sampling arithmetic, a 32-bit decoder, or a 16-bit decoder of any width in the listed range
    (generation in each mode, or a prompt alone)."""
    pick = rng.random()
    if pick < 0.12:
        return _sampling(None, _log_int(rng, 256, 32768), rng.randint(0, 8), round(rng.uniform(0.3, 1.3), 3),
                         round(rng.uniform(0.5, 1.0), 3))
    vocab = _log_int(rng, 2000, 40000)
    if pick < 0.24:
        nq, nkv, hd = rng.choice([(4, 4, 64), (6, 2, 32), (8, 8, 64), (6, 6, 64), (9, 3, 48)])
        shape = (nq * hd, nq, nkv, hd, 8 * rng.randint(40, 200), vocab, False, "fp32", 1e4)
        layers, prompt = rng.randint(2, 6), _log_int(rng, 8, 200)
    else:
        group = rng.choice([1, 1, 4, 8])
        hd = 64 if group == 4 else 128
        nkv = _log_int(rng, 3, 40) if group == 1 else rng.randint(2, 9) if group == 4 else rng.randint(1, 8)
        nq = nkv * group
        d = nq * hd
        tied = group == 4
        shape = (d, nq, nkv, hd, 8 * int(d * rng.uniform(2.6, 4.0) / 8), vocab, tied, "bf16", 5e5 if tied else 1e4)
        layers, prompt = rng.randint(2, 6 if d <= 4096 else 4), _log_int(rng, 12, 2000)
        if rng.random() < 0.3:
            return _prefill(None, shape, layers, prompt)
    control = rng.choice(["ls", "ls", "vanilla", "sample", "dynamic"])
    d_max = rng.choice([4, 8, 8, 10, 12, 18])
    gamma = 0 if control == "vanilla" else rng.randint(1, d_max)
    return _generate(None, shape, layers, prompt, rng.randint(24, 64), control, rng.randint(1, layers), gamma, d_max)


# ---- inputs -----------------------------------------------------------------------------------------------------------
def _config(c):
    return ModelConfig("case", c["layers"], c["d"], c["nq"], c["nkv"], c["hd"], c["f"], c["vocab"], c["theta"], c["tied"],
                       c["dtype"], 1.0, c["prompt"], c.get("tokens", 1), c["d_max"], 0)


def _normal(seed, layer, kind, rows, cols, std, dtype):
    gen = torch.Generator(device="cuda")
    gen.manual_seed((seed * 1000003 + (layer + 1) * 64 + kind) & 0x7FFFFFFFFFFFFFFF)
    t = torch.empty(rows, cols, dtype=dtype, device="cuda")
    t.normal_(0.0, std, generator=gen)
    return t


def _successor(c, seed):
    """Untied head: the token each token predicts (a permutation); tied: the token itself."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed * 1000003 + 17)
    return torch.randperm(c["vocab"], generator=gen, device="cuda")


def _tensors(c, seed):
    """(layer, kind, tensor) of every weight, made one at a time from the seed."""
    d, f, q, kv, L = c["d"], c["f"], c["nq"] * c["hd"], c["nkv"] * c["hd"], c["layers"]
    dt = torch.float32 if c["dtype"] == "fp32" else torch.bfloat16
    peak = PEAK if c.get("control") in (None, "ls", "vanilla") else 1.5 * PEAK
    if c["tied"]:
        # logits have standard deviation NOISE, so a row's own logit is NOISE**2 / rms of the last hidden state: the
        # branches bring that rms to where the logit is `peak`
        size = NOISE / math.sqrt(d)
        branch = NOISE * NOISE / peak / math.sqrt(L)
    else:
        size, branch = 1.0, BRANCH
    embed = _normal(seed, -1, 0, c["vocab"], d, size, dt)
    if not c["tied"]:
        head = _normal(seed, -1, 1, c["vocab"], d, NOISE / math.sqrt(d), dt)
        head[_successor(c, seed)] += embed * (peak / d)
        yield -1, "lm_head", head
        del head
    yield -1, "embed", embed
    del embed
    yield -1, "final_norm", 1.0 + _normal(seed, -1, 2, 1, d, 0.05, torch.float32)
    for l in range(L):
        yield l, "attn_norm", 1.0 + _normal(seed, l, 3, 1, d, 0.1, torch.float32)
        yield l, "wq", _normal(seed, l, 4, q, d, 1.2 / math.sqrt(d), dt)
        yield l, "wk", _normal(seed, l, 5, kv, d, 1.2 / math.sqrt(d), dt)
        yield l, "wv", _normal(seed, l, 6, kv, d, 1.2 / math.sqrt(d), dt)
        yield l, "wo", _normal(seed, l, 7, d, q, 2.0 * branch / math.sqrt(q), dt)
        yield l, "ffn_norm", 1.0 + _normal(seed, l, 8, 1, d, 0.1, torch.float32)
        yield l, "wg", _normal(seed, l, 9, f, d, 1.2 / math.sqrt(d), dt)
        yield l, "wu", _normal(seed, l, 10, f, d, 1.2 / math.sqrt(d), dt)
        yield l, "wd", _normal(seed, l, 11, d, f, branch / math.sqrt(f), dt)


def _prompt(c, seed):
    return np.random.RandomState(seed % (1 << 31)).randint(0, c["vocab"], c["prompt"]).astype(np.int32).tolist()


def _uniforms(seed, k, count):
    return np.random.RandomState((seed * 7919 + k) % (1 << 31)).randint(0, 1 << 24, count) / float(1 << 24)


TEMPERATURE, TOP_P = 0.6, 0.95


def _logits(c, seed):
    """Draft and target logits that agree as a model's early exit and its last layer do: a few dozen likely tokens over
    a bed of unlikely ones."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed * 1000003 + 29)
    V, g = c["vocab"], c["gamma"]
    ld = (V + 3) // 4 * 4
    p = torch.zeros(g + 1, ld, device="cuda")
    p[:, :V].normal_(0.0, 1.5, generator=gen)
    at = torch.randint(0, V, (g + 1, 32), generator=gen, device="cuda")
    p.scatter_add_(1, at, 6.0 + 3.0 * torch.randn(g + 1, 32, generator=gen, device="cuda"))
    q = (p[:g] + 0.4 * torch.randn(g, ld, generator=gen, device="cuda")).contiguous()
    u = torch.randint(0, 1 << 24, (2 * g + 1,), generator=gen, device="cuda").double() / float(1 << 24)
    return q, p, u.float(), ld


def prepare(case, seed):
    c = dict(case)
    if c["kind"] == "sampling":
        q, p, u, ld = _logits(c, seed)
        out = torch.zeros(3 + c["gamma"], dtype=torch.int32, device="cuda")
        return {"case": c, "q": q, "p": p, "u": u, "ld": ld, "out": out}
    cfg = _config(c)
    ctx = DelContext(cfg)
    for layer, kind, t in _tensors(c, seed):
        ctx.load_tensor(layer, kind, t)
    return {"case": c, "ctx": ctx, "prompt": _prompt(c, seed), "seed": seed}


# ---- one pass ---------------------------------------------------------------------------------------------------------
def _stats(ctx):
    st = ctx.stats()
    return {"next": np.array([st["next_E"], st["next_gamma"]]), "S_n": st["S_n"], "S_c": np.array(st["S_c"]),
            "S_tcs": np.array(st["S_tcs"]), "tau": np.array(st["tau"])}


def run(state):
    c = state["case"]
    if c["kind"] == "sampling":
        q = state["q"].data_ptr() if c["gamma"] > 0 else 0
        binding.del_spec_sample_static(q, state["p"].data_ptr(), state["ld"], c["vocab"], c["gamma"], c["temperature"],
                                       c["top_p"], state["u"].data_ptr(), state["out"].data_ptr(),
                                       torch.cuda.current_stream().cuda_stream)
        return state["out"]
    ctx, prompt, L = state["ctx"], state["prompt"], c["layers"]
    if c["kind"] == "prefill":
        first, _, _ = ctx.prefill(prompt)
        row = ctx.last_rows() - 1
        return {"tokens": np.array([first]), "logits": ctx.logits(L, row), "hidden": ctx.hidden(L, row), **_stats(ctx)}
    if c["control"] == "dynamic":
        first, _, _ = ctx.prefill(prompt)
        toks, log, E = [first], [], c["E"]
        while len(toks) < c["tokens"]:
            cap = min(c["gamma"], c["tokens"] - len(toks) - 1)
            out, g, _ = ctx.round_dynamic(E, ctx.stats()["tau"][E], cap)
            toks += out
            log.append((E, g, len(out)))
    elif c["control"] == "sample":
        seed = state["seed"]
        toks, log = controllers.generate(ctx, prompt, c["tokens"], "ls", c["E"], c["gamma"],
                                         (TEMPERATURE, TOP_P, lambda k, n: _uniforms(seed, k, n)))
    else:
        toks, log = controllers.generate(ctx, prompt, c["tokens"], c["control"], c["E"], c["gamma"])
    row = log[-1][2] - 1     # the round's last valid row
    return {"tokens": np.array(toks), "rounds": np.array(log), "logits": ctx.logits(L, row), "hidden": ctx.hidden(L, row),
            **_stats(ctx)}


# ---- what a pass cannot do without ------------------------------------------------------------------------------------
def work(case):
    c = case
    if c["kind"] == "sampling":
        n = (2 * c["gamma"] + 1) * c["vocab"]
        return {"bytes": 4.0 * n, "flops": 4.0 * n}
    es = 4 if c["dtype"] == "fp32" else 2
    L, d, q, kv, P = c["layers"], c["d"], c["nq"] * c["hd"], c["nkv"] * c["hd"], c["prompt"]
    layer = 2 * d * q + 2 * d * kv + 3 * d * c["f"]        # weights of a layer
    head = c["vocab"] * d
    row = 2 * kv                                           # cache values of a position and layer
    w = min(32, P)                                         # prompt rows that every layer's shadow head sees
    nbytes = es * (L * (layer + P * row) + head)
    flops = 2.0 * P * L * layer + 2.0 * w * L * head + 2.0 * L * q * P * (P + 1)
    if c["kind"] == "prefill":
        return {"bytes": float(nbytes + es * head), "flops": flops + 2.0 * head}
    E, left, T = c["E"], c["tokens"] - 1, P
    if c["control"] == "vanilla":
        E = 1
    while left > 0:
        g = min(c["gamma"], left - 1)
        m = g + 1
        nbytes += es * ((g * E + L) * layer + m * head)                       # every draft step streams its layers
        nbytes += es * row * (sum(E * (T + i + 1) for i in range(m)) + (L - E) * (T + m) + m * L)
        flops += 2.0 * m * L * layer + 2.0 * (g + L * m) * head + 4.0 * q * m * L * T
        left -= m
        T += m
    return {"bytes": float(nbytes + es * head), "flops": flops + 2.0 * head}


def tolerance(case):
    if case["kind"] == "sampling":
        return "exact"
    # 32-bit: sums of a few thousand terms (1.5e-7 from the 64-bit result).  16-bit: the cache holds keys and values
    # rounded to 16 bits, and a last bit there travels through the layers that follow (up to 1.3e-3 from the 64-bit
    # result, in the tied shapes, whose branches outweigh the embedding).  About four times that.
    return {"rel": 4e-6, "max": 1e-4} if case["dtype"] == "fp32" else {"rel": 5e-3, "max": 0.1}


# ---- the same in 64 bits ----------------------------------------------------------------------------------------------
def _norm(x, gain):
    return x * torch.rsqrt((x * x).mean(-1, keepdim=True) + 1e-5) * gain


class _Model:
    """The decoder in float64; keys and values are rounded to the type the cache stores them in."""

    def __init__(self, c, seed):
        self.c, self.store = c, torch.float32 if c["dtype"] == "fp32" else torch.bfloat16
        self.w = {(l, k): t for l, k, t in _tensors(c, seed)}
        cap = c["prompt"] + c.get("tokens", 0) + 1
        self.K = [torch.zeros(c["nkv"], cap, c["hd"], dtype=torch.float64, device="cuda") for _ in range(c["layers"])]
        self.V = [torch.zeros_like(k) for k in self.K]
        self.T = 0

    def lin(self, x, l, kind):
        w, out = self.w[(l, kind)], []
        for r in range(0, w.shape[0], 16384):
            out.append(x @ w[r:r + 16384].double().t())
        return torch.cat(out, -1)

    def rope(self, x, pos):
        half = self.c["hd"] // 2
        inv = self.c["theta"] ** (-2.0 * torch.arange(half, dtype=torch.float64, device="cuda") / self.c["hd"])
        a = pos.double()[:, None] * inv
        cs, sn = a.cos()[:, None], a.sin()[:, None]
        x1, x2 = x[..., :half], x[..., half:]
        return torch.cat([x1 * cs - x2 * sn, x2 * cs + x1 * sn], -1)

    def forward(self, ids, tail):
        """Hidden states [L][tail, d] of the last `tail` of these positions, which join the cache."""
        c, m = self.c, len(ids)
        nq, nkv, hd = c["nq"], c["nkv"], c["hd"]
        h = self.w[(-1, "embed")][torch.tensor(ids, device="cuda")].double()
        pos = torch.arange(self.T, self.T + m, device="cuda")
        n, got = self.T + m, []
        for l in range(c["layers"]):
            x = _norm(h, self.w[(l, "attn_norm")].double())
            q = self.rope(self.lin(x, l, "wq").view(m, nq, hd), pos)
            k = self.rope(self.lin(x, l, "wk").view(m, nkv, hd), pos)
            v = self.lin(x, l, "wv").view(m, nkv, hd)
            self.K[l][:, self.T:n] = k.to(self.store).double().transpose(0, 1)
            self.V[l][:, self.T:n] = v.to(self.store).double().transpose(0, 1)
            o = torch.empty(m, nq, hd, dtype=torch.float64, device="cuda")
            late = torch.arange(n, device="cuda")[None, :] > pos[:, None]
            for j in range(nq):
                s = (q[:, j] @ self.K[l][j * nkv // nq, :n].t()) / math.sqrt(hd)
                o[:, j] = torch.softmax(s.masked_fill_(late, -math.inf), -1) @ self.V[l][j * nkv // nq, :n]
            h = h + self.lin(o.view(m, nq * hd), l, "wo")
            x = _norm(h, self.w[(l, "ffn_norm")].double())
            h = h + self.lin(torch.nn.functional.silu(self.lin(x, l, "wg")) * self.lin(x, l, "wu"), l, "wd")
            got.append(h[-tail:])
        self.T = n
        return got

    def head(self, hidden):
        """Logits of hidden states [rows, d]."""
        return self.lin(_norm(hidden, self.w[(-1, "final_norm")].double()), -1, "embed" if self.c["tied"] else "lm_head")


def _nucleus(z, temperature, top_p):
    """Probabilities (numpy float64) of one logits row under temperature and top_p."""
    w = np.exp((z - z.max()) / temperature)
    order = np.argsort(-z, kind="stable")
    cum = np.cumsum(w[order])
    n = int(np.searchsorted(cum, top_p * cum[-1])) + 1
    p = np.zeros_like(w)
    p[order[:n]] = w[order[:n]]
    return p / p.sum()


def _pick(p, r):
    cum = np.cumsum(p)
    return min(int(np.searchsorted(cum, r * cum[-1], side="right")), int(np.nonzero(p)[0][-1]))


class _Sums:
    """The decayed statistics (decay 0.95) over the rows given to add()."""

    def __init__(self, L):
        self.L, self.Sn = L, 0.0
        self.Sc, self.St, self.Sf = np.zeros(L + 1), np.zeros(L + 1), np.zeros(L + 1)

    def add(self, ids, conf):           # [L][rows]
        hit = ids == ids[-1:]
        self.Sn = 0.95 * self.Sn + ids.shape[1]
        self.Sc[1:] = 0.95 * self.Sc[1:] + hit.sum(1)
        self.St[1:] = 0.95 * self.St[1:] + (conf * hit).sum(1)
        self.Sf[1:] = 0.95 * self.Sf[1:] + (conf * ~hit).sum(1)

    def tau(self):
        miss = self.Sn - self.Sc
        a = np.divide(self.St, self.Sc, out=np.zeros(self.L + 1), where=self.Sc > 0)
        b = np.divide(self.Sf, miss, out=np.zeros(self.L + 1), where=miss > 0)
        t = 0.5 * (a + b)
        t[0] = 0.0
        return t

    def out(self, d_max):
        L, best = self.L, (-1.0, 1, 0)
        for l in range(1, L):
            a = self.Sc[l] / self.Sn
            for d in range(d_max + 1):
                v = sum(a ** i for i in range(d + 1)) / (d * l + L)
                if v > best[0]:
                    best = (v, l, d)
        return {"next": np.array(best[1:]), "S_n": self.Sn, "S_c": self.Sc, "S_tcs": self.St, "tau": self.tau()}


def exact(case, seed):
    c = dict(case)
    if c["kind"] == "sampling":
        q, p, u, _ = _logits(c, seed)
        V, g, t, tp = c["vocab"], c["gamma"], c["temperature"], c["top_p"]
        q, p, u = (x.double().cpu().numpy() for x in (q, p, u))
        Q, P = [_nucleus(r[:V], t, tp) for r in q], [_nucleus(r[:V], t, tp) for r in p]
        drafts = [_pick(Q[i], u[i]) for i in range(g)]
        n = next((i for i in range(g) if not u[g + i] * Q[i][drafts[i]] < P[i][drafts[i]]), g)
        last = _pick(P[g] if n == g else np.maximum(P[n] - Q[n], 0.0), u[2 * g])
        return torch.tensor([n, n + 1, last] + drafts, dtype=torch.int32)
    model, L = _Model(c, seed), c["layers"]
    sums, prompt = _Sums(L), _prompt(c, seed)
    w = min(32, len(prompt))
    done = 0
    while done < len(prompt):           # in pieces, so that the scores of a long prompt fit
        n = min(2048, len(prompt) - done)
        if 0 < len(prompt) - done - n < w:
            n = len(prompt) - done
        hid = model.forward(prompt[done:done + n], min(w, n))
        done += n

    def heads(hidden):
        """Greedy ids and confidences [L][rows], and every layer's logits of the last row."""
        ids, conf, last = [], [], []
        for h in hidden:
            z = model.head(h)
            ids.append(z.argmax(-1).cpu().numpy())
            conf.append((1.0 / (z - z.amax(-1, keepdim=True)).exp().sum(-1)).cpu().numpy())
            last.append(z[-1].cpu().numpy())
        return np.array(ids), np.array(conf), last

    ids, conf, z = heads(hid)
    sums.add(ids, conf)
    first = int(ids[-1][-1])
    if c["kind"] == "prefill":
        return {"tokens": np.array([first]), "logits": z[-1], "hidden": hid[-1][-1].cpu().numpy(),
                **sums.out(c["d_max"])}
    mode, E, log = c["control"], (1 if c["control"] == "vanilla" else c["E"]), []
    if mode == "sample":
        first = _pick(_nucleus(z[-1], TEMPERATURE, TOP_P), float(np.float32(_uniforms(seed, 0, 1)[0])))
    toks = [first]
    while len(toks) < c["tokens"]:
        cap = min(c["gamma"], c["tokens"] - len(toks) - 1)
        un = np.float32(_uniforms(seed, len(log) + 1, 2 * cap + 1)).astype(np.float64) if mode == "sample" else None
        tau, drafted, token, rows, out = sums.tau()[E], cap, toks[-1], [], []
        for i in range(cap + 1):
            hid = model.forward([token], 1)
            ids, conf, z = heads(hid)
            rows.append((ids[:, 0], conf[:, 0]))
            target = int(ids[-1][0])
            if mode == "sample":
                p = _nucleus(z[-1], TEMPERATURE, TOP_P)
                if i == cap:
                    out.append(_pick(p, un[2 * cap]))
                    break
                q = _nucleus(z[E - 1], TEMPERATURE, TOP_P)
                token = _pick(q, un[i])
                if not un[cap + i] * q[token] < p[token]:
                    out.append(_pick(np.maximum(p - q, 0.0), un[2 * cap]))
                    break
                out.append(token)
                continue
            if i == cap or (mode == "dynamic" and conf[E - 1][0] < tau):
                drafted = i
                out.append(target)
                break
            token = int(ids[E - 1][0])
            out.append(target)
            if token != target:
                if mode == "dynamic":   # how far the rejected draft ran on is not followed here
                    return None
                break
        sums.add(np.array([r[0] for r in rows]).T, np.array([r[1] for r in rows]).T)
        toks += out
        log.append((E, drafted, len(out)))
    return {"tokens": np.array(toks), "rounds": np.array(log), "logits": z[-1],
            "hidden": hid[-1][-1].cpu().numpy(), **sums.out(c["d_max"])}
