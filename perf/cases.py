"""The framework's timed cases: what the Profiler does with a fingerprint, through the public
entry points (Fingerprint.prefill, decode_step, decode_steps, head and generate).

A case is one request, or one part of it, on a one-layer fingerprint (`layers` hidden layers
in general): a prefill over a prompt (time to first token), decode steps after it (time per
output token), the LM head alone, or a whole request on token ids.  Shapes are those of the
workload table (the tiny fingerprint, Llama-2 7B and 13B layers, a 1/8 tensor-parallel shard
of a 70B layer) and a generic grouped-query shape of odd sizes.  `exact` is the same layer in
plain torch in 64 bits, with values rounded to bf16 at the points where the layer defines
them to be (normalised rows, attention output, residual sums, the SwiGLU product) and the
weights and KV cache quantised as their formats say.
"""
import math
import types

import numpy as np
import torch

SHAPES = {
    # name: hidden, heads, kv heads, head_dim, ffn
    "tiny": (256, 4, 4, 64, 688),
    "7b": (4096, 32, 32, 128, 11008),
    "13b": (5120, 40, 40, 128, 13824),
    "70b-tp8": (8192, 8, 1, 128, 3584),
    "gqa-odd": (1536, 24, 6, 64, 4240),
}
VOCAB = 32000


def _case(name, kind, shape, wq, kvq, B, P, n=0, layers=1):
    H, nh, nkv, d, F = SHAPES[shape] if isinstance(shape, str) else shape
    c = {"kind": kind, "layers": layers, "hidden": H, "heads": nh, "kv_heads": nkv, "head_dim": d, "ffn": F,
         "wq": wq, "kvq": kvq, "B": B, "P": P, "n": n, "vocab": VOCAB if kind in ("generate", "head") else 0}
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest fingerprint, one sequence, one call per token: launch latency
        _case("tiny-steps", "steps", "tiny", "bf16", "bf16", 1, 32, 16),
        # time to first token of a single ordinary prompt
        _case("7b-bf16-prefill", "prefill", "7b", "bf16", "bf16", 1, 512),
        # one user's request, unquantised: the weight stream of single-sequence decode
        _case("7b-bf16-request", "request", "7b", "bf16", "bf16", 1, 512, 16),
        # a batch of requests with int8 weights and an int8 cache
        _case("7b-int8-request", "request", "7b", "int8", "int8", 16, 512, 16),
        # the same batch with 2:4 sparse weights and shorter prompts: mostly decode
        _case("7b-sp24-request", "request", "7b", "sp24", "bf16", 16, 128, 16),
        # a large batch's prompts with int4 weights
        _case("13b-int4-prefill", "prefill", "13b", "int4", "bf16", 32, 1024),
        # the same batch over shorter prompts, decode included
        _case("13b-int4-request", "request", "13b", "int4", "bf16", 32, 128, 16),
        # the largest: 64 prompts of 2048 tokens on a tensor-parallel shard, grouped queries
        _case("70b-tp8-prefill", "prefill", "70b-tp8", "int4", "int8", 64, 2048),
        # that shard's decode (many small projections per step)
        _case("70b-tp8-request", "request", "70b-tp8", "int4", "int8", 64, 128, 16),
        # a whole request on token ids with one sequence and int4 weights: embedding, layer,
        # final norm and LM head per token
        _case("7b-int4-generate", "generate", "7b", "int4", "int8", 1, 100, 16),
        # the LM head of a batch (the "other" share of TTFT and TPOT)
        _case("7b-head", "head", "7b", "bf16", "bf16", 16, 1),
        # odd sizes: ragged rows and columns, grouped queries, head_dim 64, one call per token
        _case("gqa-odd-steps", "steps", "gqa-odd", "int8", "bf16", 7, 333, 9),
    ]


def draw(rng):
    """A case of the same ranges: any kind, weight and cache format, batches of 1 to 64, prompts
    of 1 to 2048 tokens, layer shapes from the tiny one to the 13B one, costing no more than
    the largest listed case."""
    while True:
        kind = rng.choice(["prefill", "prefill", "request", "request", "steps", "generate", "head"])
        wq = rng.choice(["bf16", "int8", "int4", "sp24"])
        kvq = rng.choice(["bf16", "int8"])
        if rng.random() < 0.5:
            shape = SHAPES[rng.choice(["7b", "13b", "70b-tp8"])]
        else:
            d = rng.choice([64, 128])
            nkv = rng.choice([1, 2, 4, 5, 8, 16])
            g = rng.choice([1, 2, 3, 4, 8])
            mult = {"int4": 128, "sp24": 64}.get(wq, 16)
            if nkv * g * d % mult:
                nkv *= 2
            hid = mult * max(1, round(2 ** rng.uniform(8, 12.5) / mult))
            ffn = mult * max(1, round(hid * rng.uniform(1.5, 4) / mult))
            shape = (hid, nkv * g, nkv, d, ffn)
        B = max(1, min(64, round(2 ** rng.uniform(0, 6))))
        P = max(1, min(2048, round(2 ** rng.uniform(0, 11))))
        n = rng.randint(1, 16) if kind in ("request", "steps", "generate") else 0
        if kind == "head":
            P = 1
        c = _case(None, kind, shape, wq, kvq, B, P, n)
        top = work(listed()[7])
        w = work(c)
        if w["flops"] <= 0.5 * top["flops"] and w["bytes"] <= top["bytes"] and shape[1] * shape[3] <= 8192:
            return c


# ------------------------------------------------------------------ what a pass needs
def _dims(c):
    qd, kd = c["heads"] * c["head_dim"], c["kv_heads"] * c["head_dim"]
    return [(qd + 2 * kd, c["hidden"]), (c["hidden"], qd), (2 * c["ffn"], c["hidden"]), (c["hidden"], c["ffn"])]


def work(c):
    """Bytes and operations of one pass: every weight read once for the prefill and once more
    for each decode step (a step needs the previous one's output), the cached keys and
    values written once and read once by each step, hidden states in and out; multiply-adds
    of the projections (2:4 weights: the kept half), causal attention and the LM head."""
    H, B, P, n, L = c["hidden"], c["B"], c["P"], c["n"], c["layers"]
    per = {"bf16": 2.0, "int8": 1.0, "int4": 0.5 + 4.0 / 128, "sp24": 1.125}[c["wq"]]
    wbytes = sum(N * K for N, K in _dims(c)) * per * L
    wflops = 2.0 * sum(N * K for N, K in _dims(c)) * (0.5 if c["wq"] == "sp24" else 1.0) * L
    kv = c["kv_heads"] * (2 * c["head_dim"] * (1 if c["kvq"] == "int8" else 2) + (4 if c["kvq"] == "int8" else 0)) * L
    aflops = 4.0 * c["head_dim"] * c["heads"] * L          # per (query, key) pair
    head_b, head_f = 2.0 * c["vocab"] * H + 4.0 * B * c["vocab"], 2.0 * B * c["vocab"] * H
    if c["kind"] == "head":
        return {"bytes": head_b + 2.0 * B * H, "flops": head_f}
    b = wbytes + B * P * (kv + 4.0 * H)
    f = wflops * B * P + aflops * B * P * (P + 1) / 2
    for i in range(n):
        b += wbytes + B * kv * (P + i + 1) + B * 4.0 * H
        f += wflops * B + aflops * B * (P + i + 1)
    if c["kind"] == "generate":
        b += (n + 1) * head_b
        f += (n + 1) * head_f
    return {"bytes": b, "flops": f}


def tolerance(c):
    if c["kind"] == "head":
        # fp32 sums of exact products; a normalised value in a few tens of thousands lies so
        # close to a bf16 boundary that another order of the row's sum rounds it the other way
        return {"rel": 5e-5, "max": 1e-3}
    if c["kind"] == "prefill":
        # one layer: bf16 at six points, measured 4e-3 to 5.5e-3 from 64 bits
        return {"rel": 2e-2, "max": 0.13}
    # each decode step takes the step before it (or the cache that it left) as its input, so
    # a rounding travels on: measured 4e-3 to 2.3e-2 from 64 bits after up to 16 steps
    return {"rel": 3e-2, "max": 0.4}


# ------------------------------------------------------------------ inputs and the timed pass
def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed) % (1 << 62))


def _inputs(c, seed):
    """Prompt hidden states ~N(0, 1) [B, P, H] in bf16, or token ids (prompt, forced tokens)."""
    g = _gen(seed)
    if c["kind"] == "generate":
        ids = torch.randint(0, c["vocab"], (c["B"], c["P"]), generator=g, device="cuda", dtype=torch.int32)
        force = torch.randint(0, c["vocab"], (max(c["n"], 1), c["B"]), generator=g, device="cuda", dtype=torch.int32)
        return ids, force[:c["n"]].contiguous()
    return torch.randn(c["B"], c["P"], c["hidden"], generator=g, device="cuda", dtype=torch.bfloat16)


def prepare(c, seed):
    from paper_2501_13111_amd import Fingerprint
    shape = types.SimpleNamespace(n_layers=c["layers"], hidden=c["hidden"], n_heads=c["heads"], n_kv_heads=c["kv_heads"],
                                  head_dim=c["head_dim"], ffn=c["ffn"], max_batch=c["B"], max_prompt=c["P"],
                                  max_seq=c["P"] + c["n"], rms_eps=1e-5, rope_theta=1e4, vocab=c["vocab"])
    s = {"case": c, "fp": Fingerprint(shape, c["wq"], c["kvq"], seed=int(seed))}
    B, n = c["B"], c["n"]
    if c["kind"] == "generate":
        s["ids"], s["force"] = _inputs(c, seed)
        s["out_ids"] = torch.empty(n + 1, B, dtype=torch.int32, device="cuda")
        s["logits"] = torch.empty(n + 1, B, c["vocab"], dtype=torch.float32, device="cuda")
    elif c["kind"] == "head":
        s["y"] = _inputs(c, seed)
        s["out_ids"] = torch.empty(B, dtype=torch.int32, device="cuda")
        s["logits"] = torch.empty(B, c["vocab"], dtype=torch.float32, device="cuda")
    else:
        s["x"] = _inputs(c, seed)
        s["y"] = torch.empty_like(s["x"])
        s["a"] = torch.empty(B, c["hidden"], dtype=torch.bfloat16, device="cuda")
        s["b"] = torch.empty_like(s["a"])
    return s


def run(s):
    c, fp = s["case"], s["fp"]
    if c["kind"] == "generate":
        fp.generate(s["ids"], c["n"], s["out_ids"], logits=s["logits"], force_ids=s["force"])
        return s["logits"]
    if c["kind"] == "head":
        fp.head(s["y"], c["B"], 1, s["out_ids"], logits=s["logits"])
        return s["logits"]
    fp.prefill(s["x"], s["y"], c["B"], c["P"])
    if c["kind"] == "prefill":
        return s["y"]
    a, b = s["a"], s["b"]
    a.copy_(s["y"][:, -1, :])                     # the first decode input: the prompt's last output
    if c["kind"] == "request":
        out = fp.decode_steps(a, b, c["n"])
        return [s["y"], out, b if out is a else a]
    for _ in range(c["n"]):                       # one call per token
        fp.decode_step(a, b)
        a, b = b, a
    return [s["y"], a, b]


# ------------------------------------------------------------------ the same in 64 bits
_M = (1 << 64) - 1
_G = 0x9E3779B97F4A7C15


def _signed(v):
    v &= _M
    return v - (1 << 64) if v >> 63 else v


def _mix_int(z):
    z &= _M
    z = ((z ^ (z >> 30)) * 0xBF58476D1CE4E5B9) & _M
    z = ((z ^ (z >> 27)) * 0x94D049BB133111EB) & _M
    return z ^ (z >> 31)


def _mix(z):
    def sr(v, k):
        return (v >> k) & ((1 << (64 - k)) - 1)
    z = (z ^ sr(z, 30)) * _signed(0xBF58476D1CE4E5B9)
    z = (z ^ sr(z, 27)) * _signed(0x94D049BB133111EB)
    return z ^ sr(z, 31)


def _stream(seed, layer, tensor, n, mean, sigma):
    """The documented synthetic stream: Irwin-Hall sums of SplitMix64 words, bf16."""
    key = _mix_int(_mix_int(int(seed) & _M) + _G * (((layer + 1) << 8) | tensor))
    out = torch.empty(n, dtype=torch.bfloat16, device="cuda")
    for i0 in range(0, n, 1 << 24):
        i = torch.arange(i0, min(n, i0 + (1 << 24)), device="cuda", dtype=torch.int64)
        tot = torch.zeros_like(i)
        for k in range(3):
            w = _mix((3 * i + (k + 1)) * _signed(_G) + _signed(key))
            for sh in (0, 16, 32, 48):
                tot += (w >> sh) & 0xFFFF
        z = (tot - 393210).float() * (1.0 / 65536.0)
        v = z * torch.tensor(np.float32(sigma), device="cuda")
        out[i0:i0 + i.numel()] = (v + torch.tensor(np.float32(mean), device="cuda")).to(torch.bfloat16)
    return out


def _weight(c, seed, layer, tensor, N, K):
    """A projection's weights as its format represents them, in float64."""
    w = _stream(seed, layer, tensor, N * K, 0.0, 0.02).view(N, K)
    if c["wq"] == "bf16":
        return w.double()
    if c["wq"] == "sp24":
        g = w.view(N, K // 4, 4)
        mag = (g.view(torch.int16).to(torch.int32) & 0x7FFF) * 4 + torch.tensor([3, 2, 1, 0], device="cuda", dtype=torch.int32)
        keep = mag >= mag.topk(2, dim=-1).values[..., 1:]
        return torch.where(keep, g, torch.zeros_like(g)).view(N, K).double()
    f = w.float()
    if c["wq"] == "int8":
        return _int8(f)
    g = f.view(N, K // 128, 128)
    lo, hi = g.amin(-1).clamp(max=0), g.amax(-1).clamp(min=0)
    s = ((hi - lo) / 15.0).half().float()
    s = torch.where(hi == lo, torch.ones_like(s), s)
    z = (-lo / s).round().clamp(0, 15)
    q = ((g / s[..., None]).round() + z[..., None]).clamp(0, 15)
    return ((q.double() - z[..., None].double()) * s[..., None].double()).view(N, K)


def _int8(f):
    """float32 rows -> what symmetric int8 codes with one fp16 scale per row stand for."""
    s = (f.abs().amax(-1, keepdim=True) / 127.0).half().float()
    q = (f / torch.where(s == 0, torch.ones_like(s), s)).round().clamp(-127, 127)
    return torch.where(s == 0, torch.zeros_like(q), q).double() * s.double()


def _bf(x):
    """float64 rounded once to bf16 (nearest, ties to even), as float64."""
    m, e = torch.frexp(x)
    return torch.ldexp((m * 256.0).round(), e - 8)


def _norm(x, g):
    return _bf(x * torch.rsqrt((x * x).mean(-1, keepdim=True) + float(np.float32(1e-5))) * g)


class _Layer:
    def __init__(self, c, seed, layer, B, S):
        H, nh, nkv, d, F = c["hidden"], c["heads"], c["kv_heads"], c["head_dim"], c["ffn"]
        self.c = c
        self.g1 = _stream(seed, layer, 0, H, 1.0, 0.02).double()
        self.g2 = _stream(seed, layer, 5, H, 1.0, 0.02).double()
        rows = {1: (nh * d, H), 2: (nkv * d, H), 3: (nkv * d, H), 4: (H, nh * d), 6: (F, H), 7: (F, H), 8: (H, F)}
        self.w = {t: _weight(c, seed, layer, t, N, K).t().contiguous() for t, (N, K) in rows.items()}
        inv = float(np.float32(1e4)) ** (-2.0 * torch.arange(d // 2, device="cuda", dtype=torch.float64) / d)
        ang = torch.arange(S, device="cuda", dtype=torch.float64)[:, None] * inv
        self.cos, self.sin = ang.cos().float().double(), ang.sin().float().double()
        self.K = torch.zeros(B, nkv, S, d, dtype=torch.float64, device="cuda")
        self.V = torch.zeros_like(self.K)

    def _rope(self, u, p0):                       # u [T, heads, d] at positions p0 ..
        h = u.shape[-1] // 2
        c, s = (t[p0:p0 + u.shape[0], None, :] for t in (self.cos, self.sin))
        a, b = u[..., :h], u[..., h:]
        return torch.cat([a * c - b * s, b * c + a * s], -1)

    def attention(self, b, xn, p0):               # one sequence: xn [T, H]
        c = self.c
        nh, nkv, d = c["heads"], c["kv_heads"], c["head_dim"]
        T = xn.shape[0]
        q = self._rope((xn @ self.w[1]).view(T, nh, d), p0)
        k = self._rope((xn @ self.w[2]).view(T, nkv, d), p0)
        v = (xn @ self.w[3]).view(T, nkv, d)
        store = _bf if c["kvq"] == "bf16" else (lambda t: _int8(t.float()))
        self.K[b, :, p0:p0 + T] = store(k).transpose(0, 1)
        self.V[b, :, p0:p0 + T] = store(v).transpose(0, 1)
        end = p0 + T
        rep = nh // nkv
        Kt = self.K[b, :, :end].transpose(1, 2).repeat_interleave(rep, 0).contiguous()
        Vt = self.V[b, :, :end].repeat_interleave(rep, 0).contiguous()
        sc = torch.matmul(q.transpose(0, 1).contiguous(), Kt) * float(np.float32(1.0 / math.sqrt(d)))
        if T > 1:
            pos = torch.arange(end, device="cuda")
            sc.masked_fill_(pos[None, :] > pos[p0:end, None], -math.inf)
        return torch.matmul(torch.softmax(sc, -1), Vt).transpose(0, 1).reshape(T, nh * d)

    def mlp(self, h):
        hn = _norm(h, self.g2)
        g = hn @ self.w[6]
        return _bf(h + _bf(g * torch.sigmoid(g) * (hn @ self.w[7])) @ self.w[8])

    def step(self, x, p0):                        # x [B, T, H] float64 -> y
        B, T, H = x.shape
        h = torch.empty_like(x)
        for b in range(B):
            o = _bf(self.attention(b, _norm(x[b], self.g1), p0))
            h[b] = _bf(x[b] + o @ self.w[4])
        flat = h.view(B * T, H)
        return torch.cat([self.mlp(flat[i:i + 16384]) for i in range(0, B * T, 16384)]).view(B, T, H)


def exact(c, seed):
    B, P, n, H = c["B"], c["P"], c["n"], c["hidden"]
    if c["vocab"]:
        lm = _stream(seed, -1, 18, c["vocab"] * H, 0.0, 0.02).view(c["vocab"], H).double().t().contiguous()
        gf = _stream(seed, -1, 17, H, 1.0, 0.02).double()
    if c["kind"] == "head":
        return _norm(_inputs(c, seed)[:, -1].double(), gf) @ lm
    layers = [_Layer(c, seed, l, B, P + n) for l in range(c["layers"])]

    def forward(x, p0):
        for l in layers:
            x = l.step(x, p0)
        return x

    if c["kind"] == "generate":
        E = _stream(seed, -1, 16, c["vocab"] * H, 0.0, 0.02).view(c["vocab"], H)
        ids, force = _inputs(c, seed)
        y = forward(E[ids.long()].double(), 0)
        logits = [_norm(y[:, -1], gf) @ lm]
        for i in range(n):
            y = forward(E[force[i].long()].double()[:, None], P + i)
            logits.append(_norm(y[:, -1], gf) @ lm)
        return torch.stack(logits)
    y = forward(_inputs(c, seed).double(), 0)
    if c["kind"] == "prefill":
        return y
    outs = [y[:, -1:]]
    for i in range(n):
        outs.append(forward(outs[-1], P + i))
    return [y, outs[-1][:, 0], outs[-2][:, 0]]
