"""The calls that rollout users make, as timed cases.

A GRPO step generates groups of completions (prefill of the prompts, then one
decode step and one draw per token) and normalises their rewards.  The cases
are those calls at the widths of the 7B, 14B and 72B decoders the package names
and at the tiny fp32 model of its smoke test: whole prefills, teacher-forced
decode (the logits do not depend on a draw, so they can be compared), draws,
advantages, and one whole fp32 rollout.  The large models run with one to four
of their layers and the full vocabulary; every layer of a model costs the same,
so depth repeats what is timed here.

Inputs are synthetic: seeded weights of the library's generator, uniform prompt
tokens, normal logits, rewards on a coarse grid.  ``exact`` recomputes the
outputs in float64 from the same weights, prompts and uniforms.
"""
import math

import torch

import paper_2608_11226_amd as R

DEV = "cuda:0"
STD = 0.02
DTYPES = {"fp32": R.DTYPE_FP32, "bf16": R.DTYPE_BF16, "int4": R.DTYPE_INT4}
_stream = None


def listed():
    return [
        # advantages of one benchmark step's 8 groups of 8 completions: the smallest call
        {"name": "advantages_8x8", "kind": "advantages", "groups": 8, "G": 8},
        # the smoke test's whole rollout (2 prompts x 16 tokens, G = 4, 16 new tokens), fp32: launches and latency
        {"name": "generate_tiny", "kind": "generate", "prompts": 2, "P": 16, "G": 4, "new": 16},
        # the draw after every decode step of the 7B benchmark
        {"name": "sample_7b", "kind": "sample", "rows": 64, "temperature": 0.9, "top_p": 0.95},
        # prompts of the 7B benchmark's wave: 8 x 256 tokens
        {"name": "prefill_7b", "kind": "prefill", "model": "7b", "dtype": "bf16", "layers": 2, "prompts": 8, "P": 256, "G": 8},
        # prompts of the 14B benchmark's wave: 16 x 512 tokens
        {"name": "prefill_14b", "kind": "prefill", "model": "14b", "dtype": "bf16", "layers": 2, "prompts": 16, "P": 512, "G": 16},
        # one prompt of an odd length admitted by continuous batching while other slots decode
        {"name": "prefill_refill", "kind": "prefill", "model": "7b", "dtype": "bf16", "layers": 2, "prompts": 1, "P": 203, "G": 8},
        # a long document as prompt (contexts past 4,000 tokens, as the tests cover)
        {"name": "prefill_long", "kind": "prefill", "model": "7b", "dtype": "bf16", "layers": 2, "prompts": 1, "P": 3967, "G": 4},
        # prompts of the 72B generation proxy with int4 layer projections
        {"name": "prefill_int4", "kind": "prefill", "model": "72b", "dtype": "int4", "layers": 1, "prompts": 4, "P": 512, "G": 8},
        # the 7B benchmark's wave: 64 sequences in flight
        {"name": "decode_7b", "kind": "decode", "model": "7b", "dtype": "bf16", "layers": 4, "prompts": 8, "P": 256, "G": 8, "steps": 48},
        # the 14B benchmark's wave: 256 sequences in flight
        {"name": "decode_14b", "kind": "decode", "model": "14b", "dtype": "bf16", "layers": 2, "prompts": 16, "P": 512, "G": 16, "steps": 24},
        # one group of the paper's G = 4 with a long context: few sequences in flight
        {"name": "decode_long", "kind": "decode", "model": "7b", "dtype": "bf16", "layers": 2, "prompts": 1, "P": 2999, "G": 4, "steps": 64},
        # the 72B generation proxy's wave with int4 layer projections, ragged prompt
        {"name": "decode_int4", "kind": "decode", "model": "72b", "dtype": "int4", "layers": 1, "prompts": 8, "P": 121, "G": 8, "steps": 24},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["advantages", "generate", "sample", "prefill", "prefill", "prefill", "decode", "decode", "decode"])
    if kind == "advantages":
        return {"kind": kind, "groups": _log(rng, 1, 4096), "G": rng.randint(1, 64)}
    if kind == "generate":
        return {"kind": kind, "prompts": rng.randint(1, 8), "P": _log(rng, 3, 96), "G": rng.choice([1, 2, 4, 8]),
                "new": rng.randint(2, 24)}
    if kind == "sample":
        t = rng.choice([0.0, 0.7, 0.9, 1.0])
        return {"kind": kind, "rows": _log(rng, 1, 256), "temperature": t, "top_p": rng.choice([1.0, 0.95, 0.9])}
    model = rng.choice(["7b", "14b", "72b"])
    case = {"kind": kind, "model": model, "dtype": rng.choice(["bf16", "bf16", "int4"]), "layers": 1}
    G = rng.choice([1, 2, 4, 8, 16])
    # at most 4,096 prompt tokens and 256 sequences, below the 14B wave's
    P = _log(rng, 16, 3000)
    prompts = _log(rng, 1, max(1, min(4096 // P, 256 // G)))
    case.update({"prompts": prompts, "P": P, "G": G})
    if kind == "decode":
        case["steps"] = rng.randint(6, 20)
    return case


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _tokens(seed, stream, shape, vocab):
    g = torch.Generator().manual_seed(seed * 8 + stream)
    return torch.randint(0, vocab, shape, generator=g, dtype=torch.int32)


def _uniforms(seed, shape):
    g = torch.Generator().manual_seed(seed * 8 + 5)
    return torch.rand(shape, generator=g, dtype=torch.float32)


def _rewards(case, seed):
    g = torch.Generator().manual_seed(seed * 8 + 6)
    # closeness to a length target on a coarse grid: small groups with equal rewards occur
    return torch.floor(torch.rand(case["groups"] * case["G"], generator=g) * 16) / 16


def _logits(case, seed):
    g = torch.Generator(device=DEV).manual_seed(seed * 8 + 7)
    V = R.SHAPES["7b"][6]
    # from a random-init model's spread (1.2) to a trained model's peaked rows
    spread = 1.2 + 3.0 * torch.rand((case["rows"], 1), generator=g, device=DEV)
    return torch.randn((case["rows"], V), generator=g, device=DEV) * spread


def _seed64(seed):
    return seed % (1 << 32)


def _shape(case):
    return R.SHAPES["tiny" if case["kind"] == "generate" else case["model"]]


def _layers(case):
    return R.SHAPES["tiny"][0] if case["kind"] == "generate" else case["layers"]


def _the_stream():
    global _stream
    if _stream is None:
        _stream = torch.cuda.Stream(device=DEV)  # one stream for every engine of the program
    return _stream


def _engine(case, seed):
    S = case["prompts"] * case["G"]
    new = case.get("new", case.get("steps", 1))
    dtype = R.DTYPE_FP32 if case["kind"] == "generate" else DTYPES[case["dtype"]]
    cfg = R.model_config(_shape(case), dtype, case["P"], new, S, n_layers=_layers(case), weight_seed=_seed64(seed),
                         weight_std=STD)
    return R.Engine(cfg, group_size=case["G"], device=DEV, stream=_the_stream())


def prepare(case, seed):
    kind = case["kind"]
    st = {"case": case}
    if kind == "advantages":
        st["rewards"] = _rewards(case, seed).to(DEV)
        st["adv"] = torch.empty_like(st["rewards"])
        st["zero"] = torch.zeros(1, dtype=torch.int32, device=DEV)
        st["stream"] = _the_stream().cuda_stream
    elif kind == "sample":
        n, V = case["rows"], R.SHAPES["7b"][6]
        # the draw reads the vocabulary and the row capacity of its context, nothing of the model
        cfg = R.model_config((1, 128, 4, 4, 32, 512, V, 1e4), R.DTYPE_FP32, 8, 1, n)
        st["eng"] = R.Engine(cfg, device=DEV, stream=_the_stream())
        st["logits"] = _logits(case, seed)
        st["u"] = _uniforms(seed, (n,)).to(DEV)
        st["tokens"] = torch.empty(n, dtype=torch.int32, device=DEV)
    else:
        V, S = _shape(case)[6], case["prompts"] * case["G"]
        st["eng"] = _engine(case, seed)
        st["prompts"] = _tokens(seed, 0, (case["prompts"], case["P"]), V).to(DEV)
        st["logits"] = torch.empty((S, V), dtype=torch.float32, device=DEV)
        if kind == "decode":
            st["feed"] = _tokens(seed, 1, (case["steps"], S), V).to(DEV)
            st["first"] = torch.empty((S, V), dtype=torch.float32, device=DEV)
        if kind == "generate":
            st["u"] = _uniforms(seed, (S, case["new"])).to(DEV)
            st["tokens"] = torch.empty((S, case["new"]), dtype=torch.int32, device=DEV)
            st["last"] = torch.empty(S, dtype=torch.int32, device=DEV)
    torch.cuda.synchronize()
    return st


def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "advantages":
        R.grpo_advantages(st["rewards"], case["groups"], case["G"], 0.0, 1, st["adv"], st["zero"], st["stream"])
        return {"adv": st["adv"], "zero": st["zero"]}
    eng = st["eng"]
    if kind == "sample":
        R.rollout_sample(eng.ctx, st["logits"], case["rows"], case["temperature"], case["top_p"], st["u"], st["tokens"])
        return {"tokens": st["tokens"]}
    n, P, G = case["prompts"], case["P"], case["G"]
    if kind == "prefill":
        R.rollout_prefill(eng.ctx, st["prompts"], n, P, G, st["logits"])
        return {"logits": st["logits"]}
    if kind == "decode":
        R.rollout_prefill(eng.ctx, st["prompts"], n, P, G, st["first"])
        for t in range(case["steps"]):
            R.rollout_decode_step(eng.ctx, st["feed"][t], st["logits"])
        return {"first": st["first"], "logits": st["logits"]}
    # a whole rollout, then the logits after its last token
    R.rollout_generate(eng.ctx, st["prompts"], n, P, G, n * G, case["new"], 1.0, 1.0, st["u"], st["tokens"])
    with torch.cuda.stream(eng.stream):
        st["last"].copy_(st["tokens"][:, -1])
    R.rollout_decode_step(eng.ctx, st["last"], st["logits"])
    return {"tokens": st["tokens"], "logits": st["logits"]}


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------
def _layer_weights(t):
    d, qd, kvd, ff = t[1], t[2] * t[4], t[3] * t[4], t[5]
    return d * (qd + 2 * kvd) + qd * d + 3 * d * ff


def work(case):
    kind = case["kind"]
    if kind == "advantages":
        n = case["groups"] * case["G"]
        return {"bytes": 8 * n + 4, "flops": 6 * n}
    if kind == "sample":
        n = case["rows"] * R.SHAPES["7b"][6]
        return {"bytes": 4 * n, "flops": 3 * n}
    t, L = _shape(case), _layers(case)
    d, nh, nkv, hd, V = t[1], t[2], t[3], t[4], t[6]
    n, P, G = case["prompts"], case["P"], case["G"]
    S = n * G
    eb = 4 if kind == "generate" else 2
    params = _layer_weights(t)
    # int4: four bits a weight, an fp32 scale and a byte of zero point per 128 of them
    wb = L * (params * (0.5 + 5 / 128) if case.get("dtype") == "int4" else params * eb)
    head = V * d * eb
    kv = 2 * nkv * hd * eb * L  # a token's keys and values
    flops = 2 * n * P * L * params + 2 * n * V * d + 2 * n * P * (P + 1) * nh * hd * L
    bytes_ = wb + head + n * P * (d * eb + kv) + S * V * 4
    steps = case.get("steps", case.get("new", 0))
    for i in range(steps):
        ctx = P + i + 1
        flops += 2 * S * (L * params + V * d) + 4 * S * ctx * nh * hd * L
        # every key and value of the wave once (a group's prompt is one copy), the new token's written
        bytes_ += wb + head + (n * P + S * (i + 1)) * kv + S * (d * eb + V * 4)
    return {"bytes": bytes_, "flops": flops}


def tolerance(case):
    if case["kind"] == "sample":
        return "exact"  # the draw decides on exact sums of the fp32 exponentials
    if case["kind"] == "advantages":
        return {"rel": 1e-5}
    if case["kind"] == "generate":
        return {"rel": 1e-5, "max": 1e-3}
    # Flipped bf16 roundings: the decode attention with four and with eight waves (another order of its sums)
    # differs by 1.7e-3 after one layer, 4e-3 after two and 5.7e-3 after four, at most 0.033 of the root mean
    # square in one logit; four times that.
    return {"rel": 1.1e-2 * math.sqrt(_layers(case)), "max": 0.13}


# ---------------------------------------------------------------------------
# float64 results
# ---------------------------------------------------------------------------
def _i64(v):
    v &= (1 << 64) - 1
    return v - (1 << 64) if v >> 63 else v


def _mix(z):
    def shr(x, s):  # logical shift
        return (x >> s) & ((1 << (64 - s)) - 1)

    z = (z ^ shr(z, 30)) * _i64(0xBF58476D1CE4E5B9)
    z = (z ^ shr(z, 27)) * _i64(0x94D049BB133111EB)
    return z ^ shr(z, 31)


_GAMMA = 0x9E3779B97F4A7C15


def _weights(seed, tensor, index):
    """fp32 weights at the flat indices of one tensor: SplitMix64 hash, sum of four 16-bit limbs, scaled."""
    key = _mix(torch.tensor(_i64(_seed64(seed) ^ ((tensor * _GAMMA) & ((1 << 64) - 1))), device=DEV))
    v = _mix(key + (index + 1) * _i64(_GAMMA))
    s = (v & 0xFFFF) + ((v >> 16) & 0xFFFF) + ((v >> 32) & 0xFFFF) + ((v >> 48) & 0xFFFF)
    return (((s - 131070).double() / 65536.0) * 1.7320508075688772 * STD).float()


def _rows(seed, tensor, rows, cols, dtype):
    """Rows of a weight matrix as the model multiplies with them, float64."""
    out = torch.empty((rows.numel(), cols), dtype=torch.float64, device=DEV)
    for i in range(0, rows.numel(), 8192):
        r = rows[i:i + 8192].long()
        w = _weights(seed, tensor, r[:, None] * cols + torch.arange(cols, device=DEV)[None, :])
        if dtype == "bf16":
            w = w.bfloat16()
        elif dtype == "int4":  # groups of 128 inputs: scale (hi - lo) / 15, zero rint(-lo / s), 4-bit codes
            g = w.view(w.shape[0], cols // 128, 128)
            lo, hi = g.amin(2, keepdim=True), g.amax(2, keepdim=True)
            s = (hi - lo) / 15
            z = torch.clamp(torch.round(-lo / s), 0, 15)
            q = torch.clamp(torch.round(g / s) + z, 0, 15)
            w = ((q - z).double() * s.double()).view(w.shape[0], cols)
        out[i:i + 8192] = w.double()
    return out


def _rope(x, pos, theta):
    half = x.shape[-1] // 2
    inv = torch.pow(torch.tensor(theta, dtype=torch.float64, device=DEV),
                    -torch.arange(half, dtype=torch.float64, device=DEV) / half)
    a = pos.double()[:, None] * inv[None, :]
    c, s = torch.cos(a)[:, None, :], torch.sin(a)[:, None, :]
    x1, x2 = x[..., :half], x[..., half:]
    return torch.cat([x1 * c - x2 * s, x2 * c + x1 * s], -1)


def _norm(x):
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + 1e-6)


class _Model64:
    def __init__(self, case, seed):
        self.t, self.L, self.seed = _shape(case), _layers(case), seed
        dtype = "fp32" if case["kind"] == "generate" else case["dtype"]
        self.layer_type, self.table_type = dtype, "bf16" if dtype == "int4" else dtype

    def mat(self, layer, slot, n, k):
        return _rows(self.seed, 1 + 9 * layer + slot, torch.arange(n, device=DEV), k, self.layer_type)

    def logits(self, x):
        d, V = self.t[1], self.t[6]
        x = _norm(x)
        out = torch.empty((x.shape[0], V), dtype=torch.float64, device=DEV)
        for i in range(0, V, 8192):
            r = torch.arange(i, min(V, i + 8192), device=DEV)
            out[:, i:i + 8192] = x @ _rows(self.seed, 2 + 9 * self.L, r, d, self.table_type).T
        return out

    def attend(self, q, k, v, causal):
        """q [A, nh, hd] against k, v [B, nkv, hd]; causal: query a sees keys up to B - A + a."""
        nh, nkv, hd = self.t[2], self.t[3], self.t[4]
        out = torch.empty_like(q)
        a, b = q.shape[0], k.shape[0]
        seen = torch.arange(b, device=DEV)[None, :] <= torch.arange(b - a, b, device=DEV)[:, None]
        for h in range(nh):
            kh = h // (nh // nkv)
            s = (q[:, h] @ k[:, kh].T) / math.sqrt(hd)
            out[:, h] = torch.softmax(s.masked_fill(~seen, -math.inf), -1) @ v[:, kh]
        return out

    def forward(self, prompts, suffix):
        """Logits after each prompt [n, V], and after the last suffix token of each sequence [S, V] (suffix
        [S, T] group-major, or None)."""
        d, nh, nkv, hd, ff, theta = self.t[1], self.t[2], self.t[3], self.t[4], self.t[5], self.t[7]
        n, P = prompts.shape
        S, T = (suffix.shape if suffix is not None else (0, 0))
        G = S // n if S else 1
        ids = prompts.reshape(-1) if not S else torch.cat([prompts.reshape(-1), suffix.reshape(-1)])
        x = _rows(self.seed, 0, ids.to(DEV), d, self.table_type)
        pos = torch.arange(P, device=DEV).repeat(n)
        if S:
            pos = torch.cat([pos, (P + torch.arange(T, device=DEV)).repeat(S)])
        for l in range(self.L):
            a = _norm(x)
            q = _rope((a @ self.mat(l, 1, nh * hd, d).T).view(-1, nh, hd), pos, theta)
            k = _rope((a @ self.mat(l, 2, nkv * hd, d).T).view(-1, nkv, hd), pos, theta)
            v = (a @ self.mat(l, 3, nkv * hd, d).T).view(-1, nkv, hd)
            o = torch.empty_like(q)
            for p in range(n):
                r = slice(p * P, (p + 1) * P)
                o[r] = self.attend(q[r], k[r], v[r], True)
                for g in range(G if S else 0):
                    i = n * P + (p * G + g) * T
                    w = slice(i, i + T)
                    o[w] = self.attend(q[w], torch.cat([k[r], k[w]]), torch.cat([v[r], v[w]]), True)
            x = x + o.view(-1, nh * hd) @ self.mat(l, 4, d, nh * hd).T
            b = _norm(x)
            m = torch.nn.functional.silu(b @ self.mat(l, 6, ff, d).T) * (b @ self.mat(l, 7, ff, d).T)
            x = x + m @ self.mat(l, 8, d, ff).T
        first = self.logits(x[P - 1:n * P:P])
        return first, self.logits(x[n * P + T - 1::T]) if S else None


def exact(case, seed):
    kind = case["kind"]
    if kind == "sample":
        return None  # token ids, decided on exact integer sums of the fp32 exponentials
    if kind == "advantages":
        r = _rewards(case, seed).double().view(case["groups"], case["G"])
        same = r.amax(1) == r.amin(1)
        std = r.std(1, keepdim=True) if case["G"] > 1 else torch.ones_like(r)
        adv = torch.where(same[:, None], torch.zeros_like(r), (r - r.mean(1, keepdim=True)) / std)
        return {"adv": adv.reshape(-1), "zero": same.sum().to(torch.int32).view(1)}
    V, n, G = _shape(case)[6], case["prompts"], case["G"]
    model = _Model64(case, seed)
    prompts = _tokens(seed, 0, (n, case["P"]), V).to(DEV)
    if kind == "prefill":
        return {"logits": model.forward(prompts, None)[0].repeat_interleave(G, 0)}
    if kind == "decode":
        feed = _tokens(seed, 1, (case["steps"], n * G), V).to(DEV)
        first, last = model.forward(prompts, feed.T.contiguous())
        return {"first": first.repeat_interleave(G, 0), "logits": last}
    u = _uniforms(seed, (n * G, case["new"])).to(DEV).double()
    z = model.forward(prompts, None)[0].repeat_interleave(G, 0)
    tokens = torch.empty((n * G, 0), dtype=torch.int32, device=DEV)
    for t in range(case["new"]):
        c = torch.cumsum(torch.exp(z - z.amax(1, keepdim=True)), 1)
        pick = (c > u[:, t:t + 1] * c[:, -1:]).int().argmax(1).int()
        tokens = torch.cat([tokens, pick[:, None]], 1)
        z = model.forward(prompts, tokens)[1]
    return {"tokens": tokens, "logits": z}
