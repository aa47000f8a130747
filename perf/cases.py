"""The work a user of this library has it do, as cases that can be timed and compared.

Every case goes through the Python binding's public calls (Engine.prefill, Engine.round,
Engine.train_loss) on the model shapes of sd2_inputs/configs.py:

  generate   prefill of the prompts, then a few rounds, the emitted tokens kept after each: a whole
             short generation on the two small workloads, where launches and latency count
  first      prefill of the prompts and the first round: the time until the first tokens
  round      one round of a running generation: the decoding loop's body
  loss       the training objective's forward over one token sequence

Calls with few sequences run free (sd2_round).  With four sequences or more the decisions are given
(sd2_round_forced): among hundreds of sampled decisions one near-tie a run would else send two
correct implementations down different tokens, after which nothing can be compared; the kernels
are the same.  Logits are returned where they lie, in the caller's own workspace.
"""
import functools
import math

import numpy as np
import torch

from paper_2511_09844_amd import binding as B
from sd2_inputs import configs

STD = 0.02            # of every weight matrix, as sd2_inputs draws them
GAIN_STD = 0.1        # RMSNorm and LayerNorm gains are 1 + N(0, 0.1)
LN_EPS = 1e-5
RANK = 256            # hidden width of the conditional bias
FORMS = {"input": B.STEER_INPUT, "none": B.STEER_NONE, "mlp": B.STEER_MLP, "mlp-out": B.STEER_MLP_OUT,
         "cond": B.STEER_MLP_COND}
BASE = {"tiny": configs.TINY, "small": configs.SMALL, "8b": configs.LLAMA8B, "70b": configs.LLAMA70B}
ROOM = 1024           # tokens a running generation may still grow by


def _case(name, kind, model, batch=1, k=5, lo=512, hi=512, t=1.0, steer="input", rounds=1, lv=0, ld=0, n=0, chunk=0):
    base = BASE[model]
    c = {"kind": kind, "model": model, "batch": batch, "k": k, "lo": lo, "hi": hi, "t": t, "steer": steer,
         "rounds": rounds, "lv": lv or base.verifier.n_layers, "ld": ld or base.drafter.n_layers, "n": n,
         "chunk": chunk}
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest configuration, fp32 weights: launches and latency
        _case("tiny-f32-generate", "generate", "tiny", k=4, lo=32, hi=32, rounds=4),
        # a small greedy pair at its configured prompt
        _case("small-greedy-generate", "generate", "small", lo=128, hi=128, t=0.0, rounds=6),
        # single-user decoding, the benchmark's workload
        _case("8b-round", "round", "8b"),
        # single-user time to the first tokens
        _case("8b-first", "first", "8b"),
        # single-user decoding late in a long context, odd length
        _case("8b-long-round", "round", "8b", lo=6001, hi=6001),
        # the paper's own steering (three verifier layers, per-layer biases)
        _case("8b-mlp-round", "round", "8b", lo=301, hi=301, steer="mlp"),
        # two users, short drafts, short ragged prompts
        _case("8b-b2-round", "round", "8b", batch=2, k=3, lo=37, hi=333),
        # a few users
        _case("8b-b4-round", "round", "8b", batch=4, lo=201, hi=901),
        # the batched benchmark workload: 16 ragged sequences
        _case("8b-b16-round", "round", "8b", batch=16, k=7, lo=256, hi=2048, t=0.7),
        # 16 ragged prompts arriving together: time to their first tokens
        _case("8b-b16-first", "first", "8b", batch=16, k=7, lo=64, hi=512, t=0.7),
        # the 70B verifier's layers (16 of the 80, so that several states fit one card), batch 4
        _case("70b-16l-b4-round", "round", "70b", batch=4, k=8, lo=1024, hi=1024, lv=16),
        # training objective over one sequence, an odd length in chunks of 512
        _case("8b-loss", "loss", "8b", n=1001, chunk=512),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, round(math.exp(rng.uniform(math.log(lo), math.log(hi + 0.5))))))


def draw(rng):
    kind = rng.choice(["generate", "generate", "round", "round", "round", "first", "first", "loss"])
    t = rng.choice([0.0, 0.7, 1.0])
    if kind == "generate":
        hi = _log_int(rng, 2, 512)
        return _case(None, kind, rng.choice(["tiny", "small"]), batch=_log_int(rng, 1, 8), k=rng.randint(1, 8),
                     lo=_log_int(rng, 1, hi), hi=hi, t=t, steer=rng.choice(["input", "input", "none"]),
                     rounds=rng.randint(1, 6))
    # half or all of the 8B pair's depth, 8 or 16 of the 70B layers
    model = rng.choice(["8b", "8b", "8b", "70b"])
    lv, ld = rng.choice([(16, 8), (32, 16)]) if model == "8b" else rng.choice([(8, 8), (16, 16)])
    steer = rng.choice(["input", "input", "input", "none", "mlp", "mlp-out", "cond"])
    if kind == "loss":
        n = _log_int(rng, 16, 1000)
        return _case(None, kind, model, k=rng.randint(1, 8), n=n, chunk=_log_int(rng, max(1, n // 6), 512), lv=lv,
                     ld=ld)
    batch = _log_int(rng, 1, 16)
    hi = _log_int(rng, 8, min(6000, (16384 if kind == "round" else 6000) // batch))
    return _case(None, kind, model, batch=batch, k=rng.randint(1, 8), lo=_log_int(rng, 4, hi), hi=hi, t=t, steer=steer,
                 lv=lv, ld=ld)


# ---- shapes ---------------------------------------------------------------------------------

def _workload(case):
    base = BASE[case["model"]]
    dims = [configs.Dims(case[key], d.d_model, d.n_heads, d.n_kv_heads, d.d_ff, d.vocab, d.rope_theta, d.rms_eps)
            for key, d in (("lv", base.verifier), ("ld", base.drafter))]
    room = {"round": ROOM, "loss": 1}.get(case["kind"], case["rounds"] * (case["k"] + 1) + 1)
    hi = case["n"] if case["kind"] == "loss" else case["hi"]
    return configs.Workload("case", dims[0], dims[1], base.dtype, case["k"], case["batch"], (case["lo"], hi), room,
                            case["t"])


def _lens(case):
    """Prompt lengths: spread evenly over the range, the longest one first."""
    b, lo, hi = case["batch"], case["lo"], case["hi"]
    return [hi - (hi - lo) * i // max(1, b - 1) for i in range(b)]


def _forced(case):
    return case["batch"] >= 4


def _shapes(dm, which):
    hd = dm.head_dim
    for name, shape in (("embed", (dm.vocab, dm.d_model)), ("final_norm", (dm.d_model,)),
                        ("lm_head", (dm.vocab, dm.d_model))):
        yield (which, name), shape
    for layer in range(dm.n_layers):
        for name, shape in (("attn_norm", (dm.d_model,)), ("wq", (dm.n_heads * hd, dm.d_model)),
                            ("wk", (dm.n_kv_heads * hd, dm.d_model)), ("wv", (dm.n_kv_heads * hd, dm.d_model)),
                            ("wo", (dm.d_model, dm.n_heads * hd)), ("ffn_norm", (dm.d_model,)),
                            ("w_gate", (dm.d_ff, dm.d_model)), ("w_up", (dm.d_ff, dm.d_model)),
                            ("w_down", (dm.d_model, dm.d_ff))):
            yield (which, layer, name), shape


def _steer_shapes(wl, steer):
    dv, dd, ld, f = wl.verifier.d_model, wl.drafter.d_model, wl.drafter.n_layers, wl.drafter.d_ff
    if steer == "none":
        return
    if steer == "input":
        yield "w_s", (dd, dv)
        return
    yield "w_s", {"mlp": (ld * f, dv), "mlp-out": (dd, dv), "cond": (ld * RANK, dv)}[steer]
    yield "w_hml", (dv, 3 * dv)
    yield "ln_gain", (dv,)
    yield "ln_bias", (dv,)
    if steer == "cond":
        yield "w_cf", (ld * RANK, dd)
        yield "w_cu", (ld * f, RANK)


def _inputs(case, seed):
    """Every input, on the GPU, from the seed alone: weights, prompts, decisions, loss inputs."""
    wl = _workload(case)
    gen = torch.Generator("cuda").manual_seed(seed * 7919 + 17)
    dt = torch.bfloat16 if wl.dtype == "bf16" else torch.float32

    def tensor(name, shape):
        gain = name.endswith("_norm") or name == "ln_gain"
        return torch.empty(shape, dtype=dt, device="cuda").normal_(1.0 if gain else 0.0, GAIN_STD if gain else STD,
                                                                   generator=gen)

    w = {key: tensor(key[-1], shape) for which, dm in ((0, wl.verifier), (1, wl.drafter))
         for key, shape in _shapes(dm, which)}
    for name, shape in _steer_shapes(wl, case["steer"]):
        w[name] = tensor(name, shape)

    def ints(lo, hi, shape):
        return torch.randint(lo, hi, shape, dtype=torch.int32, device="cuda", generator=gen)

    vocab, b, k = wl.verifier.vocab, case["batch"], case["k"]
    x = {"w": w, "wl": wl}
    if case["kind"] == "loss":
        x["tokens"], x["deltas"] = ints(0, vocab, (case["n"],)), ints(1, k + 1, (case["n"],))
        return x
    x["tokens"] = ints(0, vocab, (b, case["hi"]))
    x["lens"] = torch.tensor(_lens(case), dtype=torch.int32).cuda()
    if _forced(case):
        x["forced"] = torch.cat([ints(0, vocab, (b, k)), ints(0, min(k, 2) + 1, (b, 1)), ints(0, vocab, (b, 1))],
                                dim=1).contiguous()
    return x


class _Weights:
    """A model's device tensors as the library takes them."""

    def __init__(self, w, which, n_layers):
        names = ("attn_norm", "wq", "wk", "wv", "wo", "ffn_norm", "w_gate", "w_up", "w_down")
        ptrs = [w[(which, layer, name)].data_ptr() for layer in range(n_layers) for name in names]
        self.arr = (B.P * len(ptrs))(*ptrs)
        self.w = B.Weights(w[(which, "embed")].data_ptr(), self.arr, w[(which, "final_norm")].data_ptr(),
                           w[(which, "lm_head")].data_ptr())


def _view(eng, what):
    """The buffer a debug selector copies from, as a view of the caller's workspace."""
    want = torch.from_numpy(eng.debug(what)).cuda()
    ref, n = want.reshape(-1), want.numel()
    ws = eng.workspace[: eng.workspace.numel() // 4 * 4].view(torch.float32)
    step = 1 << 28
    for at in range(0, ws.numel() - n + 1, step):
        part = ws[at: at + step]
        for i in (part == ref[0]).nonzero()[:, 0].tolist():
            if at + i + n <= ws.numel() and torch.equal(ws[at + i: at + i + n], ref):
                return ws[at + i: at + i + n].view(want.shape)
    raise RuntimeError("the buffer is not in the workspace")


# ---- the framework's side -------------------------------------------------------------------

@functools.lru_cache(maxsize=1)
def _stream():
    """The program's stream: its generations follow each other on it."""
    return torch.cuda.Stream()


def prepare(case, seed):
    x = _inputs(case, seed)
    wl, w = x["wl"], x["w"]
    steer = case["steer"]
    cfg = B.config_of(wl, seed=seed, steering=FORMS[steer], cond_rank=RANK if steer == "cond" else 0)
    mlp = None
    if steer in ("mlp", "mlp-out", "cond"):
        mlp = {key: w[key] for key, _ in _steer_shapes(wl, steer)}
        mlp["ln_eps"] = LN_EPS
    stream = _stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        eng = B.Engine(cfg, _Weights(w, 0, wl.verifier.n_layers), _Weights(w, 1, wl.drafter.n_layers),
                       w["w_s"] if steer == "input" else None, stream=stream, mlp=mlp)
        state = {"x": x, "eng": eng, "stream": stream, "case": case}
        if case["kind"] != "loss":
            # one round on the prompts' first tokens shows where the outputs lie
            lens = torch.full((case["batch"],), 2, dtype=torch.int32, device="cuda")
            head = x["tokens"][:, :2].contiguous()
            torch.cuda.synchronize()
            eng.prefill(head, lens, 2)
            eng.round(x.get("forced"))
            views = {"logits_v": B.DBG_LOGITS_V, "logits_d": B.DBG_LOGITS_D}
            if steer != "none":
                views["steer"] = B.DBG_STEER if steer == "input" else B.DBG_UBIAS
            state["views"] = {key: _view(eng, what) for key, what in views.items()}
        if case["kind"] == "round":
            eng.prefill(x["tokens"], x["lens"], case["hi"])
    torch.cuda.synchronize()
    return state


def run(state):
    x, eng, case = state["x"], state["eng"], state["case"]
    with torch.cuda.stream(state["stream"]):
        if case["kind"] == "loss":
            loss, kl = eng.train_loss(x["tokens"], x["deltas"], case["chunk"])
            return {"loss": loss, "kl": kl}
        if case["kind"] != "round":
            eng.prefill(x["tokens"], x["lens"], case["hi"])
        if case["kind"] != "generate":
            tokens, counts = eng.round(x.get("forced"))
            return {"tokens": tokens, "counts": counts, **state["views"]}
        got = []
        for _ in range(case["rounds"]):
            tokens, counts = eng.round(x.get("forced"))
            got.append((tokens.clone(), counts.clone()))
        return {"tokens": torch.stack([a for a, _ in got]), "counts": torch.stack([a for _, a in got]),
                **state["views"]}


# ---- what a pass cannot do without ------------------------------------------------------------

def _body(dm):
    return dm.n_layers * (2 * dm.n_heads * dm.head_dim * dm.d_model + 2 * dm.n_kv_heads * dm.head_dim * dm.d_model
                          + 3 * dm.d_ff * dm.d_model)


def work(case):
    """Every weight once per forward that is a step of its own (a prompt is one step), K/V rows read
    and appended, logits written and read; two operations per weight and token."""
    wl = _workload(case)
    v, d, k = wl.verifier, wl.drafter, case["k"]
    es = 2 if wl.dtype == "bf16" else 4
    kv = [m.n_layers * m.n_kv_heads * m.head_dim * 2 * 4 for m in (v, d)]
    at = [4 * m.n_layers * m.n_heads * m.head_dim for m in (v, d)]  # operations per (query, key) pair
    params = [_body(m) for m in (v, d)]
    heads = [m.vocab * m.d_model for m in (v, d)]
    steer = sum(int(np.prod(s)) for _, s in _steer_shapes(wl, case["steer"]))
    by = fl = 0.0
    if case["kind"] == "loss":
        n = case["n"] - 1
        by = es * (sum(params) + sum(heads) + steer) + n * sum(kv) + 2 * 4.0 * n * v.vocab
        fl = 2.0 * n * (sum(params) + sum(heads) + steer) + sum(at) * n * n / 2
        return {"bytes": by, "flops": fl}
    lens = _lens(case)
    if case["kind"] != "round":
        for p in lens:
            fl += 2.0 * (p - 1) * sum(params) + sum(at) * (p - 1) ** 2 / 2
            by += (p - 1) * sum(kv)
        by += es * sum(params) + es * steer
        fl += 2.0 * len(lens) * steer
    for _ in range(case["rounds"]):
        b, ctx = len(lens), sum(lens)
        by += es * (params[0] + heads[0] + k * (params[1] + heads[1]) + steer)
        by += (ctx + b * (2 * k + 1)) * kv[0] + (k * ctx + b * (k * (k - 1) / 2 + k + 1)) * kv[1]
        by += 4.0 * b * (2 * k + 1) * v.vocab
        fl += 2.0 * b * ((k + 1) * (params[0] + heads[0]) + k * (params[1] + heads[1]) + steer)
        fl += (k + 1) * ctx * at[0] + k * ctx * at[1]
    return {"bytes": by, "flops": fl}


def tolerance(case):
    """About four times what the library is off the 64-bit result.  fp32 weights: 2.5e-7.  bf16 weights:
    the activations enter the products as a bf16 pair (16 bits): up to 8e-5 on logits over the models'
    depth.  The loss averages that over the vocabulary: 1.2e-6."""
    if case["model"] == "tiny":
        return {"rel": 1e-6, "max": 1e-5}
    return {"rel": 5e-6, "max": 1e-4} if case["kind"] == "loss" else {"rel": 3e-4, "max": 3e-3}


# ---- the same in 64 bits, plain torch ------------------------------------------------------------

class _Ref:
    """One model in float64 with a K/V cache; tokens of several sequences go through together."""

    def __init__(self, w, which, dm, batch, cap):
        self.w, self.which, self.dm = w, which, dm
        shape = (dm.n_layers, batch, dm.n_kv_heads, cap, dm.head_dim)
        self.k = torch.zeros(shape, dtype=torch.float64, device="cuda")
        self.v = torch.zeros(shape, dtype=torch.float64, device="cuda")
        half = dm.head_dim // 2
        inv = dm.rope_theta ** (-2.0 * torch.arange(half, dtype=torch.float64, device="cuda") / dm.head_dim)
        ang = torch.arange(cap, dtype=torch.float64, device="cuda")[:, None] * inv
        self.cos, self.sin = ang.cos(), ang.sin()

    def norm(self, x, name):
        key = (self.which, name) if isinstance(name, str) else (self.which, *name)
        return x * torch.rsqrt((x * x).mean(-1, keepdim=True) + self.dm.rms_eps) * self.w[key].double()

    def mat(self, x, key):
        return x @ self.w[(self.which, *key)].double().T

    def rope(self, x, pos):
        half = self.dm.head_dim // 2
        c, s = self.cos[pos][:, None, :], self.sin[pos][:, None, :]
        a, b = x[..., :half], x[..., half:]
        return torch.cat([a * c - b * s, b * c + a * s], dim=-1)

    def forward(self, rows, add=None, up=None, out=None, taps=None):
        """rows: (sequence, first position, tokens) triples.  add: [rows][d] joins the embeddings;
        up(layer, x) joins the up projection; out joins every MLP's output; taps: layers whose
        residual is kept.  Returns the final residual, or (residual, {layer: residual})."""
        dm, hd, g = self.dm, self.dm.head_dim, self.dm.n_heads // self.dm.n_kv_heads
        tok = torch.cat([torch.as_tensor(r[2], device="cuda").long() for r in rows])
        pos = torch.cat([torch.arange(r[1], r[1] + len(r[2]), device="cuda") for r in rows])
        x = self.w[(self.which, "embed")][tok].double()
        if add is not None:
            x = x + add
        kept = {}
        for layer in range(dm.n_layers):
            bias = up(layer, x) if up else None
            a = self.norm(x, (layer, "attn_norm"))
            q = self.rope(self.mat(a, (layer, "wq")).view(-1, dm.n_heads, hd), pos)
            kk = self.rope(self.mat(a, (layer, "wk")).view(-1, dm.n_kv_heads, hd), pos)
            vv = self.mat(a, (layer, "wv")).view(-1, dm.n_kv_heads, hd)
            o, at = torch.empty_like(q), 0
            for b, p0, t in rows:
                n = len(t)
                self.k[layer, b, :, p0: p0 + n] = kk[at: at + n].transpose(0, 1)
                self.v[layer, b, :, p0: p0 + n] = vv[at: at + n].transpose(0, 1)
                ks, vs = self.k[layer, b, :, : p0 + n], self.v[layer, b, :, : p0 + n]
                for i in range(0, n, 1024):
                    m = min(1024, n - i)
                    qs = q[at + i: at + i + m].view(m, dm.n_kv_heads, g, hd).permute(1, 2, 0, 3)
                    s = torch.matmul(qs.reshape(dm.n_kv_heads, g * m, hd), ks.transpose(1, 2).contiguous())
                    s = s.view(dm.n_kv_heads, g, m, p0 + n) / math.sqrt(hd)
                    future = torch.arange(p0 + n, device="cuda")[None, :] > pos[at + i: at + i + m, None]
                    p = torch.softmax(s.masked_fill_(future, -math.inf), dim=-1)
                    r = torch.matmul(p.view(dm.n_kv_heads, g * m, p0 + n), vs.contiguous())
                    o[at + i: at + i + m] = r.view(dm.n_heads, m, hd).transpose(0, 1)
                    del s, p
                at += n
            x = x + self.mat(o.reshape(-1, dm.n_heads * hd), (layer, "wo"))
            a = self.norm(x, (layer, "ffn_norm"))
            u = self.mat(a, (layer, "w_up"))
            if bias is not None:
                u = u + bias
            x = x + self.mat(torch.nn.functional.silu(self.mat(a, (layer, "w_gate"))) * u, (layer, "w_down"))
            if out is not None:
                x = x + out
            if taps and layer in taps:
                kept[layer] = x
        return (x, kept) if taps else x

    def logits(self, x):
        return self.mat(self.norm(x, "final_norm"), ("lm_head",))


def _philox(c0, c1, c2, c3, seed):
    """Philox4x32-10 (Salmon et al., SC'11) on int64 tensors of 32-bit words."""
    mask = 0xFFFFFFFF
    x = [c0 & mask] + [torch.full_like(c0, c & mask) for c in (c1, c2, c3)]
    k0, k1 = seed & mask, (seed >> 32) & mask

    def mul(a, b):  # high and low word of a 32-bit product
        lo, hi = (b & 0xFFFF) * a, (b >> 16) * a
        return (hi + (lo >> 16)) >> 16, (lo + ((hi & 0xFFFF) << 16)) & mask

    for _ in range(10):
        ah, al = mul(0xD2511F53, x[0])
        bh, bl = mul(0xCD9E8D57, x[2])
        x = [bh ^ x[1] ^ k0, bl, ah ^ x[3] ^ k1, al]
        k0, k1 = (k0 + 0x9E3779B9) & mask, (k1 + 0xBB67AE85) & mask
    return x


def _uniform(w):
    return ((w >> 9).double() + 0.5) / 8388608.0


def _gumbel(vocab, step, t, purpose, b, seed):
    q = torch.arange((vocab + 3) // 4, device="cuda")
    w = torch.stack(_philox(q, step, t, (purpose << 24) | b, seed), dim=1).reshape(-1)[:vocab]
    return -torch.log(-torch.log(_uniform(w)))


def _exact_round(case, seed, ref, seqs, forced, bias):
    """One round of every sequence; `seqs` are dicts with t, len_d and hist.  `bias`: the steering
    of each sequence.  Returns the verifier's and the drafter's logits and the new steering rows'
    residuals (final, taps)."""
    ver, dr = ref
    k, temp, vocab = case["k"], case["t"], ver.dm.vocab
    nb = len(seqs)
    drafts = [[] for _ in seqs]
    ld = torch.empty((nb, k, vocab), dtype=torch.float64, device="cuda")
    for j in range(1, k + 1):
        rows = []
        for b, s in enumerate(seqs):
            p0 = s["len_d"] if j == 1 else s["t"] + j - 2
            rows.append((b, p0, s["hist"][p0: s["t"]] if j == 1 else [drafts[b][-1]]))
        who = torch.tensor([b for b, _, t in rows for _ in t], device="cuda")
        kw = bias(who)
        last = torch.cumsum(torch.tensor([len(r[2]) for r in rows], device="cuda"), 0) - 1
        ld[:, j - 1] = dr.logits(dr.forward(rows, **kw)[last])
        for b, s in enumerate(seqs):
            if forced is not None:
                drafts[b].append(int(forced[b][j - 1]))
            elif temp > 0:
                drafts[b].append(int((ld[b, j - 1] / temp + _gumbel(vocab, j, s["t"], 1, b, seed)).argmax()))
            else:
                drafts[b].append(int(ld[b, j - 1].argmax()))
    tl = sorted({ver.dm.n_layers - 3, ver.dm.n_layers // 2 - 1, 2})
    rows = [(b, s["t"] - 1, [s["hist"][s["t"] - 1]] + drafts[b]) for b, s in enumerate(seqs)]
    x, kept = ver.forward(rows, taps=tl if ver.dm.n_layers >= 3 else [0])
    lv = ver.logits(x).view(nb, k + 1, vocab)
    at = []
    for b, s in enumerate(seqs):
        if forced is not None:
            n, y = int(forced[b][k]), int(forced[b][k + 1])
        elif temp > 0:
            lp, lq = torch.log_softmax(lv[b] / temp, -1), torch.log_softmax(ld[b] / temp, -1)
            n = 0
            while n < k:
                w = _philox(torch.tensor([n], device="cuda"), 0, s["t"], (2 << 24) | b, seed)[0]
                if not float(torch.log(_uniform(w))) < float(lp[n, drafts[b][n]] - lq[n, drafts[b][n]]):
                    break
                n += 1
            g = _gumbel(vocab, 0, s["t"], 3, b, seed)
            r = (lp[n].exp() - lq[n].exp()).clamp_min(0) if n < k else None
            y = int(((r.log() if r is not None and float(r.max()) > 0 else lv[b, n] / temp) + g).argmax())
        else:
            best = lv[b].argmax(-1).tolist()
            n = next((i for i in range(k) if best[i] != drafts[b][i]), k)
            y = best[n]
        s["hist"] = s["hist"][: s["t"]] + drafts[b][:n] + [y]
        s["len_d"] = min(s["t"] + k - 1, s["t"] + n)
        s["t"] += n + 1
        at.append(b * (k + 1) + n)
    return lv, ld, x[at], {layer: r[at] for layer, r in kept.items()}


@torch.no_grad()
def exact(case, seed):
    x = _inputs(case, seed)
    w, wl, steer = x["w"], x["wl"], case["steer"]
    v, d = wl.verifier, wl.drafter
    loss = case["kind"] == "loss"
    cap = case["n"] if loss else case["hi"] + case["rounds"] * (case["k"] + 1) + 1
    ver, dr = _Ref(w, 0, v, case["batch"], cap), _Ref(w, 1, d, case["batch"], cap)
    if loss:
        n, tok, delta = case["n"], x["tokens"], x["deltas"].long()
        hv = ver.forward([(0, 0, tok[: n - 1])])
        src = torch.arange(n - 1, device="cuda") - delta[1:]
        s = (ver.norm(hv, "final_norm") @ w["w_s"].double().T)[src.clamp_min(0)] * (src >= 0)[:, None]
        hd = dr.forward([(0, 0, tok[: n - 1])], add=s)
        kl = torch.zeros(n, dtype=torch.float64, device="cuda")
        for i in range(0, n - 1, 256):
            lp, lq = torch.log_softmax(ver.logits(hv[i: i + 256]), -1), torch.log_softmax(dr.logits(hd[i: i + 256]), -1)
            kl[1 + i: 1 + i + lp.shape[0]] = (lp.exp() * (lp - lq)).sum(-1)
        return {"loss": float(kl[1:].mean()), "kl": kl}

    def steering(final, kept, live):
        """The steering rows of each sequence from the verifier's residual rows."""
        if steer == "none":
            return None
        if steer == "input":
            r = ver.norm(final, "final_norm")
        else:
            z = torch.cat([kept[i] for i in (v.n_layers - 3, v.n_layers // 2 - 1, 2)], dim=1)
            r = torch.nn.functional.layer_norm(z @ w["w_hml"].double().T, (v.d_model,), w["ln_gain"].double(),
                                               w["ln_bias"].double(), LN_EPS)
        return (r @ w["w_s"].double().T) * live

    def joined(s):
        """How the steering rows `s` enter the drafter's forward, for rows of the sequences `who`."""
        if steer == "none":
            return lambda who: {}
        if steer == "input":
            return lambda who: {"add": s[who]}
        if steer == "mlp":
            return lambda who: {"up": lambda layer, _: s[who, layer * d.d_ff: (layer + 1) * d.d_ff]}
        if steer == "mlp-out":
            return lambda who: {"out": s[who]}

        def cond(who):
            def up(layer, f):
                h = f @ w["w_cf"][layer * RANK: (layer + 1) * RANK].double().T
                h = torch.nn.functional.silu(h + s[who, layer * RANK: (layer + 1) * RANK])
                return h @ w["w_cu"][layer * d.d_ff: (layer + 1) * d.d_ff].double().T
            return {"up": up}
        return cond

    lens, nb = _lens(case), case["batch"]
    toks = x["tokens"].tolist()
    seqs = [{"t": p, "len_d": p - 1, "hist": toks[b][:p]} for b, p in enumerate(lens)]
    live = torch.tensor([[float(p > 1)] for p in lens], dtype=torch.float64, device="cuda")
    s = None
    tl = sorted({v.n_layers - 3, v.n_layers // 2 - 1, 2}) if v.n_layers >= 3 else [0]
    rows = [(b, 0, toks[b][: p - 1]) for b, p in enumerate(lens) if p > 1]
    final = torch.zeros((nb, v.d_model), dtype=torch.float64, device="cuda")
    kept = {layer: torch.zeros_like(final) for layer in tl}
    if rows:
        h, hk = ver.forward(rows, taps=tl)
        at = (torch.cumsum(torch.tensor([len(r[2]) for r in rows]), 0) - 1).cuda()
        who = torch.tensor([r[0] for r in rows], device="cuda")
        final[who] = h[at]
        for layer in tl:
            kept[layer][who] = hk[layer][at]
        del h, hk
        dr.forward(rows)
    s = steering(final, kept, live)
    forced = x["forced"].tolist() if "forced" in x else None
    for _ in range(case["rounds"]):
        lv, ld, final, kept = _exact_round(case, seed, (ver, dr), seqs, forced, joined(s))
        s = steering(final, kept, 1.0)
    got = {"tokens": None, "counts": None, "logits_v": lv, "logits_d": ld}
    if steer == "mlp":
        got["steer"] = s.view(nb, d.n_layers, d.d_ff)
    elif steer == "cond":
        got["steer"] = s.view(nb, d.n_layers, RANK)
    elif steer != "none":
        got["steer"] = s
    return got
