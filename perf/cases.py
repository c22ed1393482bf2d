"""Timed cases of the speculative-decoding library: what a serving program has it do.

Every case builds one model from seeded weights through the C ABI binding and makes one
of three calls per pass:

  "round"    one speculative round of a running session (prefilled and one round old, so
             that the rejected-trajectory conditioning is active);
  "request"  a new request: prefill of the prompts, then `rounds` speculative rounds;
  "steps"    `rounds` target-only decoding steps, the baseline speculation is compared to.

Shapes are the repository's workload presets.  Weights follow the usual initialisation of
deep decoders: unit-variance embeddings, projections N(0, 0.02), the projections that
write the residual stream scaled down by 1 / sqrt(2 layers).  The vocabulary matrix is the
embedding moved by one row and scaled, so that the model predicts its input token's
successor with a clear margin, as a trained model's predictions are peaked: tokens are
then decided by the model and not by the rounding of near-ties.

Beside the tokens a pass returns the final hidden states of the drafter and of the target
(the vocabulary projection's inputs), which the library retains in the caller's workspace;
a request returns the last layers' key caches as well, and with sampling, where the logits
are stored, a pass returns those too.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2608_29748_amd import binding as B
from paper_2608_29748_amd.engine import config_from
from workloads import PRESETS, cond_layer_ids

DEVICE = "cuda:0"
EPS, THETA = 1e-6, 1e6


# ------------------------------------------------------------------ the cases

def _case(name, kind, preset, batch, ctx, layers=None, draft=None, rounds=1, budget=1024, block=16,
          temperature=0.0, cond="retrace"):
    wl = PRESETS[preset]
    c = dict(kind=kind, preset=preset, batch=batch, ctx_lo=ctx[0], ctx_hi=ctx[1],
             layers=layers or wl.target.n_layers, draft=draft or wl.draft_layers, rounds=rounds,
             budget=budget, block=block, temperature=temperature, cond=cond)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest call: a whole short request on the tiny fp32 model, where launches
        # and host work count
        _case("tiny-f32 request", "request", "tiny-f32", 1, (64, 64), rounds=16, budget=24, block=8),
        # a small model's session at batch 1: launch latency against a 1.2 GB weight stream
        _case("0.6b round", "round", "qwen3-0.6b-shape", 1, (512, 512)),
        # target-only decoding with sampling (temperature 1, top-k 20, top-p 0.95)
        _case("0.6b steps sampled", "steps", "qwen3-0.6b-shape", 1, (512, 512), rounds=16, budget=8192,
              temperature=1.0),
        # the headline: one round of a single 4B session at a 4096-token context
        _case("4b round", "round", "qwen3-4b-shape", 1, (4096, 4096)),
        # its prompt: time to the first committed block of a 4096-token request
        _case("4b prompt", "request", "qwen3-4b-shape", 1, (4096, 4096), rounds=1, budget=64),
        # concurrent serving of short prompts: sampled rounds of eight sequences ...
        _case("4b serve b8 sampled", "round", "qwen3-4b-serve", 8, (96, 320), temperature=1.0),
        # ... greedy rounds of thirty-two ...
        _case("4b serve b32", "round", "qwen3-4b-serve", 32, (96, 320), budget=512),
        # ... and the admission of sixteen new prompts
        _case("4b admit b16", "request", "qwen3-4b-serve", 16, (96, 320), rounds=1, budget=64),
        # three ragged sequences (48 rows) with the low-rank conditioning path; a third of
        # the depth
        _case("4b b3 lowrank", "round", "qwen3-4b-serve", 3, (701, 3037), layers=12, draft=2, cond="lowrank"),
        # wide models in ragged batches at a third and a quarter of their depth
        _case("8b b8 round", "round", "qwen3-8b-shape-b8", 8, (1031, 8192), layers=12, draft=2, budget=512),
        _case("14b b16 round", "round", "qwen3-14b-shape-b16", 16, (8192, 16384), layers=10, draft=2, budget=256),
        # odd widths (17 and 33 k tiles) and ragged short prompts, a whole request
        _case("odd b10 request", "request", "mini-bf16-odd", 10, (21, 79), rounds=4, budget=16),
    ]


def draw(rng):
    def logint(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    kind = rng.choice(["round", "round", "round", "request", "request", "steps"])
    preset = rng.choice(["tiny-f32", "qwen3-0.6b-shape", "qwen3-4b-shape", "qwen3-4b-serve", "qwen3-8b-shape-b8",
                         "qwen3-14b-shape-b16", "mini-bf16-odd", "mini-bf16-w4096"])
    batch = logint(1, 32)
    small = preset.startswith(("tiny", "mini"))
    hi = logint(24, min(4096 if not small else 700, max(64, 24576 // batch)))
    lo = rng.randint(max(1, hi // 4), hi)
    block = 8 if preset == "tiny-f32" else rng.choice([16, 16, 16, 8, rng.randint(3, 16)])
    layers = 2 if small else rng.randint(3, 8)
    sampled = not small and rng.random() < 0.25
    return _case(None, kind, preset, batch, (lo, hi), layers=layers, draft=1 if small else rng.randint(1, 3),
                 rounds={"round": 1, "request": rng.randint(1, 6), "steps": logint(1, 24)}[kind],
                 budget={"round": 768, "request": 128, "steps": 4096}[kind], block=block,
                 temperature=1.0 if sampled or kind == "steps" and not small else 0.0,
                 cond=rng.choice(["retrace", "retrace", "lowrank", "raw_gated", "off"]))


# ------------------------------------------------------------------ the model of a case

def _dims(case):
    t = PRESETS[case["preset"]].target
    L = case["layers"]
    ids = cond_layer_ids(L, 5) if L >= 7 else tuple(range(min(L, 3)))
    f32 = PRESETS[case["preset"]].dtype == "f32"
    return t, L, case["draft"], ids, f32


def _lengths(case):
    """Prompt lengths: spread over the range, the same for every seed."""
    lo, hi, n = case["ctx_lo"], case["ctx_hi"], case["batch"]
    return [lo + int((hi - lo) * ((0.5 + 0.6180339887 * i) % 1.0)) for i in range(n)]


def _prompts(case, seed):
    g = np.random.Generator(np.random.PCG64([int(seed), 11]))
    V = PRESETS[case["preset"]].target.vocab
    return [g.integers(0, V - 2048 if V > 4096 else V // 2, size=n).astype(np.int32) for n in _lengths(case)]


def _weights(case, seed):
    """The model's tensors in the canonical order of rt_init_models, on the GPU."""
    t, L, LD, ids, f32 = _dims(case)
    d, q, kv, F = t.hidden, t.n_q_heads * t.head_dim, t.n_kv_heads * t.head_dim, t.ffn
    g = torch.Generator(device=DEVICE)
    g.manual_seed(int(seed))
    dt = torch.float32 if f32 else torch.bfloat16

    def mat(n, k, std=0.02):
        return torch.empty((n, k), dtype=dt, device=DEVICE).normal_(0.0, std, generator=g)

    def norm(n):
        return (1.0 + 0.1 * torch.empty(n, device=DEVICE).normal_(generator=g)).to(dt)

    def layer(depth):
        out = 0.02 / math.sqrt(2.0 * depth)
        return [norm(d), mat(q, d), mat(kv, d), mat(kv, d), norm(t.head_dim), norm(t.head_dim), mat(d, q, out),
                norm(d), mat(F, d), mat(F, d), mat(d, F, out)]

    embed = mat(t.vocab, d, 1.0)
    w = [embed]
    for _ in range(L):
        w += layer(L)
    w += [norm(d), embed.roll(1, 0) * 0.02, mat(d, len(ids) * d), norm(d)]
    for _ in range(LD):
        w += layer(LD)
    w += [norm(d), mat(d, 2 * d), mat(d, d), mat(d, 2 * d)]
    if case["cond"] == "lowrank":
        w += [mat(64, d), mat(32, 2 * d), mat(64, 32, 0.1), mat(d, 64, 0.1), mat(d, 64, 0.1)]
    return w


class _Session:
    """A model handle with its workspace, as a serving program holds it."""

    def __init__(self, case, seed):
        t, L, LD, ids, f32 = _dims(case)
        self.case, self.n, self.bk = case, case["batch"], case["block"]
        self.prompts = _prompts(case, seed)
        self.row = t.n_kv_heads * t.head_dim * (4 if f32 else 2)   # bytes of one position's keys
        self.cfg = config_from(
            _Shape(t, L), dtype="f32" if f32 else "bf16", draft_layers=LD, cond_layers=ids, block_size=self.bk,
            mask_token_id=t.vocab - 1, max_batch=self.n,
            max_seq_len=max(len(p) for p in self.prompts) + case["budget"] + self.bk,
            cond_mode=B.COND_MODES[case["cond"]], temperature=case["temperature"], sample_seed=int(seed))
        w = _weights(case, seed)
        size = B.rt_workspace_bytes(self.cfg)
        self.ws = torch.empty(size + 256, dtype=torch.uint8, device=DEVICE)
        self.off = -self.ws.data_ptr() % 256
        self.stream = torch.cuda.Stream(device=DEVICE)
        torch.cuda.synchronize()
        self.h = B.rt_init_models(self.cfg, [x.data_ptr() for x in w], self.ws.data_ptr() + self.off, size,
                                  self.stream.cuda_stream)
        del w
        self._find_outputs(t, f32)

    def _find_outputs(self, t, f32):
        """Views of the results that the library keeps in the caller's workspace: their
        place is found from what the read hook says after one call on one-token prompts."""
        case, n, bk = self.case, self.n, self.bk
        B.rt_prefill(self.h, [p[:1] for p in self.prompts], 8)
        self.views = {}
        keep = torch.float32 if f32 else torch.float16
        if case["kind"] == "steps":
            B.rt_ar_steps(self.h, n, 1)
            if case["temperature"] > 0:
                self.views["logits"] = self._view(B.RT_T_AR_LOGITS, torch.float32, (n, t.vocab))
            return
        B.rt_spec_round(self.h, n, bk)
        self.views["h_draft"] = self._view(B.RT_T_HD, keep, (n, bk, t.hidden))
        self.views["h_target"] = self._view(B.RT_T_HT, keep, (n, bk, t.hidden))
        if case["kind"] == "request":   # the last layers' key caches, which the prompts fill
            pages = n * ((self.cfg.max_seq_len + 15) // 16)
            kv = (pages, t.n_kv_heads, 16, t.head_dim)
            store = torch.float32 if f32 else torch.bfloat16
            self.views["k_target"] = self._view(B.RT_T_TARGET_K + case["layers"] - 1, store, kv)
            self.views["k_draft"] = self._view(B.RT_T_DRAFT_K + case["draft"] - 1, store, kv)
        if case["temperature"] > 0:
            self.views["logits"] = self._view(B.RT_T_VERIFY_LOGITS, torch.float32, (n, bk, t.vocab))

    def _view(self, tensor_id, dtype, shape):
        # (a key row of one position is contiguous for one head only: 128 bytes at least)
        raw = bytearray(B.rt_debug_read(self.h, tensor_id, 0, self.row))[:128]
        want = torch.frombuffer(raw, dtype=torch.int64).to(DEVICE)
        body = self.ws[self.off: self.off + (self.ws.numel() - self.off) // 8 * 8].view(torch.int64)
        step = 1 << 28
        for lo in range(0, body.numel(), step):
            for i in (body[lo:lo + step] == want[0]).nonzero().flatten().tolist():
                if torch.equal(body[lo + i: lo + i + want.numel()], want):
                    at = self.off + 8 * (lo + i)
                    size = math.prod(shape) * torch.empty((), dtype=dtype).element_size()
                    return self.ws[at: at + size].view(dtype).view(shape)
        raise RuntimeError(f"tensor {tensor_id} was not found in the workspace")

    def __del__(self):
        if getattr(self, "h", None):
            B.rt_destroy(self.h)
            self.h = None


class _Shape:
    """A preset's model shape at the case's depth."""

    def __init__(self, t, layers):
        self.vocab, self.hidden, self.n_layers = t.vocab, t.hidden, layers
        self.n_q_heads, self.n_kv_heads, self.head_dim, self.ffn = t.n_q_heads, t.n_kv_heads, t.head_dim, t.ffn


def prepare(case, seed):
    s = _Session(case, seed)
    if case["kind"] != "request":
        B.rt_prefill(s.h, s.prompts, case["budget"])
        if case["kind"] == "round":
            B.rt_spec_round(s.h, s.n, s.bk)
        else:
            B.rt_ar_steps(s.h, s.n, 1)
    return s


def run(s):
    case = s.case
    if case["kind"] == "round":
        tok, n, a = B.rt_spec_round(s.h, s.n, s.bk)
        return dict(s.views, tokens=tok, n_committed=n, accept_len=a)
    if case["kind"] == "steps":
        tok, n = B.rt_ar_steps(s.h, s.n, case["rounds"])
        return dict(s.views, tokens=tok, n_committed=n)
    first = B.rt_prefill(s.h, s.prompts, case["budget"])
    got = [B.rt_spec_round(s.h, s.n, s.bk) for _ in range(case["rounds"])]
    return dict(s.views, first=first, tokens=np.stack([g[0] for g in got]), n_committed=np.stack([g[1] for g in got]),
                accept_len=np.stack([g[2] for g in got]))


# ------------------------------------------------------------------ work and tolerance

def _parts(case):
    """(bytes, flops) of the prefill, of one round and of one target-only step."""
    t, L, LD, ids, f32 = _dims(case)
    e = 4 if f32 else 2
    d, q, kv = t.hidden, t.n_q_heads * t.head_dim, t.n_kv_heads * t.head_dim
    layer = (q + 2 * kv) * d + q * d + 3 * t.ffn * d
    head, ctx = t.vocab * d, len(ids) * d * d + LD * 2 * kv * d
    cond = {"retrace": 5 * d * d, "raw_gated": 3 * d * d, "lowrank": 64 * d * 5, "off": 0}[case["cond"]]
    lens, n, bk = _lengths(case), case["batch"], case["block"]
    rows, tokens, keys = n * bk, sum(lens), sum(lens) + n * bk
    pre = (e * (L * layer + head + ctx) + e * tokens * 2 * kv * (L + LD),
           2.0 * tokens * (L * layer + ctx) + 2.0 * n * head + sum(2.0 * x * x * q * L for x in lens))
    rnd = (e * ((L + LD) * layer + 2 * head + ctx + cond) + e * keys * 2 * kv * (L + LD),
           2.0 * rows * ((L + LD) * layer + 2 * head + ctx + cond) + 4.0 * keys * bk * q * (L + LD))
    step = (e * (L * layer + head) + e * sum(lens) * 2 * kv * L,
            2.0 * n * (L * layer + head) + 4.0 * sum(lens) * q * L)
    return pre, rnd, step


def work(case):
    pre, rnd, step = _parts(case)
    k = case["rounds"]
    b, f = {"round": rnd, "steps": (k * step[0], k * step[1]),
            "request": (pre[0] + k * rnd[0], pre[1] + k * rnd[1])}[case["kind"]]
    return {"bytes": b, "flops": f}


def tolerance(case):
    if _dims(case)[4]:
        return {"rel": 2e-6, "max": 2e-5}      # measured against 64 bits: 8e-8
    # measured against 64 bits: up to 3e-3 at 41 layers and 7e-3 at the widest shapes
    return {"rel": 1.5e-2, "max": 0.2}


# ------------------------------------------------------------------ 64-bit reference

def exact(case, seed):
    pre, rnd, step = _parts(case)
    if pre[1] + 3 * rnd[1] > 3e14:      # beyond about 20 seconds in 64 bits
        return None
    if case["kind"] == "steps" and case["temperature"] == 0:
        return None
    r = _Reference(case, _weights(case, seed))
    seqs = [r.prefill(p) for p in _prompts(case, seed)]
    if case["kind"] == "steps":
        got = [[r.step(s) for _ in range(1 + case["rounds"])][1:] for s in seqs]
        return dict(logits=torch.stack([g[-1][1] for g in got]), tokens=np.array([[x[0] for x in g] for g in got]),
                    n_committed=None)
    first = np.array([s["anchor"] for s in seqs])
    rounds = 2 if case["kind"] == "round" else case["rounds"]
    got = [[r.round(s) for _ in range(rounds)] for s in seqs]
    out = dict(h_draft=torch.stack([g[-1]["hd"] for g in got]), h_target=torch.stack([g[-1]["ht"] for g in got]))
    if case["temperature"] > 0:
        out["logits"] = torch.stack([r.logits(g[-1]["ht"]) for g in got])
    toks = np.array([[g[k]["tokens"] for g in got] for k in range(rounds)])
    if case["kind"] == "round":
        return dict(out, tokens=toks[-1], n_committed=None, accept_len=None)
    return dict(out, k_target=None, k_draft=None, first=first, tokens=toks, n_committed=None, accept_len=None)


class _Reference:
    """The model in float64: prefill, rounds and steps of one sequence.  Sampled cases
    take the argmax, which is all that top-p leaves of their peaked distributions."""

    def __init__(self, case, w):
        self.case = case
        self.t, self.L, self.LD, self.ids, _ = _dims(case)
        L, LD = self.L, self.LD
        self.embed, self.tl = w[0], [w[1 + 11 * i: 12 + 11 * i] for i in range(L)]
        b = 1 + 11 * L
        self.t_norm, self.head, self.fc, self.h_norm = w[b:b + 4]
        b += 4
        self.dl = [w[b + 11 * i: b + 11 + 11 * i] for i in range(LD)]
        b += 11 * LD
        self.d_norm, self.w_c, self.w_v, self.w_g = w[b:b + 4]
        self.lowrank = w[b + 4:]

    @staticmethod
    def lin(x, w):
        """x W^T, the weight widened in parts."""
        out = torch.empty((x.shape[0], w.shape[0]), dtype=torch.float64, device=DEVICE)
        for lo in range(0, w.shape[0], 32768):
            out[:, lo:lo + 32768] = x @ w[lo:lo + 32768].double().t()
        return out

    @staticmethod
    def rms(x, w):
        return x / torch.sqrt(x.square().mean(-1, keepdim=True) + EPS) * w.double()

    def rope(self, x, pos):
        half = x.shape[-1] // 2
        i = torch.arange(half, dtype=torch.float64, device=DEVICE)
        inv = (THETA ** (-2.0 * i / (2 * half))).float().double()
        ang = (pos.double()[:, None] * inv).float().double()[:, None, :]
        a, b = x[..., :half], x[..., half:]
        return torch.cat([a * ang.cos() - b * ang.sin(), b * ang.cos() + a * ang.sin()], -1)

    def kv(self, h, lw, pos):
        t = self.t
        k = self.lin(h, lw[2]).view(-1, t.n_kv_heads, t.head_dim)
        return self.rope(self.rms(k, lw[5]), pos), self.lin(h, lw[3]).view(-1, t.n_kv_heads, t.head_dim)

    def layer(self, x, lw, pos, keys, vals, causal):
        """One decoder layer on rows x at positions pos over the cached keys / vals and its own."""
        t = self.t
        h = self.rms(x, lw[0])
        q = self.rope(self.rms(self.lin(h, lw[1]).view(-1, t.n_q_heads, t.head_dim), lw[4]), pos)
        k, v = self.kv(h, lw, pos)
        k, v = torch.cat([keys, k]), torch.cat([vals, v])
        G, out = t.n_q_heads // t.n_kv_heads, []
        kt, vt = k.permute(1, 2, 0).contiguous(), v.permute(1, 0, 2).contiguous()
        kpos = torch.arange(k.shape[0], device=DEVICE)
        for lo in range(0, x.shape[0], 512):
            qq = q[lo:lo + 512]
            n = qq.shape[0]
            s = torch.bmm(qq.view(n, t.n_kv_heads, G, -1).permute(1, 2, 0, 3).reshape(t.n_kv_heads, G * n, -1), kt)
            s = s.view(t.n_kv_heads, G, n, -1) / math.sqrt(t.head_dim)
            if causal:
                s = s.masked_fill(kpos[None, :] > pos[lo:lo + 512, None], -math.inf)
            o = torch.bmm(torch.softmax(s, -1).view(t.n_kv_heads, G * n, -1), vt)
            out.append(o.view(t.n_kv_heads, G, n, -1).permute(2, 0, 1, 3).reshape(n, -1))
        x = x + self.lin(torch.cat(out), lw[6])
        h = self.rms(x, lw[7])
        return x + self.lin(torch.nn.functional.silu(self.lin(h, lw[8])) * self.lin(h, lw[9]), lw[10]), k, v

    def target(self, s, tokens, pos0):
        """Rows `tokens` from pos0 on: final states, captured states; the K / V are kept."""
        x = self.embed[torch.as_tensor(tokens, device=DEVICE, dtype=torch.long)].double()
        pos, g = pos0 + torch.arange(len(tokens), device=DEVICE), []
        for l, lw in enumerate(self.tl):
            x, s["k"][l], s["v"][l] = self.layer(x, lw, pos, s["k"][l][:pos0], s["v"][l][:pos0], True)
            if l in self.ids:
                g.append(x)
        return self.rms(x, self.t_norm), torch.cat(g, -1)

    def logits(self, h):
        return self.lin(h, self.head)

    def append(self, s, g, pos0):
        f = self.rms(self.lin(g, self.fc), self.h_norm)
        pos = pos0 + torch.arange(g.shape[0], device=DEVICE)
        for l, lw in enumerate(self.dl):
            k, v = self.kv(f, lw, pos)
            s["ck"][l], s["cv"][l] = torch.cat([s["ck"][l][:pos0], k]), torch.cat([s["cv"][l][:pos0], v])

    def prefill(self, prompt):
        z = torch.zeros((0, self.t.n_kv_heads, self.t.head_dim), dtype=torch.float64, device=DEVICE)
        s = dict(k=[z] * self.L, v=[z] * self.L, ck=[z] * self.LD, cv=[z] * self.LD, P=len(prompt), cond=0)
        h, g = self.target(s, prompt, 0)
        if self.case["kind"] != "steps":
            self.append(s, g, 0)
        s["anchor"] = int(self.logits(h[-1:]).argmax())
        return s

    def step(self, s):
        h, _ = self.target(s, [s["anchor"]], s["P"])
        y = self.logits(h)[0]
        s["anchor"], s["P"] = int(y.argmax()), s["P"] + 1
        return s["anchor"], y

    def conditioned(self, s, e):
        """The block's inputs: rows 1..cond take the previous round's rejected suffix in."""
        n, r, mode = s["cond"], s.get("r", 0), self.case["cond"]
        if n == 0 or mode == "off":
            return e
        m, u, em, d = s["hd"][r + 1:r + 1 + n], s["ht"][r:r + n], e[1:1 + n], e.shape[1]
        if mode == "lowrank":
            a, down, up, V, G = self.lowrank
            rho = self.lin(m, a) + self.lin(self.lin(torch.cat([m, u], -1), down), up)
            add = self.lin(rho, V) * torch.sigmoid(self.lin(em, self.w_g[:, :d]) + self.lin(rho, G))
        else:
            rr = m if mode == "raw_gated" else m + self.lin(torch.cat([m, u], -1), self.w_c)
            add = self.lin(rr, self.w_v) * torch.sigmoid(self.lin(torch.cat([em, rr], -1), self.w_g))
        return torch.cat([e[:1], em + add, e[1 + n:]])

    def round(self, s):
        bk, P, mask = self.case["block"], s["P"], self.t.vocab - 1
        Bn = bk - 1
        pos = P + torch.arange(bk, device=DEVICE)
        x = self.conditioned(s, self.embed[torch.tensor([s["anchor"]] + [mask] * Bn, device=DEVICE)].double())
        for l, lw in enumerate(self.dl):
            x, _, _ = self.layer(x, lw, pos, s["ck"][l][:P], s["cv"][l][:P], False)
        hd = self.rms(x, self.d_norm)
        drafts = self.logits(hd)[1:].argmax(-1).tolist()
        ht, g = self.target(s, [s["anchor"]] + drafts, P)
        y = self.logits(ht).argmax(-1).tolist()
        A = next((i for i in range(Bn) if drafts[i] != y[i]), Bn)
        self.append(s, g[:A + 1], P)
        s["P"], s["anchor"] = P + A + 1, y[A]
        s["hd"], s["ht"], s["r"], s["cond"] = hd, ht, A + 1, Bn - A - 1 if A < Bn - 1 else 0
        return dict(hd=hd, ht=ht, tokens=drafts[:A] + [y[A]] + [-1] * (Bn - A))
