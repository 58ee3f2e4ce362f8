"""The work a user of the library has it do, as cases that can be timed and checked.

Every case goes through the public binding (paper_2606_31580_amd.laser).  A pass is one call
of a serving loop:

  decode   one greedy decode step of a batch over its paged KV cache (laser_decode_step);
  probe    the trial-answer confidence probe at an action transition point
           (laser_probe_confidence);
  mixed    a decode step in which half of the batch also runs its probe (laser_step_mixed);
  prefill  a prompt, or the forced conclusion's tokens after a long chain of thought
           (laser_prefill);
  import   a request's dense K/V moved into the paged pools (laser_kv_import);
  export   the inverse (laser_kv_export).

Shapes are the model shapes of configs.py; most cases keep a few of their layers (`layers`),
so that a pass is those decoder blocks and the LM head, and three cases run a whole model.
Weights, norm gains, tokens and K/V are random from the seed; the final norm's gain of 8 gives
the peaked token distributions that a confidence probe is made for.
"""
from __future__ import annotations

import math
from dataclasses import replace

import torch

from paper_2606_31580_amd import laser as L
from paper_2606_31580_amd import synth
from paper_2606_31580_amd.configs import SHAPES

DEV = "cuda"
SUFFIX, TRIALS = 8, 4      # the benchmark's answer-inducing suffix and trial-answer lengths
FINAL_GAIN = 8.0
RESET_EVERY = 64           # decode steps after which the requests start over at their length

TINY, Q15, Q7, L8 = "tiny-2L-d256", "qwen2-1.5B-shape", "qwen2-7B-shape", "llama-8B-shape"


def listed():
    return [
        # the smallest call: a float32 toy model, one request; launches and latency count
        {"name": "decode-tiny", "kind": "decode", "shape": TINY, "layers": 2, "batch": 1, "lo": 200, "hi": 200},
        # whole models, one request: the decode step that a chain of thought repeats thousands of times
        {"name": "decode-1.5b", "kind": "decode", "shape": Q15, "layers": 28, "batch": 1, "lo": 4096, "hi": 4096},
        {"name": "decode-7b-long", "kind": "decode", "shape": Q7, "layers": 28, "batch": 1, "lo": 14336, "hi": 14336},
        # several requests of ragged lengths in one step
        {"name": "decode-7b-b4", "kind": "decode", "shape": Q7, "layers": 4, "batch": 4, "lo": 3000, "hi": 14000},
        {"name": "decode-8b-b8", "kind": "decode", "shape": L8, "layers": 4, "batch": 8, "lo": 3000, "hi": 14000},
        # the same with the fp8 KV cache, an odd batch
        {"name": "decode-8b-b11-fp8", "kind": "decode", "shape": L8 + "-fp8kv", "layers": 4, "batch": 11, "lo": 3000,
         "hi": 14000},
        # the confidence probe of one request at the end of a long chain of thought
        {"name": "probe-7b", "kind": "probe", "shape": Q7, "layers": 4, "batch": 1, "lo": 14001, "hi": 14001},
        # a busy server: every step, half of eight requests probe beside the decode rows
        {"name": "mixed-8b-b8", "kind": "mixed", "shape": L8, "layers": 4, "batch": 8, "lo": 3000, "hi": 14000},
        # prompts (50 to 275 tokens), with a wide workspace and with the binding's default of 16 rows
        {"name": "prefill-7b-256", "kind": "prefill", "shape": Q7, "layers": 4, "n": 256, "ctx": 0, "max_rows": 64},
        {"name": "prefill-1.5b-203", "kind": "prefill", "shape": Q15, "layers": 8, "n": 203, "ctx": 0, "max_rows": 16},
        # the forced conclusion: its prompt appended after a long chain of thought
        {"name": "prefill-8b-conclusion", "kind": "prefill", "shape": L8, "layers": 4, "n": 37, "ctx": 9001,
         "max_rows": 64},
        # a request's K/V arrives from elsewhere and is laid out in pages
        {"name": "import-7b", "kind": "import", "shape": Q7, "layers": 8, "ctx": 6001},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["decode", "decode", "decode", "probe", "mixed", "prefill", "prefill", "import", "export"])
    shape = rng.choice([Q15, Q7, L8])
    layers = rng.randint(3, 5)
    if kind in ("decode", "probe", "mixed") and rng.random() < 0.25:
        shape += "-fp8kv"
    if kind in ("decode", "mixed"):
        batch = _log_int(rng, 1, 16) if kind == "decode" else rng.randint(2, 12)
        lo = _log_int(rng, 100, 14000)
        return {"kind": kind, "shape": shape, "layers": layers, "batch": batch, "lo": lo, "hi": rng.randint(lo, 14336)}
    if kind == "probe":
        lo = _log_int(rng, 1000, 14000)
        return {"kind": kind, "shape": shape, "layers": layers, "batch": rng.randint(1, 6), "lo": lo,
                "hi": rng.randint(lo, 14336)}
    if kind == "prefill":
        ctx = 0 if rng.random() < 0.6 else _log_int(rng, 1000, 14000)
        n = rng.randint(50, 400) if ctx == 0 else rng.randint(5, 80)
        return {"kind": kind, "shape": shape, "layers": layers, "n": n, "ctx": ctx, "max_rows": rng.choice([16, 32, 64])}
    return {"kind": kind, "shape": shape, "layers": layers, "ctx": _log_int(rng, 100, 14336)}


# ------------------------------------------------------------------------------ inputs

def _shape(case):
    return replace(SHAPES[case["shape"]], n_layers=case["layers"])


def _lengths(case, seed):
    """KV lengths of the batch: the two ends of the range, the rest uniform between them."""
    b, lo, hi = case["batch"], case["lo"], case["hi"]
    g = torch.Generator().manual_seed(4000 + seed)
    mid = [int(x) for x in torch.randint(lo, hi + 1, (b,), generator=g)]
    return [lo] + mid[2:] + ([hi] if b > 1 else [])


def _base(seed):
    return 1000 + 100003 * (int(seed) % 10007)


def _weights(shape, seed):
    w = synth.make_weights(shape, device=DEV, seed_base=_base(seed))
    g = torch.Generator(device=DEV).manual_seed(_base(seed) + 50000)
    for name, t in w.items():
        if name.endswith("norm"):
            t.copy_(1.0 + 0.1 * torch.randn(t.shape, generator=g, device=DEV))
    w["final_norm"].mul_(FINAL_GAIN)
    return w


def _dense_kv(shape, length, request, seed):
    return synth.make_prefill_kv(shape, length, request, device=DEV, seed_base=_base(seed) + 60000)


def _tokens(n, shape, seed, salt):
    return synth.make_tokens(n, shape.vocab, _base(seed) + 70000 + salt).to(DEV)


def _probing(case):
    """The probing half of a mixed step's batch."""
    return list(range(0, case["batch"] - case["batch"] % 2, 2))


def _rows(case):
    """Rows of the widest forward: what the caller sizes the workspace for."""
    if case["kind"] == "decode":
        return case["batch"]
    if case["kind"] == "probe":
        return SUFFIX * case["batch"]
    if case["kind"] == "mixed":
        return case["batch"] + SUFFIX * len(_probing(case))
    return case.get("max_rows", 16)


def _pages(n):
    return (n + 15) // 16


def _dt(shape):
    return {"fp8": torch.float8_e4m3fn, "bf16": torch.bfloat16, "f32": torch.float32}[shape.kv_storage]


def prepare(case, seed):
    shape = _shape(case)
    kind = case["kind"]
    w = _weights(shape, seed)
    model = L.Model(shape, w, max_rows=max(_rows(case), 1))
    st = {"case": case, "shape": shape, "model": model, "steps": 0}
    if kind in ("decode", "probe", "mixed"):
        lens = _lengths(case, seed)
        room = 128
        kv = L.KVCache(model, sum(_pages(n + room) for n in lens), len(lens), _pages(max(lens) + room))
        for b, n in enumerate(lens):
            kv.add_seq(b, n)
            kv.import_kv(b, *_dense_kv(shape, n, b, seed))
        B = len(lens)
        st.update(kv=kv, lens=lens, seqs=list(range(B)), tok=_tokens(B, shape, seed, 1),
                  next=torch.zeros(B, dtype=torch.int32, device=DEV), p=torch.zeros(B, device=DEV))
        if kind == "decode":
            st["logits"] = torch.zeros(B, shape.vocab, device=DEV)
        else:
            n = B if kind == "probe" else len(_probing(case))
            st.update(suffix=_tokens(SUFFIX, shape, seed, 2), conf=torch.zeros(n, device=DEV),
                      arg=torch.zeros(n * TRIALS, dtype=torch.int32, device=DEV))
        if kind == "probe":
            st["logits"] = torch.zeros(B, TRIALS, shape.vocab, device=DEV)
        return st
    if kind == "prefill":
        n, ctx = case["n"], case["ctx"]
        kv = L.KVCache(model, _pages(ctx) + _pages(ctx + n) + 2, 2, _pages(ctx + n) + 1)
        kv.k_pool.zero_()
        kv.v_pool.zero_()
        if ctx:
            kv.add_seq(0, ctx)
            kv.import_kv(0, *_dense_kv(shape, ctx, 0, seed))
        st.update(kv=kv, tok=_tokens(n, shape, seed, 1), logits=torch.zeros(shape.vocab, device=DEV), live=False)
        return st
    ctx = case["ctx"]
    kv = L.KVCache(model, _pages(ctx) + 1, 1, _pages(ctx) + 1)
    kv.k_pool.zero_()
    kv.v_pool.zero_()
    k, v = _dense_kv(shape, ctx, 0, seed)
    st.update(kv=kv, k=k, v=v)
    kv.add_seq(0, ctx)
    if kind == "export":
        kv.import_kv(0, k, v)
        st.update(k=torch.zeros_like(k), v=torch.zeros_like(v))
    return st


# ------------------------------------------------------------------------------ one pass

def _pools(st):
    kv, dt = st["kv"], _dt(st["shape"])
    return {"k": kv.k_pool.view(dt), "v": kv.v_pool.view(dt)}


def _start_over(st):
    """The requests finish and others of the same lengths take their slots (and pages)."""
    for b in st["seqs"]:
        st["kv"].free_seq(b)
    for b, n in zip(st["seqs"], st["lens"]):
        st["kv"].add_seq(b, n)


def run(st):
    case, model, kv = st["case"], st["model"], st["kv"]
    kind = case["kind"]
    if kind in ("decode", "mixed"):
        if st["steps"] == RESET_EVERY:
            _start_over(st)
            st["steps"] = 0
        st["steps"] += 1
    if kind == "decode":
        L.laser_decode_step(model, kv, st["seqs"], st["tok"], st["tok"], st["p"], st["logits"])
        return {"next": st["tok"], "p": st["p"], "logits": st["logits"]}
    if kind == "probe":
        L.laser_probe_confidence(model, kv, st["seqs"], st["suffix"], TRIALS, st["conf"], st["arg"], st["logits"])
        return {"conf": st["conf"], "arg": st["arg"], "logits": st["logits"]}
    if kind == "mixed":
        L.laser_step_mixed(model, kv, st["seqs"], st["tok"], st["next"], st["p"], _probing(case), st["suffix"], TRIALS,
                           st["conf"], st["arg"])
        st["tok"], st["next"] = st["next"], st["tok"]
        return {"next": st["tok"], "p": st["p"], "conf": st["conf"], "arg": st["arg"]}
    if kind == "prefill":
        if st["live"]:
            kv.free_seq(1)  # the last pass's request is done
        if case["ctx"]:
            kv.fork(0, 1)
        else:
            kv.add_seq(1, 0)
        st["live"] = True
        L.laser_prefill(model, kv, 1, st["tok"], st["logits"])
        return {"logits": st["logits"], **_pools(st)}
    if kind == "import":
        kv.free_seq(0)
        kv.add_seq(0, case["ctx"])
        kv.import_kv(0, st["k"], st["v"])
        return _pools(st)
    kv.export_kv(0, st["k"], st["v"])
    return {"k": st["k"], "v": st["v"]}


# ------------------------------------------------------------------------------ what a pass needs

def work(case):
    shape = _shape(case)
    kind = case["kind"]
    per_tok = shape.kv_bytes_per_token()
    if kind in ("import", "export"):
        return {"bytes": 2.0 * case["ctx"] * per_tok, "flops": 0.0}
    es = 2 if shape.dtype == "bf16" else 4
    head = shape.vocab * shape.d_model
    blocks = shape.weight_bytes() // es - head
    attn = 4.0 * shape.n_layers * shape.n_q_heads * shape.head_dim  # flops per row and position

    def forward(rows, outs, positions, reads):
        """Weights once, the K/V that the rows see once, logits written."""
        return (es * (blocks + (head if outs else 0)) + reads * per_tok + rows * per_tok,
                2.0 * rows * blocks + 2.0 * outs * head + attn * positions)

    if kind == "prefill":
        n, ctx = case["n"], case["ctx"]
        b, f = forward(n, 1, n * ctx + n * (n + 1) / 2, ctx)
        return {"bytes": b + 4.0 * shape.vocab, "flops": f}
    lens = _lengths(case, 0)
    B, tot = len(lens), sum(lens)
    if kind == "decode":
        b, f = forward(B, B, tot, tot)
        return {"bytes": b + 4.0 * B * shape.vocab, "flops": f}
    probing = list(range(B)) if kind == "probe" else _probing(case)
    n, ptot = len(probing), sum(lens[i] for i in probing)
    extra = (B, B, tot, tot) if kind == "mixed" else (0, 0, 0, ptot)
    b, f = forward(SUFFIX * n + extra[0], n + extra[1], SUFFIX * ptot + extra[2], extra[3])
    for _ in range(TRIALS - 1):
        tb, tf = forward(n, n, ptot, ptot)
        b, f = b + tb, f + tf
    if kind == "probe":
        b += 4.0 * n * TRIALS * shape.vocab
    return {"bytes": b, "flops": f}


def tolerance(case):
    if case["kind"] in ("import", "export"):
        return "exact"  # bytes are moved, nothing is computed
    if case["kind"] == "prefill":
        # appended K/V are rounded to bf16: a last-bit difference before the rounding
        # moves a value by one step of its type
        return {"rel": 3e-3, "max": 2e-2}
    return {"rel": 6e-4, "max": 2e-3, "differ": 0.3}


# ------------------------------------------------------------------------------ 64 bits

class _Exact:
    """The decoder of configs.ModelShape in float64 torch; K/V rounded to their storage type when appended."""

    def __init__(self, shape, w):
        self.s, self.w = shape, w
        half = shape.head_dim // 2
        # the library takes rope_theta and rms_eps as float32
        theta = float(torch.tensor(shape.rope_theta, dtype=torch.float32))
        self.eps = float(torch.tensor(shape.rms_eps, dtype=torch.float32))
        i = torch.arange(half, dtype=torch.float64, device=DEV)
        self.freq = theta ** (-2.0 * i / shape.head_dim)
        self.k, self.v = {}, {}  # seq -> [layer] -> [len][hkv][hd]

    def load(self, seq, k, v):
        self.k[seq] = [t.double() for t in k]
        self.v[seq] = [t.double() for t in v]

    def new(self, seq):
        s = self.s
        self.k[seq] = [torch.zeros(0, s.n_kv_heads, s.head_dim, dtype=torch.float64, device=DEV) for _ in range(s.n_layers)]
        self.v[seq] = [t.clone() for t in self.k[seq]]

    def cut(self, seq, n):
        self.k[seq] = [t[:n] for t in self.k[seq]]
        self.v[seq] = [t[:n] for t in self.v[seq]]

    def len(self, seq):
        return self.k[seq][0].shape[0]

    def _mm(self, x, name):
        w = self.w[name]
        return torch.cat([x @ c.double().t() for c in w.split(16384)], dim=1)

    def _norm(self, h, name):
        return h * torch.rsqrt(h.square().mean(1, keepdim=True) + self.eps) * self.w[name].double()

    def _rope(self, x, pos):
        half = self.s.head_dim // 2
        a = pos.double()[:, None] * self.freq[None, :]
        c, s = torch.cos(a)[:, None, :], torch.sin(a)[:, None, :]
        lo, hi = x[..., :half], x[..., half:]
        return torch.cat([lo * c - hi * s, hi * c + lo * s], dim=-1)

    def forward(self, spans):
        """spans: (seq, tokens) lists; the rows are appended.  Returns the logits of each span's last row."""
        s = self.s
        hq, hkv, hd = s.n_q_heads, s.n_kv_heads, s.head_dim
        tok = torch.cat([t.long() for _, t in spans])
        pos = torch.cat([torch.arange(len(t), device=DEV) + self.len(q) for q, t in spans])
        h = self.w["embed"][tok].double()
        at = [0]
        for _, t in spans:
            at.append(at[-1] + len(t))
        for i in range(s.n_layers):
            p = "layers.%d." % i
            x = self._norm(h, p + "attn_norm")
            q, k, v = (self._mm(x, p + "w" + c) for c in "qkv")
            if s.qkv_bias:
                q, k, v = (y + self.w[p + "b" + c].double() for y, c in zip((q, k, v), "qkv"))
            q = self._rope(q.view(-1, hq, hd), pos)
            k = self._rope(k.view(-1, hkv, hd), pos).to(torch.float32).to(_dt(s)).double()
            v = v.view(-1, hkv, hd).to(torch.float32).to(_dt(s)).double()
            o = torch.zeros_like(q)
            for j, (sq, _) in enumerate(spans):
                a, b = at[j], at[j + 1]
                self.k[sq][i] = K = torch.cat([self.k[sq][i], k[a:b]])
                self.v[sq][i] = V = torch.cat([self.v[sq][i], v[a:b]])
                qs = q[a:b].view(b - a, hkv, hq // hkv, hd).permute(1, 2, 0, 3).reshape(hkv, -1, hd)
                sc = (qs @ K.permute(1, 2, 0).contiguous()) / math.sqrt(hd)
                sc = sc.view(hkv, hq // hkv, b - a, -1)
                seen = torch.arange(K.shape[0], device=DEV)[None, :] <= pos[a:b, None]
                pr = torch.softmax(sc.masked_fill(~seen, float("-inf")), dim=-1).view(hkv, -1, K.shape[0])
                ov = pr @ V.permute(1, 0, 2).contiguous()
                o[a:b] = ov.view(hkv, hq // hkv, b - a, hd).permute(2, 0, 1, 3).reshape(b - a, hq, hd)
            h = h + self._mm(o.reshape(-1, hq * hd), p + "wo")
            x = self._norm(h, p + "mlp_norm")
            g = self._mm(x, p + "w_gate")
            h = h + self._mm(g * torch.sigmoid(g) * self._mm(x, p + "w_up"), p + "w_down")
        x = self._norm(h[[e - 1 for e in at[1:]]], "final_norm")
        return self._mm(x, "embed" if s.tied_embeddings else "lm_head")


def _pmax(lg):
    return torch.softmax(lg, dim=1).max(dim=1).values


def _trials(m, probing, logits):
    """The fed-back trial tokens after a probe's suffix: (confidences, argmax, logits)."""
    toks, ps, lgs = [logits.argmax(1)], [_pmax(logits)], [logits]
    for _ in range(TRIALS - 1):
        lg = m.forward([(b, toks[-1][i:i + 1]) for i, b in enumerate(probing)])
        toks.append(lg.argmax(1))
        ps.append(_pmax(lg))
        lgs.append(lg)
    return torch.stack(ps).mean(0), torch.stack(toks, 1).reshape(-1), torch.stack(lgs, 1)


def _page_order(t, k):
    """Dense [layers][len][hkv][hd] values in the pools' order (include/laser.h), pages in order of position."""
    nl, n, hkv, hd = t.shape
    pages = _pages(n)
    full = torch.zeros(nl, pages * 16, hkv, hd, dtype=t.dtype, device=t.device)
    full[:, :n] = t
    full = full.view(nl, pages, 16, hkv, hd).transpose(2, 3)  # [layer][page][head][16][hd]
    if k:
        x = full.view(nl, pages, hkv, 16, hd // 8, 8).transpose(3, 4)
    else:
        x = full.view(nl, pages, hkv, 4, 4, hd // 16, 16).permute(0, 1, 2, 5, 3, 6, 4)
    return x.reshape(nl, pages, -1)


def exact(case, seed):
    shape = _shape(case)
    kind = case["kind"]
    if kind in ("import", "export"):
        k, v = _dense_kv(shape, case["ctx"], 0, seed)
        if kind == "export":
            return {"k": k, "v": v}
        out = {}
        for name, t in (("k", k), ("v", v)):
            x = _page_order(t.double(), name == "k")
            pool = torch.zeros(shape.n_layers, _pages(case["ctx"]) + 1, x.shape[2], dtype=torch.float64, device=DEV)
            pool[:, : x.shape[1]] = x
            out[name] = pool.reshape(-1)
        return out
    m = _Exact(shape, _weights(shape, seed))
    if kind == "prefill":
        n, ctx = case["n"], case["ctx"]
        if ctx:
            m.load(0, *_dense_kv(shape, ctx, 0, seed))
        else:
            m.new(0)
        lg = m.forward([(0, _tokens(n, shape, seed, 1))])
        out = {"logits": lg[0]}
        pages = _pages(ctx) + _pages(ctx + n) + 2
        for name, t in (("k", torch.stack(m.k[0])), ("v", torch.stack(m.v[0]))):
            x = _page_order(t, name == "k")
            pool = torch.zeros(shape.n_layers, pages, x.shape[2], dtype=torch.float64, device=DEV)
            whole = ctx // 16  # the fork shares these; its own pages come after all of the first request's
            pool[:, :whole] = x[:, :whole]
            if ctx % 16:
                pool[:, whole] = _page_order(t[:, whole * 16:ctx], name == "k")[:, 0]
            own = x[:, whole:]
            pool[:, _pages(ctx):_pages(ctx) + own.shape[1]] = own
            out[name] = pool.reshape(-1)
        return out
    lens = _lengths(case, seed)
    B = len(lens)
    for b, n in enumerate(lens):
        m.load(b, *_dense_kv(shape, n, b, seed))
    tok = _tokens(B, shape, seed, 1)
    if kind == "decode":
        lg = m.forward([(b, tok[b:b + 1]) for b in range(B)])
        return {"next": None, "p": _pmax(lg), "logits": lg}
    suffix = _tokens(SUFFIX, shape, seed, 2)
    if kind == "probe":
        conf, _, lgs = _trials(m, list(range(B)), m.forward([(b, suffix) for b in range(B)]))
        return {"conf": conf, "arg": None, "logits": lgs}
    probing = _probing(case)
    lg = m.forward([(b, tok[b:b + 1]) for b in range(B)])
    conf, _, _ = _trials(m, probing, m.forward([(b, suffix) for b in probing]))
    return {"next": None, "p": _pmax(lg), "conf": conf, "arg": None}
