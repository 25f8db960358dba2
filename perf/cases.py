"""The work that users of this library have it do, as timed and compared cases.

Five kinds of case, each one pass through the public entry points of
``paper_2109_08008_amd.nt``:

* ``proj``      one dense projection, ``nt_op_gemm``;
* ``proj_ln``   one projection with its pre-norm LayerNorm folded in, ``nt_op_gemm_ln``;
* ``select``    one beam selection over a matrix of logits, ``nt_op_select``;
* ``score``     a batch encoded and its given targets scored step by step (``nt_encode``,
                ``nt_decode_step`` with forced tokens and copied-out logits);
* ``translate`` a whole job, ``nt_translate``: sorting, batching, encoder, search, results
                back in host memory.

Weights follow the benchmark's recipe (N(0, 0.02), LayerNorm gains around 1, DLCL rows
around the mean of their entries), with the matrices on the fp16 grid as a half-precision
checkpoint has them; sentences have log-normal lengths and Zipf word frequencies.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2109_08008_amd import nt

PAD, BOS, EOS, FIRST_WORD = 0, 1, 2, 4
LN_EPS = 1e-5
F8_MAX = 448.0
TORCH = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16, "f8w": torch.float16}
BYTES = {"f32": 4, "f16": 2, "bf16": 2, "f8w": 2}
_SIZES = ("d", "heads", "ffn", "n_enc", "n_dec", "vocab")
_TINY = dict(zip(_SIZES, (128, 4, 512, 6, 1, 1000)))
_BASE = dict(zip(_SIZES, (512, 8, 2048, 6, 6, 32000)))
_DEEP = dict(zip(_SIZES, (512, 8, 2048, 35, 1, 32000)))
_SMALL = dict(zip(_SIZES, (256, 4, 1024, 9, 1, 32000)))
_WIDE = dict(zip(_SIZES, (1024, 16, 4096, 30, 6, 32000)))


def listed():
    return [
        # a decoder step's query/key/value projection while few sentences are live (16 x beam 4)
        {"name": "qkv_step_small", "kind": "proj_ln", "dtype": "f16", "m": 64, "n": 1536, "k": 512, "relu": False},
        # the first FFN projection of a wide decoder's step at an ordinary batch (540 x beam 4)
        {"name": "ffn1_step_wide", "kind": "proj_ln", "dtype": "f16", "m": 2160, "n": 4096, "k": 1024, "relu": True},
        # the second FFN projection of the wide encoder on a full 16384-token batch
        {"name": "ffn2_enc_wide", "kind": "proj", "dtype": "f16", "m": 16384, "n": 1024, "k": 4096, "epi": "resid"},
        # the first FFN projection of a base encoder in bf16 on a batch that fills no tile evenly
        {"name": "ffn1_enc_ragged", "kind": "proj", "dtype": "bf16", "m": 5003, "n": 2048, "k": 512, "epi": "relu"},
        # the base encoder's query/key/value projection with FP8 weights on a full batch
        {"name": "qkv_enc_fp8", "kind": "proj", "dtype": "f8w", "m": 8192, "n": 1536, "k": 512, "epi": "store"},
        # an fp32 model's attention output projection
        {"name": "out_enc_f32", "kind": "proj", "dtype": "f32", "m": 4096, "n": 512, "k": 512, "epi": "resid"},
        # the tied output projection of a step, its logits wanted (325 x beam 4)
        {"name": "vocab_logits", "kind": "proj", "dtype": "f16", "m": 1300, "n": 32000, "k": 512, "epi": "logits"},
        # the beam's candidates out of a step's logits
        {"name": "beam_select", "kind": "select", "rows": 1300, "vocab": 32000, "k": 8},
        # 96 reference translations scored with the base model: encoder, then forced decoding
        {"name": "score_base", "kind": "score", **_BASE, "dtype": "f16", "n_sent": 96, "mean": 25.0, "longest": 60,
         "steps": 12},
        # the smallest whole job: a tiny fp32 model, eight short sentences, greedy
        {"name": "translate_tiny", "kind": "translate", **_TINY, "dtype": "f32", "n_sent": 8, "mean": 12.0,
         "longest": 16, "beam": 1, "alpha": 0.0, "budget": 8192},
        # a deep encoder with a shallow decoder, greedy, some hundreds of sentences
        {"name": "translate_deep", "kind": "translate", **_DEEP, "dtype": "f16", "n_sent": 1024, "mean": 25.0,
         "longest": 150, "beam": 1, "alpha": 0.0, "budget": 8192},
        # the wide teacher model, beam 4
        {"name": "translate_wide", "kind": "translate", **_WIDE, "dtype": "f16", "n_sent": 512, "mean": 30.0,
         "longest": 200, "beam": 4, "alpha": 0.0, "budget": 16384},
    ]


def draw(rng):
    def spread(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(("proj", "proj", "proj_ln", "proj_ln", "select", "score", "translate", "translate"))
    if kind in ("proj", "proj_ln"):
        d = rng.choice((128, 256, 384, 512, 768, 1024))
        n, k = rng.choice(((d, d), (3 * d, d), (4 * d, d)) + (((d, 4 * d),) if kind == "proj" else ()))
        c = {"kind": kind, "dtype": rng.choice(("f16", "f16", "f16", "bf16", "f32", "f8w")),
             "m": spread(1, 16384 if kind == "proj" else 6000), "n": n, "k": k}
        if kind == "proj_ln":
            return dict(c, relu=n == 4 * d)
        epi = "relu" if n == 4 * d else "store" if n == 3 * d else "resid"
        if rng.random() < 0.2 and c["dtype"] != "f8w":     # the tied output projection
            c.update(m=min(c["m"], 2600), n=spread(1000, 40000), k=d)
            epi = "logits"
        return dict(c, epi=epi)
    if kind == "select":
        return {"kind": kind, "rows": spread(1, 4000), "vocab": spread(500, 40000), "k": rng.choice((4, 8, 10, 16))}
    shape = dict(rng.choice((_TINY, _SMALL, _BASE, _DEEP)))
    shape["vocab"] = spread(1000, 36000)
    c = {"kind": kind, **shape, "dtype": rng.choice(("f16", "f16", "bf16", "f32")), "mean": round(rng.uniform(12, 30), 1),
         "longest": rng.randint(40, 120)}
    if kind == "score":
        return dict(c, n_sent=spread(1, 96), steps=rng.randint(4, 12))
    beam = rng.choice((1, 1, 2, 4, 5, 8))
    return dict(c, n_sent=spread(1, 400 if beam == 1 else 160), beam=beam, alpha=rng.choice((0.0, 0.6)),
                budget=rng.choice((4096, 8192, 16384)))


# ---- inputs ------------------------------------------------------------------------------
def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _normal(g, *shape):
    return torch.randn(shape, generator=g, device="cuda")


def _proj_inputs(c, seed):
    """A projection's operands: LayerNorm'd or ReLU'd activations, weights of the recipe."""
    g, dt, m, n, k = _gen(seed), TORCH[c["dtype"]], c["m"], c["n"], c["k"]
    s = {"a": _normal(g, m, k), "bias": 0.02 * _normal(g, n)}
    if c["kind"] == "proj_ln":
        s["a"] = 1.5 * s["a"] + 0.3 * _normal(g, m, 1)      # a residual stream, row means off zero
    elif k > n:
        s["a"] = s["a"].clamp(min=0)                        # FFN hidden values
    s["a"] = s["a"].to(dt)
    w = (0.02 if c.get("epi") != "logits" else 1 / math.sqrt(k)) * _normal(g, n, k)
    if c["dtype"] == "f8w":
        s["scale"] = w.abs().amax(1) / F8_MAX
        s["w"] = (w / s["scale"][:, None]).to(torch.float8_e4m3fn)
        if c["kind"] == "proj_ln":
            s["colsum"] = (s["w"].double().sum(1) * s["scale"].double()).float()
    else:
        s["w"] = w.to(dt)
        if c["kind"] == "proj_ln":
            s["colsum"] = s["w"].double().sum(1).float()
    if c.get("epi") == "resid":
        s["resid"] = _normal(g, m, n).to(dt)
    return s


def _layout(c):
    """The weight blob's entries in their canonical order: (name, shape, recipe)."""
    d, f, v = c["d"], c["ffn"], c["vocab"]
    ln = lambda p: [(p + ".g", (d,), "gain"), (p + ".b", (d,), "vector")]  # noqa: E731
    mat = lambda p, i, o: [(p, (i, o), "matrix"), (p + ".b", (o,), "vector")]  # noqa: E731
    out = [("E", (v, d), "matrix")]
    for k in range(c["n_enc"] + 1):
        out += ln("hist%d" % k)
    for row in range(1, c["n_enc"] + 2):
        out.append(("dlcl%d" % row, (row,), "mean"))
    for i in range(c["n_enc"]):
        p = "e%d." % i
        out += ln(p + "ln1") + mat(p + "qkv", d, 3 * d) + mat(p + "o", d, d) + ln(p + "ln2")
        out += mat(p + "w1", d, f) + mat(p + "w2", f, d)
    out += ln("enc_out")
    for j in range(c["n_dec"]):
        p = "d%d." % j
        out += ln(p + "ln1") + mat(p + "qkv", d, 3 * d) + mat(p + "o", d, d) + ln(p + "ln2") + mat(p + "q", d, d)
        out += mat(p + "kv", d, 2 * d) + mat(p + "oc", d, d) + ln(p + "ln3") + mat(p + "w1", d, f) + mat(p + "w2", f, d)
    return out + ln("dec_out")


def _blob(c, seed):
    """The fp32 weight blob on the GPU, and its entries by name."""
    lay = _layout(c)
    blob = 0.02 * _normal(_gen(seed), sum(math.prod(s) for _, s, _ in lay))
    named, at = {}, 0
    for name, shape, recipe in lay:
        v = blob[at:at + math.prod(shape)].view(shape)
        at += v.numel()
        if recipe == "matrix":
            v.copy_(v.half())
        elif recipe == "gain":
            v.add_(1.0)
        elif recipe == "mean":
            v.add_(1.0 / shape[0])
        named[name] = v
    # Untrained weights say nothing about where a sentence ends, and leave a beam's hypotheses
    # near ties.  Without an EOS row every hypothesis runs to its length limit, whatever the
    # seed; with a longer first row that word follows itself with a probability of about 0.7,
    # which keeps the best hypothesis apart from the others, as training does.
    d, limit = c["d"], math.log(c["vocab"]) + 1.0
    rest = d / 2 + c["n_dec"] * d * ((4e-4 * d) ** 2 + 8e-8 * d * c["ffn"])   # positions and sublayers, squared
    x = 1.0
    while x * x / math.sqrt(x * x + rest) < limit:
        x *= 1.01
    named["E"][EOS].zero_()
    named["E"][BOS].mul_(x / (0.02 * d)).copy_(named["E"][BOS].half())
    return blob, named


def _sentences(c, seed):
    """Source sentences as the library takes them: IDs and offsets on the host.  The lengths
    are the log-normal's quantiles in the seed's order, so that a case's size is its own."""
    r = np.random.default_rng(seed)
    at = torch.special.ndtri((torch.arange(c["n_sent"], dtype=torch.float64) + 0.5) / c["n_sent"]).numpy()
    lens = np.clip(np.rint(np.exp(math.log(c["mean"]) - 0.125 + 0.5 * at)), 1, c["longest"])
    lens = r.permutation(lens)
    offs = np.zeros(c["n_sent"] + 1, np.int64)
    offs[1:] = np.cumsum(lens.astype(np.int64))
    p = np.arange(1, c["vocab"] - FIRST_WORD + 1) ** -1.1
    ids = FIRST_WORD + np.searchsorted(np.cumsum(p) / p.sum(), r.random(int(offs[-1])))
    return np.minimum(ids, c["vocab"] - 1).astype(np.int32), offs


def _padded(ids, offs):
    lens = np.diff(offs).astype(np.int32)
    src = np.zeros((len(lens), lens.max()), np.int32)
    for i, n in enumerate(lens):
        src[i, :n] = ids[offs[i]:offs[i + 1]]
    return src, lens


def _targets(c, seed):
    """Forced target words [steps, n_sent]."""
    r = np.random.default_rng(seed + 1)
    return r.integers(FIRST_WORD, c["vocab"], (c["steps"], c["n_sent"]), dtype=np.int32)


class _Shape:
    def __init__(self, c):
        self.d_model, self.n_heads, self.d_ffn = c["d"], c["heads"], c["ffn"]
        self.n_enc, self.n_dec, self.vocab = c["n_enc"], c["n_dec"], c["vocab"]
        self.max_positions = 1024


def _search(c):
    if c["kind"] == "score":
        return nt.nt_search_cfg(1, 0.0, 0.0, c["steps"], 0, 0, 0, 1, 1)
    return nt.nt_search_cfg(c["beam"], c["alpha"], 1.5, 10, 0, c["budget"], 0, 1, 1)


def prepare(case, seed):
    c, kind = case, case["kind"]
    s = {"case": c, "stream": torch.cuda.current_stream().cuda_stream}
    if kind in ("proj", "proj_ln"):
        s.update(_proj_inputs(c, seed))
        s["out"] = torch.empty(c["m"], c["n"], device="cuda",
                               dtype=torch.float32 if c.get("epi") == "logits" else TORCH[c["dtype"]])
        return s
    if kind == "select":
        s["logits"] = 2.0 * _normal(_gen(seed), c["rows"], c["vocab"])
        s["topv"] = torch.empty(c["rows"], c["k"], device="cuda")
        s["topi"] = torch.empty(c["rows"], c["k"], dtype=torch.int32, device="cuda")
        s["lse"] = torch.empty(c["rows"], device="cuda")
        return s
    s["model"] = nt.Model(_Shape(c), _blob(c, seed)[0].cpu().numpy(), c["dtype"])
    s["search"] = _search(c)
    s["ids"], s["offs"] = _sentences(c, seed)
    if kind == "translate":
        s["ws"] = s["model"].workspace(nt.nt_translate_workspace_size(s["model"].handle, s["search"], s["offs"]))
        s["cap"] = sum(nt.max_target_tokens(s["search"], int(n)) for n in np.diff(s["offs"]))
        return s
    src, s["lens"] = _padded(s["ids"], s["offs"])
    s["src"], s["d_lens"] = torch.from_numpy(src).cuda(), torch.from_numpy(s["lens"]).cuda()
    s["forced"] = torch.from_numpy(_targets(c, seed)).cuda()
    s["logits"] = torch.empty(c["steps"], c["n_sent"], c["vocab"], device="cuda")
    s["ws"] = s["model"].workspace(nt.nt_workspace_size(s["model"].handle, s["search"], *src.shape))
    return s


# ---- one pass ------------------------------------------------------------------------------
def run(state):
    s, c = state, state["case"]
    kind = c["kind"]
    if kind == "select":
        nt.nt_op_select(s["logits"].data_ptr(), c["rows"], c["vocab"], c["k"], s["topv"].data_ptr(),
                        s["topi"].data_ptr(), s["lse"].data_ptr(), stream=s["stream"])
        return {"values": s["topv"], "words": s["topi"], "lse": s["lse"]}
    if kind == "proj_ln":
        nt.nt_op_gemm_ln("f16" if c["dtype"] == "f8w" else c["dtype"], s["a"].data_ptr(), c["k"], s["w"].data_ptr(),
                         c["m"], c["n"], c["k"], s["colsum"].data_ptr(), LN_EPS, s["bias"].data_ptr(),
                         s["out"].data_ptr(), c["n"], relu=c["relu"],
                         d_bscale=s["scale"].data_ptr() if "scale" in s else None, stream=s["stream"])
        return s["out"]
    if kind == "proj":
        epi = c["epi"]
        nt.nt_op_gemm("f16" if c["dtype"] == "f8w" else c["dtype"], s["a"].data_ptr(), c["k"], s["w"].data_ptr(),
                      c["m"], c["n"], c["k"], None if epi == "logits" else s["bias"].data_ptr(),
                      s["resid"].data_ptr() if epi == "resid" else None, s["out"].data_ptr(), c["n"],
                      out_f32=epi == "logits", relu=epi == "relu",
                      d_bscale=s["scale"].data_ptr() if "scale" in s else None, stream=s["stream"])
        return s["out"]
    if kind == "translate":
        tokens, offs, score, logp = nt.nt_translate(s["model"].handle, s["search"], s["ids"], s["offs"], s["cap"],
                                                    s["ws"].data_ptr(), s["ws"].numel(), stream=s["stream"])
        return {"tokens": tokens, "offsets": offs, "score": score, "logp": logp}
    st = nt.nt_encode(s["model"].handle, s["src"].data_ptr(), s["d_lens"].data_ptr(), s["lens"], c["n_sent"],
                      s["src"].shape[1], s["search"], s["ws"].data_ptr(), s["ws"].numel(), stream=s["stream"])
    try:
        for t in range(c["steps"]):
            nt.nt_decode_step(st, s["forced"][t].data_ptr(), s["logits"][t].data_ptr(), stream=s["stream"])
        _, score, logp = nt.nt_dec_state_read(st, stream=s["stream"])
    finally:
        nt.nt_free_state(st)
    return {"logits": s["logits"], "score": score, "logp": np.stack(logp)}


# ---- what a pass cannot do without -----------------------------------------------------------
def _model_work(c, lens, targets, beam):
    """Bytes and flops of encoding sentences of `lens` and decoding `targets` steps of each."""
    d, f, v, el, dl = c["d"], c["ffn"], c["vocab"], c["n_enc"], c["n_dec"]
    eb = BYTES[c["dtype"]]
    enc, dec = 4 * d * d + 2 * d * f, 6 * d * d + 2 * d * f
    n, sq = float(lens.sum()), float((lens.astype(np.float64) ** 2).sum())
    h = float(beam * targets.sum())
    ctx = beam * float((targets * (targets + 1) / 2 + targets * lens).sum())
    flops = 2 * n * (el * enc + 2 * dl * d * d) + 4 * d * el * sq + n * d * el * (el + 1) + 2 * h * (dl * dec + d * v) + 4 * d * dl * ctx
    return {"bytes": eb * (v * d + el * enc + dl * (dec + 2 * d * d)) + 4 * n + 8 * float(targets.sum()), "flops": flops}


def work(case):
    c, kind = case, case["kind"]
    if kind in ("proj", "proj_ln"):
        m, n, k, eb = c["m"], c["n"], c["k"], BYTES[c["dtype"]]
        out = 4 if c.get("epi") == "logits" else eb
        moved = m * k * eb + n * k * (1 if c["dtype"] == "f8w" else eb) + m * n * out * (1 if c.get("epi") != "resid" else 2)
        return {"bytes": moved + 4 * n, "flops": 2.0 * m * n * k}
    if kind == "select":
        return {"bytes": 4.0 * c["rows"] * (c["vocab"] + 2 * c["k"] + 1), "flops": 3.0 * c["rows"] * c["vocab"]}
    lens = np.diff(_sentences(c, 0)[1])
    if kind == "score":
        w = _model_work(c, lens, np.full(len(lens), c["steps"]), 1)
        w["bytes"] += 4.0 * c["steps"] * c["n_sent"] * c["vocab"]
        return w
    return _model_work(c, lens, np.floor(1.5 * lens) + 10, c["beam"])


def tolerance(case):
    # One rounding of the result to 11, 8 or 24 bits of mantissa (2.1e-4, 1.7e-3 and 1e-7 of it
    # measured), times four; sums over k in fp32.
    dt = case["dtype"] if "dtype" in case else "f32"
    if case["kind"] in ("proj", "proj_ln"):
        if case.get("epi") == "logits" or dt == "f32":
            return {"rel": 4e-6}
        return {"rel": 7e-3 if dt == "bf16" else 1e-3}
    if case["kind"] == "select":     # chosen values exactly; the log-sum-exp sums V exponentials
        return {"rel": 1e-6, "differ": 0.0}
    # whole models: roundings of the activations travel through every layer (logits 1e-3 and
    # log-probs 6e-4 off at fp16, 4e-3 at bf16, 5e-6 at fp32); a near tie may fall either way
    return {"rel": {"f32": 2e-5, "bf16": 2e-2}.get(dt, 4e-3), "differ": 0.002}


# ---- the same in 64 bits ---------------------------------------------------------------------
def _norm(x, eps=LN_EPS):
    mu = x.mean(-1, keepdim=True)
    return (x - mu) / torch.sqrt(((x - mu) ** 2).mean(-1, keepdim=True) + eps)


class _Exact:
    """The model in fp64: DLCL encoder, and a decoder that steps over cached keys and values."""

    def __init__(self, c, seed):
        self.c, self.d, self.h = c, c["d"], c["heads"]
        self.w = {k: v.double() for k, v in _blob(c, seed)[1].items()}
        m = torch.arange(self.d // 2, dtype=torch.float64, device="cuda")
        ang = torch.arange(1024, dtype=torch.float64, device="cuda")[:, None] / 10000.0 ** (2 * m / self.d)
        self.pe = torch.stack((ang.sin(), ang.cos()), -1).reshape(1024, self.d)

    def ln(self, x, p):
        return _norm(x) * self.w[p + ".g"] + self.w[p + ".b"]

    def mm(self, x, p):
        return x @ self.w[p] + self.w[p + ".b"]

    def split(self, x):                     # [rows, n, d] -> [rows, heads, n, d_head]
        return x.view(x.shape[0], -1, self.h, self.d // self.h).transpose(1, 2).contiguous()

    def attend(self, q, k, v, ok=None):     # q, k, v by head; ok: keys that may be read
        s = q @ k.transpose(2, 3).contiguous() / math.sqrt(self.d // self.h)
        if ok is not None:
            s = s.masked_fill(~ok, -math.inf)
        o = torch.softmax(s, -1) @ v
        return o.transpose(1, 2).reshape(q.shape[0], -1, self.d)

    def encode(self, src, lens):
        """Keys and values of every decoder layer over the padded batch, and its mask."""
        c = self.c
        ok = (torch.arange(src.shape[1], device="cuda") < lens[:, None])[:, None, None, :]
        y = math.sqrt(self.d) * self.w["E"][src] + self.pe[:src.shape[1]]
        hist = [self.ln(y, "hist0")]
        for i in range(c["n_enc"]):
            p = "e%d." % i
            x = sum(w * h for w, h in zip(self.w["dlcl%d" % (i + 1)], hist))
            q, k, v = (self.split(t) for t in self.mm(self.ln(x, p + "ln1"), p + "qkv").chunk(3, -1))
            x = x + self.mm(self.attend(q, k, v, ok), p + "o")
            y = x + self.mm(self.mm(self.ln(x, p + "ln2"), p + "w1").clamp(min=0), p + "w2")
            hist.append(self.ln(y, "hist%d" % (i + 1)))
        x = sum(w * h for w, h in zip(self.w["dlcl%d" % (c["n_enc"] + 1)], hist))
        enc = self.ln(x, "enc_out")
        self.ok = ok
        self.cross = [[self.split(t) for t in self.mm(enc, "d%d.kv" % j).chunk(2, -1)] for j in range(c["n_dec"])]
        self.cache = [None] * c["n_dec"]

    def step(self, tok, t, beam):
        """Logits [sentences, beam, V] of step t for the last words tok [sentences, beam]."""
        b = tok.shape[0]
        z = (math.sqrt(self.d) * self.w["E"][tok] + self.pe[t]).view(b * beam, 1, self.d)
        for j in range(self.c["n_dec"]):
            p = "d%d." % j
            q, k, v = (self.split(x) for x in self.mm(self.ln(z, p + "ln1"), p + "qkv").chunk(3, -1))
            if t:
                k, v = (torch.cat((a, n), 2) for a, n in zip(self.cache[j], (k, v)))
            self.cache[j] = [k, v]
            z = z + self.mm(self.attend(q, k, v), p + "o")
            q = self.split(self.mm(self.ln(z, p + "ln2"), p + "q").view(b, beam, self.d))
            z = z + self.mm(self.attend(q, *self.cross[j], self.ok), p + "oc").view(b * beam, 1, self.d)
            z = z + self.mm(self.mm(self.ln(z, p + "ln3"), p + "w1").clamp(min=0), p + "w2")
        return (self.ln(z, "dec_out") @ self.w["E"].T).view(b, beam, -1)

    def reorder(self, rows):
        self.cache = [[x[rows] for x in kv] for kv in self.cache]


def _exact_search(ref, src, lens, limit, beam, alpha):
    """The search on one batch: [(tokens, log-probs, score)] of its sentences.  Greedy takes
    the best word until EOS or the limit.  The beam walks the 2K best of all K x V
    continuations: EOS finishes a hypothesis with its length-penalised score, the others
    are the next K; a sentence ends once a finished one scores at least every live one, or
    at its limit."""
    ref.encode(src, lens)
    b, pen = src.shape[0], lambda n: ((5.0 + n) / 6.0) ** (alpha if beam > 1 else 0.0)
    live = [[([], [], 0.0)] for _ in range(b)]
    best = [None] * b
    done = [False] * b
    tok = torch.full((b, beam), BOS, device="cuda")
    score = torch.full((b, beam), -math.inf, dtype=torch.float64, device="cuda")
    score[:, 0] = 0.0
    for t in range(max(limit)):
        lp = torch.log_softmax(ref.step(tok, t, beam), -1)
        v = lp.shape[-1]
        top, at = torch.topk((score[:, :, None] + lp).view(b, -1), 1 if beam == 1 else min(2 * beam, beam * v), -1)
        word = lp.view(b, -1).gather(1, at).tolist()
        top, at = top.tolist(), at.tolist()
        rows, n = list(range(b * beam)), t + 1
        for i in range(b):
            if done[i]:
                continue
            kept, parents = [], []
            for cand, k, one in zip(top[i], at[i], word[i]):
                if cand == -math.inf:
                    continue
                old = live[i][k // v]
                if k % v == EOS:
                    if best[i] is None or cand / pen(n) > best[i][2]:
                        best[i] = (old[0], old[1], cand / pen(n))
                    done[i] = done[i] or beam == 1
                elif len(kept) < beam:
                    kept.append((old[0] + [k % v], old[1] + [one], cand))
                    parents.append(k // v)
            live[i] = kept
            if n >= limit[i]:
                for x in kept:
                    if best[i] is None or x[2] / pen(n) > best[i][2]:
                        best[i] = (x[0], x[1], x[2] / pen(n))
                done[i] = True
            elif not kept or (beam > 1 and best[i] is not None and best[i][2] >= max(x[2] for x in kept) / pen(n)):
                done[i] = True
            for k, p in enumerate(parents):
                rows[i * beam + k] = i * beam + p
        if all(done):
            break
        fill = lambda f, none: [[f(x[k]) if k < len(x) else none for k in range(beam)] for x in live]  # noqa: E731
        tok = torch.tensor(fill(lambda x: x[0][-1] if x[0] else BOS, EOS), device="cuda")
        score = torch.tensor(fill(lambda x: x[2], -math.inf), dtype=torch.float64, device="cuda")
        if beam > 1:
            ref.reorder(torch.tensor(rows, device="cuda"))
    return best


def exact(case, seed):
    c, kind = case, case["kind"]
    if kind in ("proj", "proj_ln"):
        s = _proj_inputs(c, seed)
        a, w = s["a"].double(), s["w"].double()
        if "scale" in s:
            w = w * s["scale"].double()[:, None]
        if kind == "proj_ln":
            out = _norm(a) @ w.T + s["bias"].double()
            return out.clamp(min=0) if c["relu"] else out
        out = a @ w.T
        if c["epi"] != "logits":
            out += s["bias"].double()
        if c["epi"] == "resid":
            out += s["resid"].double()
        return out.clamp(min=0) if c["epi"] == "relu" else out
    if kind == "select":
        x = (2.0 * _normal(_gen(seed), c["rows"], c["vocab"])).double()
        v, i = torch.topk(x, c["k"], -1)
        return {"values": v, "words": i.int(), "lse": torch.logsumexp(x, -1)}
    ref = _Exact(c, seed)
    ids, offs = _sentences(c, seed)
    if kind == "score":
        src, lens = (torch.from_numpy(x).cuda() for x in _padded(ids, offs))
        ref.encode(src.long(), lens)
        forced = torch.from_numpy(_targets(c, seed)).cuda().long()
        logits = []
        for t in range(c["steps"]):
            tok = forced[t - 1] if t else torch.full_like(forced[0], BOS)
            logits.append(ref.step(tok[:, None], t, 1)[:, 0])
        logits = torch.stack(logits)
        logp = torch.log_softmax(logits, -1).gather(2, forced[:, :, None])[:, :, 0].T
        return {"logits": logits, "score": logp.sum(1), "logp": logp}
    sents = [ids[offs[i]:offs[i + 1]] for i in range(c["n_sent"])]
    order = sorted(range(c["n_sent"]), key=lambda i: -len(sents[i]))
    found = [None] * c["n_sent"]
    for at in range(0, len(order), 128):
        part = order[at:at + 128]
        o = np.concatenate(([0], np.cumsum([len(sents[i]) for i in part])))
        src, lens = _padded(np.concatenate([sents[i] for i in part]), o)
        limit = [int(math.floor(1.5 * n)) + 10 for n in lens]
        got = _exact_search(ref, torch.from_numpy(src).cuda().long(), torch.from_numpy(lens).cuda(), limit, c["beam"],
                            c["alpha"])
        for i, g in zip(part, got):
            found[i] = g
    return {"tokens": np.concatenate([np.asarray(f[0], np.int32) for f in found]),
            "offsets": np.concatenate(([0], np.cumsum([len(f[0]) for f in found]))).astype(np.int64),
            "score": np.array([f[2] for f in found]), "logp": np.concatenate([np.asarray(f[1]) for f in found])}
