"""The calls whose time matters to a user of this library, and their inputs.

Two kinds of calls.  Whole encodes: one SuperBatch of packed texts in HBM
(surge_encode_superbatch), from a single query to a full SuperBatch, and a
partition-grouped input in host memory (surge_encode_all_streamed).  Single
layers through their own entry points: the linear layers with their fused
epilogues, the varlen attention, the embedding, the LayerNorm and the
pooling.  Encoder shapes, text-length mixes and SuperBatch sizes are those of
`paper_2605_01060_amd.workload`.

Every case is a dict of plain values.  The order of its texts' lengths, its
partition sizes, token IDs and activations are drawn from the seed; the
lengths themselves come from the case, so its work does not change.  An encoder and its weights are
what a program keeps between calls: one per shape, made once per process.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2605_01060_amd import surge as S
from paper_2605_01060_amd import workload as W

SHAPES = {"tiny": W.TINY, "minilm": W.MINILM, "bge": W.BGE, "large": W.LARGE}
DEV = "cuda"
CHUNK_TOKENS = 1 << 20  # the binding's default workspace


def listed():
    return [
        # A search query embedded on its own while a user waits: latency and
        # launches, 12 layers over 24 tokens.
        {"name": "bge_query", "kind": "encode", "shape": "bge", "texts": 1, "median": 24, "lo": 24,
         "hi": 24, "parts": 1},
        # A small partition encoded by its own call (the paper's
        # per-partition baseline): 57 texts of ~36 tokens.
        {"name": "minilm_partition", "kind": "encode", "shape": "minilm", "texts": 57,
         "median": 32, "lo": 4, "hi": 128, "parts": 1},
        # A mean partition of the large encoder, 24 layers, long texts.
        {"name": "large_partition", "kind": "encode", "shape": "large", "texts": 250,
         "median": 96, "lo": 8, "hi": 512, "parts": 1},
        # The headline: one SuperBatch of the bge workload over 20 partitions.
        {"name": "bge_superbatch", "kind": "encode", "shape": "bge", "texts": 4878, "median": 48,
         "lo": 4, "hi": 256, "parts": 20},
        # Host tokens in, host embeddings out, SuperBatch by SuperBatch.
        {"name": "minilm_stream", "kind": "stream", "shape": "minilm", "texts": 20_000,
         "median": 32, "lo": 4, "hi": 128, "parts": 80, "b_min": 4096, "n_max": 20_000,
         "overlap": 2},
        # FFN up-projection with GELU of a small chunk (MiniLM shape), odd rows.
        {"name": "linear_gelu_small", "kind": "linear", "m": 777, "n": 1536, "k": 384, "epi": 1},
        # QKV projection with the LayerNorm of its input folded in (large
        # shape), a chunk of a few thousand tokens.
        {"name": "linear_qkv_mid", "kind": "linear", "m": 5003, "n": 3072, "k": 1024, "epi": 3},
        # FFN up-projection, LayerNorm folded in, GELU (bge), a SuperBatch's rows.
        {"name": "linear_ffn1_big", "kind": "linear", "m": 200_003, "n": 3072, "k": 768, "epi": 4},
        # FFN down-projection with LayerNorm-ed residual and row statistics
        # (bge), a mean partition's rows.
        {"name": "linear_ffn2_mid", "kind": "linear", "m": 13_579, "n": 768, "k": 3072, "epi": 6},
        # Attention of one bge layer over short texts, some at the limit.
        {"name": "attention_64", "kind": "attention", "texts": 1500, "heads": 12, "dh": 64,
         "median": 48, "lo": 4, "hi": 512},
        # Attention of one MiniLM layer (32-dimensional heads), a small call.
        {"name": "attention_32", "kind": "attention", "texts": 300, "heads": 12, "dh": 32,
         "median": 32, "lo": 4, "hi": 128},
        # Embedding gather + LayerNorm of one bge chunk.
        {"name": "embed_768", "kind": "embed", "texts": 2000, "d": 768, "median": 48, "lo": 4,
         "hi": 256},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["encode", "encode", "stream", "linear", "linear", "linear", "linear",
                       "attention", "attention", "embed", "layernorm", "pool"])
    if kind in ("encode", "stream"):
        shape = rng.choice(["tiny", "minilm", "minilm", "bge", "bge", "large", "large"])
        lo, hi = {"tiny": (8, 64), "minilm": (4, 128), "bge": (4, 256), "large": (8, 512)}[shape]
        if rng.random() < 0.25:  # texts of any length up to the position limit
            lo, hi = 1, SHAPES[shape].max_positions
        median = _log_int(rng, 12, hi // 2)
        cap = {"tiny": 40_000, "minilm": 20_000, "bge": 4_500, "large": 500}[shape]
        cap = max(1, min(cap, int(cap * 48 / median)))
        texts = _log_int(rng, 1, cap)
        c = {"kind": kind, "shape": shape, "texts": texts, "median": median, "lo": lo, "hi": hi,
             "parts": _log_int(rng, 1, min(texts, 64))}
        if kind == "stream":
            c["b_min"] = _log_int(rng, max(1, texts // 8), texts)
            c["n_max"] = rng.choice([0, 5 * c["b_min"]])
            c["overlap"] = rng.choice([0, 1, 2])
        return c
    if kind == "linear":
        d, f = rng.choice([(128, 512), (384, 1536), (768, 3072), (1024, 4096)])
        n, k, epi = rng.choice([(3 * d, d, 0), (3 * d, d, 3), (d, d, 2), (d, d, 5), (d, d, 6),
                                (f, d, 1), (f, d, 4), (d, f, 2), (d, f, 6)])
        return {"kind": "linear", "m": _log_int(rng, 1, 200_000), "n": n, "k": k, "epi": epi}
    lo, hi = rng.choice([(4, 128), (4, 256), (8, 512), (1, 512)])
    median = _log_int(rng, 12, hi // 2)
    texts = _log_int(rng, 1, 200_000 // median)
    c = {"kind": kind, "texts": texts, "median": median, "lo": lo, "hi": hi}
    if kind == "attention":
        c["heads"], c["dh"] = rng.choice([(2, 64), (12, 32), (12, 64), (16, 64)])
    else:
        c["d"] = rng.choice([128, 384, 768, 1024])
    return c


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------

def _cu(case, seed):
    """int64 [texts+1]: log-normal text lengths (sigma 0.5) clipped to [lo, hi],
    the same ones for every seed in another order."""
    z = np.random.default_rng([case["texts"], case["median"]]).standard_normal(case["texts"])
    length = np.clip(np.rint(case["median"] * np.exp(0.5 * z)), case["lo"], case["hi"])
    length = np.random.default_rng([seed, 1]).permutation(length)
    cu = np.zeros(case["texts"] + 1, np.int64)
    np.cumsum(length.astype(np.int64), out=cu[1:])
    return cu


def _tokens(cu, seed):
    return W.token_ids(np.random.default_rng([seed, 2]), cu)


def _part_offsets(case, seed):
    sizes = W.partition_sizes(np.random.default_rng([seed, 3]), case["texts"], case["parts"], 1.72)
    return np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)


def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(seed)


def _weights(shape):
    """The encoder's arrays in the fixed order, on the GPU, drawn as the
    workload module describes: N(0, 0.02), LayerNorm gamma 1 + N(0, 0.02)."""
    g = _gen(shape.d_model + shape.n_layers)
    dtype = torch.bfloat16 if shape.weight_dtype == "bf16" else torch.float32
    out = []
    for name, dims in W.weight_shapes(shape):
        w = torch.randn(dims, generator=g, device=DEV) * 0.02
        out.append((w + 1.0 if name.endswith("_g") else w).to(dtype))
    return out


_encoders = {}


def _encoder(name):
    if name not in _encoders:
        s = SHAPES[name]
        bf16 = s.weight_dtype == "bf16"
        desc = S.make_desc(s.n_layers, s.d_model, s.n_heads, s.d_ff, s.vocab_size, s.max_positions,
                           s.ln_eps, S.SURGE_WEIGHTS_BF16 if bf16 else S.SURGE_WEIGHTS_F32)
        host = [(w.view(torch.int16) if bf16 else w).cpu().numpy() for w in _weights(s)]
        host = [h.view(np.uint16) if bf16 else h for h in host]
        _encoders[name] = S.Encoder(desc, host, CHUNK_TOKENS)
    return _encoders[name]


def _linear_inputs(case, seed):
    """Activations and weights of one linear layer.  Epilogues 3, 4 and 6
    read the row statistics of the raw rows (partials of 64 features)."""
    g = _gen(seed)
    m, n, k, epi = case["m"], case["n"], case["k"], case["epi"]

    def randn(*dims):
        return torch.randn(dims, generator=g, device=DEV)

    p = {"x": randn(m, k).bfloat16(), "bias": randn(n) * 0.02}
    if epi in (2, 5, 6):
        p["res"] = randn(m, n).bfloat16()
    w = randn(n, k) * 0.02
    if epi in (3, 4):  # gamma of the input's LayerNorm is part of the weight
        w = w * (1 + 0.02 * randn(k))
    p["w"] = w.bfloat16()
    if epi in (3, 4):
        p["col_s"] = p["w"].double().sum(1).float()
    if epi in (3, 4, 6):
        rows = p["res"] if epi == 6 else p["x"]
        part = rows.float().view(m, -1, 64)
        p["stats_in"] = torch.stack([part.mean(2), part.var(2, unbiased=False)], 2) \
            .transpose(0, 1).contiguous()
    if epi == 6:
        p["gamma"], p["beta"] = 1 + 0.02 * randn(n), 0.02 * randn(n)
    return p


def prepare(case, seed):
    kind = case["kind"]
    st = {"kind": kind, "case": case}
    if kind == "linear":
        st.update(_linear_inputs(case, seed))
        st["y"] = torch.empty(case["m"], case["n"], dtype=torch.bfloat16, device=DEV)
        if case["epi"] >= 5:
            st["stats_out"] = torch.empty(case["n"] // 64, case["m"], 2, device=DEV)
        return st
    cu = _cu(case, seed)
    st["cu"] = cu
    t = int(cu[-1])
    if kind in ("encode", "stream"):
        enc = _encoder(case["shape"])
        d = enc.desc.d_model
        offs = _part_offsets(case, seed)
        st["enc"], st["offs"] = enc, offs
        tokens = torch.from_numpy(_tokens(cu, seed))
        if kind == "stream":
            st["tokens"] = tokens.pin_memory()
            st["out"] = torch.empty(case["texts"], d, pin_memory=True)
            if case["overlap"] == 1:
                st["copy_stream"] = torch.cuda.Stream()
                st["stream"] = torch.cuda.Stream()
            return st
        st["tokens"] = tokens.to(DEV)
        st["out"] = torch.empty(case["texts"], d, device=DEV)
        st["segs"] = S.segments_array([(int(offs[p]), int(offs[p + 1] - offs[p]), p, 0)
                                       for p in range(case["parts"])])
        st["sizes"] = np.diff(offs)
        st["ptrs"] = st["out"].data_ptr() + offs[:-1] * d * 4
        return st
    g = _gen(seed)
    if kind == "attention":
        d = case["heads"] * case["dh"]
        st["x"] = torch.randn(t, 3 * d, generator=g, device=DEV).bfloat16()
        st["y"] = torch.empty(t, d, dtype=torch.bfloat16, device=DEV)
        return st
    d = case["d"]
    st["gamma"] = 1 + 0.02 * torch.randn(d, generator=g, device=DEV)
    st["beta"] = 0.02 * torch.randn(d, generator=g, device=DEV)
    if kind == "embed":
        st["tokens"] = torch.from_numpy(_tokens(cu, seed)).to(DEV)
        st["word"] = (0.02 * torch.randn(W.BGE.vocab_size, d, generator=g, device=DEV)).bfloat16()
        st["pos"] = (0.02 * torch.randn(512, d, generator=g, device=DEV)).bfloat16()
        st["y"] = torch.empty(t, d, dtype=torch.bfloat16, device=DEV)
    else:
        st["x"] = torch.randn(t, d, generator=g, device=DEV).bfloat16()
        if kind == "layernorm":
            st["y"] = torch.empty_like(st["x"])
        else:
            st["y"] = torch.empty(case["texts"], d, device=DEV)
    return st


# ---------------------------------------------------------------------------
# One pass
# ---------------------------------------------------------------------------

def run(st):
    case, kind = st["case"], st["kind"]
    if kind == "encode":
        st["enc"].encode_superbatch(case["texts"], int(st["cu"][-1]), st["tokens"], st["cu"],
                                    st["segs"], st["ptrs"], st["sizes"])
        return st["out"]
    if kind == "stream":
        st["enc"].encode_all_streamed(case["texts"], st["tokens"], st["cu"], st["offs"],
                                      case["b_min"], case["n_max"], st["out"], case["overlap"],
                                      st.get("stream"), st.get("copy_stream"))
        return st["out"]
    if kind == "linear":
        m, n, k, epi = case["m"], case["n"], case["k"], case["epi"]
        if epi <= 2:
            S.surge_op_linear(m, n, k, st["x"], st["w"], st["bias"], st.get("res"), epi, st["y"])
            return st["y"]
        parts = 0 if epi == 5 else (n if epi == 6 else k) // 64
        S.surge_op_linear_ln_noalloc(m, n, k, st["x"], st["w"], st["bias"], st.get("res"), epi,
                                     st.get("stats_in"), parts, st.get("col_s"), st.get("gamma"),
                                     st.get("beta"), 1e-12, st.get("stats_out"), st["y"])
        return {"y": st["y"], "stats": st["stats_out"]} if epi >= 5 else st["y"]
    if kind == "attention":
        S.surge_op_attention(st["cu"], case["heads"], case["dh"], st["x"], st["y"])
    elif kind == "embed":
        S.surge_op_embed_ln(st["cu"], st["tokens"], st["word"], W.BGE.vocab_size, st["pos"], 512,
                            st["gamma"], st["beta"], 1e-12, case["d"], st["y"])
    elif kind == "layernorm":
        S.surge_op_layernorm(int(st["cu"][-1]), case["d"], st["x"], st["gamma"], st["beta"], 1e-12,
                             st["y"])
    else:
        S.surge_op_pool_l2(st["cu"], case["d"], st["x"], st["y"])
    return st["y"]


# ---------------------------------------------------------------------------
# What a pass cannot do without, and how far outputs may be off
# ---------------------------------------------------------------------------

def work(case):
    kind = case["kind"]
    if kind == "linear":
        m, n, k, epi = case["m"], case["n"], case["k"], case["epi"]
        b = 2 * (m * k + n * k + m * n) + 4 * n
        b += 2 * m * n if epi in (2, 5, 6) else 0
        b += 8 * m * ((n if epi == 6 else k) // 64) if epi in (3, 4, 6) else 0
        b += 8 * m * (n // 64) if epi >= 5 else 0
        return {"bytes": b, "flops": 2 * m * n * k}
    length = np.diff(_cu(case, 0)).astype(np.float64)
    t, t2, n = float(length.sum()), float((length * length).sum()), case["texts"]
    if kind in ("encode", "stream"):
        s = SHAPES[case["shape"]]
        d, f, layers = s.d_model, s.d_ff, s.n_layers
        per_layer = 4 * d * d + 2 * d * f
        gathered = min(t, s.vocab_size) * d * 2
        return {"bytes": 2 * layers * per_layer + gathered + 4 * t + 4 * n * d,
                "flops": layers * (2 * t * per_layer + 4 * d * t2)}
    if kind == "attention":
        d = case["heads"] * case["dh"]
        return {"bytes": 8 * t * d, "flops": 4 * d * t2}
    d = case["d"]
    if kind == "embed":
        return {"bytes": t * (4 + 2 * d) + 2 * d * min(t, W.BGE.vocab_size), "flops": 8 * t * d}
    if kind == "layernorm":
        return {"bytes": 4 * t * d, "flops": 8 * t * d}
    return {"bytes": 2 * t * d + 4 * n * d, "flops": t * d}


def tolerance(case):
    # Errors measured against `exact`, times about four: whole encodes 0.0037
    # to 0.0048 (bf16 weights and activations through every layer); one layer
    # 0.0017 (bf16 rounding of its output); pooling 6e-8 (fp32 throughout).
    kind = case["kind"]
    if kind in ("encode", "stream"):
        return {"rel": 2e-2, "max": 0.3}
    if kind == "pool":
        return {"rel": 5e-7, "max": 1e-5}
    return {"rel": 7e-3, "max": 0.05}


# ---------------------------------------------------------------------------
# The same results in 64 bits
# ---------------------------------------------------------------------------

def _ln64(v, gamma, beta, eps):
    mu = v.mean(-1, keepdim=True)
    var = ((v - mu) ** 2).mean(-1, keepdim=True)
    return (v - mu) / torch.sqrt(var + eps) * gamma.double() + beta.double()


def _gelu64(z):
    return 0.5 * z * (1 + torch.erf(z / math.sqrt(2.0)))


def _same_length(cu, most):
    """Groups of texts of one length, of at most `most` tokens: (length, text
    indices, their token rows as [texts, length])."""
    length = np.diff(cu)
    for n in np.unique(length):
        idx = np.nonzero(length == n)[0]
        step = max(1, most // int(n))
        for a in range(0, len(idx), step):
            part = idx[a:a + step]
            rows = torch.from_numpy(cu[part][:, None] + np.arange(n)[None]).to(DEV)
            yield int(n), torch.from_numpy(part).to(DEV), rows


def _attention64(qkv, heads, dh):
    """[B, L, 3 d] in float64 -> [B, L, d]."""
    b, n, _ = qkv.shape
    q, k, v = (x.reshape(b, n, heads, dh).permute(0, 2, 1, 3).reshape(b * heads, n, dh)
               for x in qkv.chunk(3, dim=2))
    s = torch.bmm(q, k.transpose(1, 2).contiguous()) / math.sqrt(dh)
    o = torch.bmm(torch.softmax(s, -1), v)
    return o.reshape(b, heads, n, dh).permute(0, 2, 1, 3).reshape(b, n, heads * dh)


def _encode64(case, seed):
    s = SHAPES[case["shape"]]
    w = [x.double() for x in _weights(s)]
    cu = _cu(case, seed)
    tokens = torch.from_numpy(_tokens(cu, seed)).to(DEV).long()
    out = torch.empty(case["texts"], s.d_model, dtype=torch.float64, device=DEV)
    for n, part, rows in _same_length(cu, 1 << 15):
        x = _ln64(w[0][tokens[rows]] + w[1][:n], w[2], w[3], s.ln_eps)
        for l in range(s.n_layers):
            wq, bq, wo, bo, g1, b1, w1, c1, w2, c2, g2, b2 = w[4 + 12 * l:16 + 12 * l]
            a = _attention64(x @ wq + bq, s.n_heads, s.d_head)
            x = _ln64(x + a @ wo + bo, g1, b1, s.ln_eps)
            x = _ln64(x + _gelu64(x @ w1 + c1) @ w2 + c2, g2, b2, s.ln_eps)
        e = x.mean(1)
        out[part] = e / e.norm(dim=1, keepdim=True).clamp_min(1e-12)
    return out


def _rows64(stats):
    """(mean, variance) of each row from its 64-feature partials [p, m, 2]."""
    st = stats.double()
    mu = st[..., 0].mean(0)
    return mu[:, None], (st[..., 1].mean(0) + ((st[..., 0] - mu) ** 2).mean(0))[:, None]


def _linear64(case, seed):
    p, epi, eps = _linear_inputs(case, seed), case["epi"], 1e-12
    m, n = case["m"], case["n"]
    y = torch.empty(m, n, dtype=torch.float64, device=DEV)
    stats = torch.empty(n // 64, m, 2, dtype=torch.float64, device=DEV)
    w = p["w"].double().t().contiguous()
    for a in range(0, m, 1 << 15):
        r = slice(a, min(m, a + (1 << 15)))
        v = p["x"][r].double() @ w
        if epi in (3, 4):
            mu, var = _rows64(p["stats_in"][:, r])
            v = (v - mu * p["col_s"].double()) / torch.sqrt(var + eps)
        v = v + p["bias"].double()
        if epi in (1, 4):
            v = _gelu64(v)
        if epi in (2, 5):
            v = v + p["res"][r].double()
        if epi == 6:
            mu, var = _rows64(p["stats_in"][:, r])
            v = v + (p["res"][r].double() - mu) / torch.sqrt(var + eps) * p["gamma"].double() \
                + p["beta"].double()
        y[r] = v
        if epi >= 5:
            part = v.view(v.shape[0], -1, 64)
            stats[:, r] = torch.stack([part.mean(2), part.var(2, unbiased=False)], 2).transpose(0, 1)
    return {"y": y, "stats": stats} if epi >= 5 else y


def exact(case, seed):
    kind = case["kind"]
    if kind in ("encode", "stream"):
        return _encode64(case, seed)
    if kind == "linear":
        return _linear64(case, seed)
    st = prepare(case, seed)
    if kind == "layernorm":
        return _ln64(st["x"].double(), st["gamma"], st["beta"], 1e-12)
    out = torch.empty(st["y"].shape, dtype=torch.float64, device=DEV)
    for n, part, rows in _same_length(st["cu"], 1 << 15):
        if kind == "attention":
            out[rows] = _attention64(st["x"][rows].double(), case["heads"], case["dh"])
        elif kind == "embed":
            v = st["word"][st["tokens"][rows].long()].double() + st["pos"][:n].double()
            out[rows] = _ln64(v, st["gamma"], st["beta"], 1e-12)
        else:
            e = st["x"][rows].double().mean(1)
            out[part] = e / e.norm(dim=1, keepdim=True).clamp_min(1e-12)
    return out
