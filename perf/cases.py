"""Workloads of this package, from the smallest call to the largest: what a program that encodes RL
states with a frozen ternary backbone and trains the heads on top of it has the library do.

`listed()` are the sizes the package's own benchmark and tests quote, `draw(rng)` gives others of the
same ranges.  `prepare` makes weights and inputs on the GPU from a seed (masters ~ N(0, 0.02^2) through
the library's own quantiser, gains 1 + 0.1 N(0, 1), activations N(0, 1), token ids uniform), `run` is one
pass through the public entry points, `work` what a pass cannot do without, `tolerance` how far another
correct implementation of the same arithmetic may be off.

Kinds of case
  linear    one BitLinear layer on a batch of tokens (ternary or int8 weights)
  pair      decode: 1 - 4 tokens up and down through two BitLinear layers, one call each
  batch     many such products of one shape queued and streamed by one call
  ffn       one feed-forward block
  chain     one agent step: state vectors -> text -> token ids -> encoder -> heads
  encoder   token ids already on the GPU -> encoder -> heads (padded, or stored back to back)
  ppo       advantages and one update of the heads on a cached rollout
  quantise  loading: every matrix of one backbone layer from fp32 masters to packed weights
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2604_24273_amd import binding as B
from paper_2604_24273_amd import runtime as R
from paper_2604_24273_amd import synth

EPS = 1e-5
SHAPES = {"2b": synth.SHAPE_2B, "3b": synth.SHAPE_3B}


# ---------------------------------------------------------------- the cases

def listed():
    return [
        # a layer on the tokens of one short state: a call of microseconds
        {"name": "layer_16", "kind": "linear", "m": 16, "n": 2048, "k": 2048, "dtype": "f32", "residual": False,
         "weights": "ternary"},
        # decoding: one token through the up and the down matrix, one call each
        {"name": "decode_pair", "kind": "pair", "m": 1, "d": 2560, "f": 6912, "dtype": "f32"},
        # the same products, many queued: every weight byte read once
        {"name": "decode_batch_256", "kind": "batch", "m": 1, "d": 2560, "f": 6912, "count": 256, "dtype": "f32"},
        # one block on a few hundred tokens, activations in bf16
        {"name": "ffn_256", "kind": "ffn", "m": 256, "d": 2560, "f": 6912, "dtype": "bf16"},
        # an agent acting in one environment: one 25-dimensional state, 27 tokens
        {"name": "agent_step", "kind": "chain", "shape": "2b", "states": 1, "dims": 25},
        # vectorised environments: a few dozen states of different lengths, no padding
        {"name": "states_64", "kind": "encoder", "shape": "2b", "states": 64, "lo": 15, "hi": 40, "layout": "packed",
         "weights": "ternary"},
        # the headline batch: states padded to one length
        {"name": "encode_64x128", "kind": "encoder", "shape": "2b", "states": 64, "lo": 128, "hi": 128,
         "layout": "uniform", "weights": "ternary"},
        # a rollout's worth of states encoded at once
        {"name": "states_1024", "kind": "encoder", "shape": "2b", "states": 1024, "lo": 15, "hi": 40, "layout": "packed",
         "weights": "ternary"},
        # large-batch prefill of long states at the wider shape
        {"name": "prefill_64x512", "kind": "encoder", "shape": "3b", "states": 64, "lo": 512, "hi": 512,
         "layout": "uniform", "weights": "ternary"},
        # the higher-precision critic: int8 weights, three value heads averaged
        {"name": "critic_int8_64x128", "kind": "encoder", "shape": "2b", "states": 64, "lo": 128, "hi": 128,
         "layout": "uniform", "weights": "int8"},
        # training: one update of both heads on a 2048-step rollout, four epochs of 64-step mini-batches
        {"name": "ppo_2048", "kind": "ppo", "steps": 2048, "envs": 1, "epochs": 4, "batch": 64, "hidden": "256",
         "d": 2560, "actions": 18},
        # loading a backbone: the seven matrices of one layer
        {"name": "quantise_layer", "kind": "quantise", "shape": "2b", "weights": "ternary"},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["linear", "linear", "pair", "batch", "ffn", "ffn", "chain", "encoder", "encoder", "encoder", "ppo",
                       "quantise"])
    dtype = rng.choice(["f32", "bf16"])
    weights = rng.choice(["ternary", "ternary", "int8"])
    if kind == "linear":
        return {"kind": kind, "m": _log(rng, 5, 8192), "n": _log(rng, 128, 9216), "k": 8 * _log(rng, 64, 1152),
                "dtype": dtype, "residual": rng.random() < 0.5, "weights": weights}
    if kind == "pair":
        return {"kind": kind, "m": rng.randint(1, 4), "d": 8 * rng.randint(64, 480), "f": 8 * rng.randint(128, 1152),
                "dtype": dtype}
    if kind == "batch":
        return {"kind": kind, "m": rng.randint(1, 4), "d": 8 * rng.randint(128, 400), "f": 8 * rng.randint(256, 1080),
                "count": _log(rng, 8, 256), "dtype": dtype}
    if kind == "ffn":
        return {"kind": kind, "m": _log(rng, 5, 8192), "d": 8 * rng.randint(128, 400), "f": 8 * rng.randint(256, 1080),
                "dtype": dtype}
    if kind == "chain":
        return {"kind": kind, "shape": "2b", "states": _log(rng, 1, 32), "dims": rng.randint(13, 38)}
    if kind == "encoder":
        shape = rng.choice(["2b", "2b", "3b"])
        hi = _log(rng, 16, 512)
        layout = rng.choice(["packed", "uniform", "padded"])
        lo = hi if layout == "uniform" else rng.randint(max(1, hi // 3), hi)
        most = 24576 if shape == "2b" else 16384
        return {"kind": kind, "shape": shape, "states": _log(rng, 2, max(3, most // hi)), "lo": lo, "hi": hi,
                "layout": layout, "weights": weights}
    if kind == "ppo":
        batch = _log(rng, 16, 256)
        return {"kind": kind, "steps": rng.randint(4, 32) * batch // 4 * 4, "envs": rng.choice([1, 2, 4]), "epochs": rng.randint(1, 4),
                "batch": batch, "hidden": rng.choice(["64", "256", "256,128"]), "d": rng.choice([1024, 2560, 3200]),
                "actions": rng.randint(2, 24)}
    # a layer of a backbone of another size
    return {"kind": kind, "d": 8 * rng.randint(64, 400), "dkv": 8 * rng.randint(16, 64), "f": 8 * rng.randint(128, 1080),
            "weights": weights}


# ---------------------------------------------------------------- making weights and inputs

class _Draw:
    """Seeded normal tensors on the GPU."""

    def __init__(self, seed):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(seed)

    def normal(self, *shape, scale=1.0, shift=0.0, dtype=torch.float32):
        t = torch.randn(*shape, generator=self.g, device="cuda", dtype=torch.float32)
        if scale != 1.0:
            t.mul_(scale)
        if shift != 0.0:
            t.add_(shift)
        return t.to(dtype)

    def weight(self, n, k):
        return self.normal(n, k, scale=synth.W_STD)

    def gain(self, n):
        return self.normal(n, scale=0.1, shift=1.0)


def _dtype(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float32


def _lengths(case, rng):
    return rng.integers(case["lo"], case["hi"] + 1, size=case["states"]).astype(np.int32)


def _layer_matrices(d, dq, dkv, f):
    return [("q", dq, d), ("k", dkv, d), ("v", dkv, d), ("o", d, dq), ("gate", f, d), ("up", f, d), ("down", d, f)]


def _backbone(draw, shape, int8):
    """A frozen encoder: packed weights of every layer, gains, embedding table, and the struct the library takes."""
    d, f = shape.d, shape.f
    dq, dkv = shape.n_heads * shape.head_dim, shape.n_kv_heads * shape.head_dim
    keep = []
    layers = (B.brl_layer_weights * shape.n_layers)()
    for l in range(shape.n_layers):
        m = {name: R.quantize_linear(draw.weight(n, k), EPS, int8=int8) for name, n, k in _layer_matrices(d, dq, dkv, f)}
        g = {name: draw.gain(n) for name, n in (("attn", d), ("attn_sub", dq), ("ffn", d), ("ffn_sub", f))}
        s = layers[l]
        s.attn_norm_g, s.attn_subln_g = g["attn"].data_ptr(), g["attn_sub"].data_ptr()
        s.wq_packed, s.wq_beta = m["q"].packed.data_ptr(), m["q"].beta.data_ptr()
        s.wk_packed, s.wk_beta = m["k"].packed.data_ptr(), m["k"].beta.data_ptr()
        s.wv_packed, s.wv_beta = m["v"].packed.data_ptr(), m["v"].beta.data_ptr()
        s.wo_packed, s.wo_beta = m["o"].packed.data_ptr(), m["o"].beta.data_ptr()
        s.ffn = B.make_ffn_weights(g["ffn"], m["gate"].packed, m["gate"].beta, m["up"].packed, m["up"].beta, g["ffn_sub"],
                                   m["down"].packed, m["down"].beta)
        keep.append((m, g))
    embedding = torch.randn(shape.vocab, d, generator=draw.g, device="cuda", dtype=torch.bfloat16)
    final_g = draw.gain(d)
    keep += [embedding, final_g, layers]
    enc = B.brl_encoder(shape.n_layers, d, shape.n_heads, shape.n_kv_heads, shape.head_dim, f, shape.vocab, shape.rope_theta,
                        EPS, EPS, B.BRL_ATTN_MFMA, B.BRL_W_INT8 if int8 else B.BRL_W_TERNARY, embedding.data_ptr(),
                        final_g.data_ptr(), layers)
    return enc, keep


def _mlp(draw, dims):
    ws = [draw.normal(o, i, scale=1.0 / math.sqrt(i)) for i, o in zip(dims[:-1], dims[1:])]
    bs = [draw.normal(o, scale=0.1) for o in dims[1:]]
    return B.make_mlp(ws, bs, B.BRL_ACT_TANH)


def _arena(*counts):
    """One fp32 buffer cut into contiguous 16-byte aligned pieces: the outputs of a pass in one tensor."""
    starts = [0]
    for c in counts:
        starts.append(starts[-1] + (c + 3) // 4 * 4)
    flat = torch.zeros(starts[-1], dtype=torch.float32, device="cuda")
    return flat, [flat[a:a + c] for a, c in zip(starts, counts)]


def _prepare_encoder(case, seed):
    shape, int8 = SHAPES[case["shape"]], case.get("weights") == "int8"
    draw, rng = _Draw(seed), np.random.default_rng(seed)
    enc, keep = _backbone(draw, shape, int8)
    n = case["states"]
    s = {"enc": enc, "keep": keep, "n": n}
    if case["kind"] == "chain":
        s["vectors"] = rng.normal(0.0, 2.5, size=(n, case["dims"])).astype(np.float32)
        s["vocab"] = shape.vocab
        s["hi"] = case["dims"] + 2
        s["ws"] = R.device_bytes(B.brl_encoder_packed_workspace_bytes(enc, n, n * s["hi"], s["hi"]))
    else:
        lens = _lengths(case, rng)
        s["hi"] = case["hi"]
        if case["layout"] == "packed":
            cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
            s["hi"] = int(lens.max())
            s["cu_host"], s["cu"] = cu, R.dev(cu)
            s["ids"] = torch.randint(0, shape.vocab, (int(cu[-1]),), generator=draw.g, device="cuda", dtype=torch.int32)
            s["ws"] = R.device_bytes(B.brl_encoder_packed_workspace_bytes(enc, n, int(cu[-1]), s["hi"]))
        else:
            s["lengths"] = R.dev(lens) if case["layout"] == "padded" else None
            s["ids"] = torch.randint(0, shape.vocab, (n, case["hi"]), generator=draw.g, device="cuda", dtype=torch.int32)
            s["ws"] = R.device_bytes(B.brl_encoder_workspace_bytes(enc, n, case["hi"]))
    if int8:       # a critic: three value heads and their mean
        mlps = [_mlp(draw, [shape.d, 256, 1]) for _ in range(3)]
        s["keep"].append(mlps)
        s["members"] = B.make_mlp_array([m for m, _ in mlps])
        s["flat"], (h, each, mean) = _arena(n * shape.d, 3 * n, n)
        s["h"], s["each"], s["mean"] = h.view(n, shape.d), each.view(3, n), mean
        s["head_ws"] = R.device_bytes(B.brl_value_ensemble_workspace_bytes(s["members"], 3, n))
    else:          # an actor: policy logits and a value
        pol, val = _mlp(draw, [shape.d, 256, shape.n_actions]), _mlp(draw, [shape.d, 256, 1])
        s["keep"] += [pol, val]
        s["head"] = B.brl_head(pol[0], val[0])
        s["flat"], (h, logits, value) = _arena(n * shape.d, n * shape.n_actions, n)
        s["h"], s["logits"], s["value"] = h.view(n, shape.d), logits.view(n, shape.n_actions), value
        s["head_ws"] = R.device_bytes(B.brl_head_workspace_bytes(s["head"], n))
    return s


def _prepare_batch(case, seed):
    draw = _Draw(seed)
    d, f, m, count = case["d"], case["f"], case["m"], case["count"]
    # a few matrices go through the quantiser, the rest are copies in buffers of their own: every product
    # reads memory that no other product reads
    up = [R.quantize_linear(draw.weight(f, d), EPS) for _ in range(min(4, count))]
    down = [R.quantize_linear(draw.weight(d, f), EPS) for _ in range(min(4, count))]
    s = {"m": m, "d": d, "f": f, "count": count, "dtype": B.BRL_BF16 if case["dtype"] == "bf16" else B.BRL_F32}
    s["x"] = draw.normal(count, m, d, dtype=_dtype(case))
    s["h"] = torch.zeros(count, m, f, device="cuda")
    s["y"] = torch.zeros(count, m, d, device="cuda")
    ptrs = lambda ts: torch.tensor([t.data_ptr() for t in ts], dtype=torch.int64, device="cuda")  # noqa: E731
    for name, ws in (("up", up), ("down", down)):
        blobs = [ws[i].packed if i < len(ws) else ws[i % len(ws)].packed.clone() for i in range(count)]
        s[name + "_blobs"], s[name + "_ws"] = blobs, ws
        s[name] = ptrs(blobs)
        s[name + "_beta"] = ptrs([ws[i % len(ws)].beta for i in range(count)])
    s["xp"], s["hp"], s["yp"] = ptrs(list(s["x"])), ptrs(list(s["h"])), ptrs(list(s["y"]))
    return s


def _prepare_ppo(case, seed):
    draw, rng = _Draw(seed), np.random.default_rng(seed)
    n, envs, d, a = case["steps"], case["envs"], case["d"], case["actions"]
    hidden = [int(v) for v in case["hidden"].split(",")]
    policy = synth.mlp_params(seed, 200, [d] + hidden + [a])
    value = synth.mlp_params(seed, 300, [d] + hidden + [1])
    t = n // envs
    return {"trainer": R.PPOTrainer(policy, value), "batch": case["batch"],
            "h": draw.normal(n, d, scale=0.5),
            "actions": torch.randint(0, a, (n,), generator=draw.g, device="cuda", dtype=torch.int32),
            "logp": draw.normal(n, scale=0.15, shift=math.log(1.0 / a)),
            "rewards": draw.normal(envs, t), "values": draw.normal(envs, t, scale=0.7),
            "dones": (torch.rand(envs, t, generator=draw.g, device="cuda") < 0.03).float(),
            "last": draw.normal(envs, scale=0.7),
            "perm": R.dev(np.stack([rng.permutation(n) for _ in range(case["epochs"])]).astype(np.int32))}


def _quantise_matrices(case):
    if "shape" in case:
        sh = SHAPES[case["shape"]]
        return _layer_matrices(sh.d, sh.n_heads * sh.head_dim, sh.n_kv_heads * sh.head_dim, sh.f)
    return _layer_matrices(case["d"], case["d"], case["dkv"], case["f"])


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("chain", "encoder"):
        s = _prepare_encoder(case, seed)
    elif kind == "batch":
        s = _prepare_batch(case, seed)
    elif kind == "ppo":
        s = _prepare_ppo(case, seed)
    elif kind == "linear":
        draw, (m, n, k) = _Draw(seed), (case["m"], case["n"], case["k"])
        s = {"m": m, "n": n, "k": k, "int8": case["weights"] == "int8",
             "w": R.quantize_linear(draw.weight(n, k), EPS, int8=case["weights"] == "int8"),
             "x": draw.normal(m, k, dtype=_dtype(case)), "y": torch.zeros(m, n, device="cuda"),
             "residual": draw.normal(m, n) if case["residual"] else None,
             "ws": R.device_bytes(B.brl_bitlinear_workspace_bytes(m, n, k))}
    elif kind == "pair":
        draw, (m, d, f) = _Draw(seed), (case["m"], case["d"], case["f"])
        s = {"m": m, "d": d, "f": f, "up": R.quantize_linear(draw.weight(f, d), EPS),
             "down": R.quantize_linear(draw.weight(d, f), EPS), "x": draw.normal(m, d, dtype=_dtype(case)),
             "h": torch.zeros(m, f, device="cuda"), "y": torch.zeros(m, d, device="cuda"),
             "ws": R.device_bytes(max(B.brl_bitlinear_workspace_bytes(m, f, d), B.brl_bitlinear_workspace_bytes(m, d, f)))}
    elif kind == "ffn":
        draw, (m, d, f) = _Draw(seed), (case["m"], case["d"], case["f"])
        g = [draw.gain(d), draw.gain(f)]
        w = [R.quantize_linear(draw.weight(*nk), EPS) for nk in ((f, d), (f, d), (d, f))]
        s = {"m": m, "d": d, "f": f, "keep": (g, w), "x": draw.normal(m, d, dtype=_dtype(case)),
             "w": B.make_ffn_weights(g[0], w[0].packed, w[0].beta, w[1].packed, w[1].beta, g[1], w[2].packed, w[2].beta),
             "y": torch.zeros(m, d, device="cuda"), "ws": R.device_bytes(B.brl_ffn_workspace_bytes(m, d, f))}
    elif kind == "quantise":
        draw = _Draw(seed)
        s = {"masters": [draw.weight(n, k) for _, n, k in _quantise_matrices(case)], "int8": case["weights"] == "int8"}
    else:
        raise ValueError("unknown kind %r" % kind)
    s["kind"] = kind
    return s


# ---------------------------------------------------------------- one pass

def run(s):
    kind = s["kind"]
    if kind == "linear":
        f = B.bitlinear_int8_forward if s["int8"] else B.bitlinear_forward
        f(s["w"].packed, s["w"].beta, s["n"], s["k"], s["x"], s["m"], EPS, s["y"], s["residual"], None, None, None, s["ws"])
        return s["y"]
    if kind == "pair":
        m, d, f = s["m"], s["d"], s["f"]
        B.bitlinear_forward(s["up"].packed, s["up"].beta, f, d, s["x"], m, EPS, s["h"], None, None, None, None, s["ws"])
        B.bitlinear_forward(s["down"].packed, s["down"].beta, d, f, s["h"], m, EPS, s["y"], None, None, None, None, s["ws"])
        return s["h"], s["y"]
    if kind == "batch":
        m, d, f, count = s["m"], s["d"], s["f"], s["count"]
        B.bitlinear_forward_batch(s["up"], s["up_beta"], f, d, s["xp"], s["dtype"], m, EPS, s["hp"], count)
        B.bitlinear_forward_batch(s["down"], s["down_beta"], d, f, s["hp"], B.BRL_F32, m, EPS, s["yp"], count)
        return s["h"], s["y"]
    if kind == "ffn":
        B.ffn_block_forward(s["w"], s["x"], s["m"], s["d"], s["f"], EPS, EPS, s["y"], s["ws"])
        return s["y"]
    if kind == "quantise":
        out = [R.quantize_linear(w, EPS, int8=s["int8"]) for w in s["masters"]]
        return [(p.packed, p.beta) for p in out]
    if kind == "ppo":
        tr = s["trainer"]
        adv, ret = R.gae(s["rewards"], s["values"], s["dones"], s["last"], 0.99, 0.95)
        stats = tr.update(s["h"], s["actions"], s["logp"], adv.view(-1), ret.view(-1), s["perm"], s["batch"])
        return {"params": tr.params, "m": tr.adam_m, "v": tr.adam_v, "adv": adv, "returns": ret, "stats": stats}
    n = s["n"]
    if kind == "chain":
        ids, cu = B.serialize_states(s["vectors"], s["vocab"])
        B.encoder_forward_packed(s["enc"], torch.from_numpy(ids).cuda(), torch.from_numpy(cu).cuda(), cu, n, s["hi"], s["h"],
                                 s["ws"])
    elif "cu" in s:
        B.encoder_forward_packed(s["enc"], s["ids"], s["cu"], s["cu_host"], n, s["hi"], s["h"], s["ws"])
    else:
        B.encoder_forward(s["enc"], s["ids"], n, s["hi"], s["lengths"], s["h"], s["ws"])
    if "members" in s:
        B.value_ensemble_forward(s["members"], 3, s["h"], n, s["mean"], s["each"], s["head_ws"])
    else:
        B.policy_value_head(s["head"], s["h"], n, s["logits"], s["value"], s["head_ws"])
    return s["flat"]


# ---------------------------------------------------------------- what a pass cannot do without

def _packed(n, k, int8=False):
    return n * k / (1 if int8 else 4)


def work(case):
    kind = case["kind"]
    xb = 2 if case.get("dtype") == "bf16" else 4
    int8 = case.get("weights") == "int8"
    if kind == "linear":
        m, n, k = case["m"], case["n"], case["k"]
        return {"bytes": _packed(n, k, int8) + m * k * xb + m * n * 4 * (2 if case["residual"] else 1), "flops": 2 * m * n * k}
    if kind in ("pair", "batch"):
        m, d, f, c = case["m"], case["d"], case["f"], case.get("count", 1)
        return {"bytes": c * (2 * _packed(f, d) + m * d * xb + m * f * 4 + m * d * 4), "flops": c * 4 * m * d * f}
    if kind == "ffn":
        m, d, f = case["m"], case["d"], case["f"]
        return {"bytes": 3 * _packed(f, d) + m * d * (xb + 4) + 4 * (d + f), "flops": 6 * m * d * f}
    if kind == "quantise":
        total = sum(n * k for _, n, k in _quantise_matrices(case))
        return {"bytes": total * 4 + _packed(total, 1, int8), "flops": 2 * total}
    if kind == "ppo":
        n, d, a = case["steps"], case["d"], case["actions"]
        hidden = [int(v) for v in case["hidden"].split(",")]
        count = sum(i * o for out in (a, 1) for i, o in zip([d] + hidden, hidden + [out]))
        seen = case["epochs"] * (n // case["batch"]) * case["batch"]
        return {"bytes": n * d * 4 + 6 * count * 4, "flops": 6 * seen * count}
    sh = SHAPES[case["shape"]]
    if kind == "chain":
        mean = case["dims"] + 2
        tokens, squares = case["states"] * mean, case["states"] * mean * mean
    else:
        lo, hi = case["lo"], case["hi"]
        mean = (lo + hi) / 2
        square = mean * mean + ((hi - lo + 1) ** 2 - 1) / 12
        tokens, squares = case["states"] * mean, case["states"] * square
    dq, dkv = sh.n_heads * sh.head_dim, sh.n_kv_heads * sh.head_dim
    macs = sum(n * k for _, n, k in _layer_matrices(sh.d, dq, dkv, sh.f))
    return {"bytes": sh.n_layers * _packed(macs, 1, int8) + tokens * (4 + 2 * sh.d) + case["states"] * sh.d * 4 + 2 * 256 * sh.d * 4,
            "flops": sh.n_layers * (2 * tokens * macs + 2 * squares * dq)}


def tolerance(case):
    kind = case["kind"]
    if kind in ("linear", "pair", "batch", "quantise"):
        # integer sums are exact; what is left is the order of two fp32 multiplications (1e-7)
        return {"rel": 1e-6}
    if kind == "ffn":
        # a norm statistic summed in another order can move the fp32 factor of a token by one unit in the last
        # place, and that the rounding of a few of its int8 codes: 2e-8 to 4e-5 seen against sums in another order
        return {"rel": 2e-4}
    if kind == "ppo":
        # against the same update in 64 bits throughout: 4e-7 on parameters, 6e-7 and 1.2e-5 on the moments
        # (single parameters up to 2e-4 of the root mean square)
        return {"rel": 5e-5, "max": 1e-3}
    # 26 to 30 layers that each round to int8 amplify the last bits of the attention sums: the two attention
    # kernels of the library, both accurate to 5e-7 per layer, leave 0.012 to 0.041 between the outputs here
    # (0.06 to 0.26 on single values)
    return {"rel": 0.03, "max": 0.5}
