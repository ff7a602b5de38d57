"""The work that a user of this framework has it do, as cases to be timed.

Every case goes through the public entry points (`binding.MarCache`,
`binding.MarHead` and the per-kernel calls), at the model sizes of
`workload.WORKLOADS` / `workload.HEADS`.  Five kinds:

decode     one refresh period of a decoding schedule on a whole stack: a full
           step and the cached steps that follow it, both pathways and
           conditional-only in turn, with the guidance after each
blocks     a few blocks of a stack: `full` steps, or two token-cached steps
           (there and back between two inputs)
head       one call of the per-token diffusion head: all sampling steps
linear     one matrix product with its bias (and GELU) on ragged sizes
attention  one attention call, every token a query or only some
selection  scores of the value rows and the selected rows

Inputs are random with the distributions of `workload`, drawn on the GPU from
the seed.  A cached step's input differs from the one before on n rows per
sequence, by noise of the rows' own size, so that which rows are selected
does not hang on rounding.
"""
from __future__ import annotations

import dataclasses
import math

import torch

from paper_2503_12450_amd import binding as B
from paper_2503_12450_amd.workload import HEADS, WORKLOADS, MarDims

DEV = "cuda"
SCALE = 4.0            # guidance scale of the decode and head cases
TDT = {"bf16": torch.bfloat16, "f32": torch.float32}


# ---------------------------------------------------------------------------
# The cases
# ---------------------------------------------------------------------------

def listed():
    return [
        # the headline workload: MAR-L, 64 images with both pathways, 50 rows
        # recomputed; a full step, then the alternating cached steps
        {"name": "decode_mar_l_64", "kind": "decode", "model": "mar-l", "images": 64, "n": 50, "dtype": "bf16"},
        # one image at a time (an interactive user): 24 blocks on 2 x 320 rows
        {"name": "decode_mar_b_1", "kind": "decode", "model": "mar-b", "images": 1, "n": 96, "dtype": "bf16"},
        # the fp32 path, one block, one image: the smallest step there is
        {"name": "decode_block_f32_1", "kind": "decode", "model": "block-f32", "images": 1, "n": 80, "dtype": "f32"},
        # dense blocks of the headline workload (refresh steps, the prefix)
        {"name": "blocks_full_mar_l", "kind": "blocks", "model": "mar-l", "slots": 128, "layers": 2, "prefix": 1,
         "n": 0, "full": True},
        # mostly cached blocks at the widest model (d_head 80), few rows each
        {"name": "blocks_cached_mar_h", "kind": "blocks", "model": "mar-h", "slots": 256, "layers": 12, "prefix": 1,
         "n": 32, "full": False},
        # long sequences: cached blocks whose attention reads 1088 keys
        {"name": "blocks_cached_hires", "kind": "blocks", "model": "mar-l-hires", "slots": 32, "layers": 8,
         "prefix": 1, "n": 218, "full": False},
        # the diffusion head on what a decoding step decodes on average (64
        # images, 256 tokens), with room for the largest step (7 per image)
        {"name": "head_mar_l_256", "kind": "head", "model": "mar-l", "tokens": 256, "max_tokens": 448},
        # the head for one image: the tokens of one late decoding step
        {"name": "head_mar_b_5", "kind": "head", "model": "mar-b", "tokens": 5, "max_tokens": 7},
        # the widest head on a large step (128 images)
        {"name": "head_mar_h_512", "kind": "head", "model": "mar-h", "tokens": 512, "max_tokens": 896},
        # a product whose sizes fit no tile: an MLP's first half on 1111 rows
        {"name": "linear_ragged", "kind": "linear", "m": 1111, "n": 3080, "k": 768, "gelu": True, "dtype": "bf16"},
        # every token a query, sequences of the high-resolution model
        {"name": "attention_hires", "kind": "attention", "slots": 32, "heads": 16, "d_head": 64, "seq": 1088,
         "per_slot": 1088, "dtype": "bf16"},
        # which rows to recompute, for a batch of sequences
        {"name": "selection_mar_l", "kind": "selection", "slots": 128, "heads": 16, "d_head": 64, "seq": 320,
         "n": 50, "dtype": "bf16"},
    ]


def _log(rng, lo, hi):
    """A whole number spread over the logarithm of [lo, hi]."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(("decode", "blocks", "blocks", "head", "head", "linear", "attention", "selection"))
    if kind == "decode":
        model = rng.choice(("mar-b", "mar-l", "mar-h", "block-f32"))
        most = {"mar-b": 64, "mar-l": 48, "mar-h": 24, "block-f32": 8}[model]
        return {"kind": kind, "model": model, "images": _log(rng, 1, most), "n": rng.randint(20, 110),
                "dtype": "f32" if model == "block-f32" else "bf16"}
    if kind == "blocks":
        model = rng.choice(("mar-b", "mar-l", "mar-h", "mar-l-hires"))
        most = {"mar-b": 128, "mar-l": 128, "mar-h": 160, "mar-l-hires": 40}[model]
        full = rng.random() < 0.3
        seq = WORKLOADS[model].dims.seq_len
        return {"kind": kind, "model": model, "slots": _log(rng, 1, most), "layers": 2 if full else rng.randint(2, 10),
                "prefix": 1, "n": 0 if full else _log(rng, seq // 20, seq // 3), "full": full}
    if kind == "head":
        model = rng.choice(("mar-b", "mar-l", "mar-h"))
        per = rng.randint(1, 7)
        images = _log(rng, 1, {"mar-b": 64, "mar-l": 64, "mar-h": 80}[model])
        return {"kind": kind, "model": model, "tokens": per * images, "max_tokens": 7 * images}
    if kind == "linear":
        return {"kind": kind, "m": _log(rng, 1, 20000), "n": 8 * _log(rng, 12, 640), "k": 64 * _log(rng, 4, 64),
                "gelu": rng.random() < 0.5, "dtype": rng.choice(("bf16", "bf16", "f32"))}
    if kind == "attention":
        seq = rng.choice((320, 320, 1088, _log(rng, 64, 1200)))
        return {"kind": kind, "slots": _log(rng, 1, 48), "heads": rng.choice((12, 16)),
                "d_head": rng.choice((64, 64, 80)), "seq": seq,
                "per_slot": seq if rng.random() < 0.5 else _log(rng, 10, seq), "dtype": "bf16"}
    seq = rng.choice((320, 1088, _log(rng, 64, 1200)))
    return {"kind": "selection", "slots": _log(rng, 1, 128), "heads": rng.choice((12, 16)), "d_head": 64, "seq": seq,
            "n": _log(rng, 1, seq), "dtype": rng.choice(("bf16", "bf16", "f32"))}


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------

def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed) * 7919 + 17)


def _normal(g, shape, std=1.0, dtype=torch.float32, mean=0.0):
    return (torch.randn(shape, generator=g, device=DEV) * std + mean).to(dtype)


def _dims(case):
    d = WORKLOADS[case["model"]].dims
    if case["kind"] == "decode":
        return dataclasses.replace(d, max_slots=2 * case["images"])
    return dataclasses.replace(d, max_slots=case["slots"], n_layers=case["layers"], full_prefix=case["prefix"])


def _block_weights(d: MarDims, g):
    D, F, t = d.d_model, d.d_mlp, TDT[d.dtype]
    std = 0.02
    return {"ln1_w": _normal(g, D, std, mean=1.0), "ln1_b": _normal(g, D, std),
            "qkv_w": _normal(g, (3 * D, D), std, t), "qkv_b": _normal(g, 3 * D, std),
            "proj_w": _normal(g, (D, D), std, t), "proj_b": _normal(g, D, std),
            "ln2_w": _normal(g, D, std, mean=1.0), "ln2_b": _normal(g, D, std),
            "fc1_w": _normal(g, (F, D), std, t), "fc1_b": _normal(g, F, std),
            "fc2_w": _normal(g, (D, F), std, t), "fc2_b": _normal(g, D, std)}


def _changed(x, n, g, slots=None):
    """x with n rows of each of the first `slots` sequences moved by N(0, 1)."""
    y = x.clone()
    k = x.shape[0] if slots is None else slots
    rows = torch.rand((k, x.shape[1]), generator=g, device=DEV).argsort(1)[:, :n]
    at = torch.arange(k, device=DEV)[:, None]
    y[at, rows] = (y[at, rows].float() + _normal(g, (k, n, x.shape[2]))).to(x.dtype)
    return y


def _step_inputs(case, d, g):
    x = [_normal(g, (d.max_slots, d.seq_len, d.d_model), 1.0, TDT[d.dtype])]
    if case["kind"] == "decode":
        # both pathways change on the two-pathway steps, the conditional
        # slots alone on the conditional-only ones
        for k in range(4):
            x.append(_changed(x[-1], case["n"], g, case["images"] if k % 2 else None))
    elif not case["full"]:
        x.append(_changed(x[0], case["n"], g))
    return x


def _head_dims(case):
    return dataclasses.replace(HEADS[case["model"]], max_rows=case["max_tokens"])


def _head_inputs(case, seed):
    hd, g, bf = _head_dims(case), _gen(seed), torch.bfloat16
    w, D, T, R, std = hd.width, hd.cond_dim, hd.token_dim, case["tokens"], 0.02
    W = {"z_w": _normal(g, (w, D), std, bf), "z_b": _normal(g, w, std),
         "t1_w": _normal(g, (w, hd.freq_dim), 0.1, bf), "t1_b": _normal(g, w, std),
         "t2_w": _normal(g, (w, w), std, bf), "t2_b": _normal(g, w, std),
         "in_w": _normal(g, (w, T), 0.25, bf), "in_b": _normal(g, w, std),
         "ada_w": _normal(g, (hd.n_mod * w, w), std, bf), "ada_b": _normal(g, hd.n_mod * w, std),
         "fc1_w": _normal(g, (hd.depth, w, w), std, bf), "fc1_b": _normal(g, (hd.depth, w), std),
         "fc2_w": _normal(g, (hd.depth, w, w), std, bf), "fc2_b": _normal(g, (hd.depth, w), std),
         "out_w": _normal(g, (T, w), 1.0 / math.sqrt(w), bf), "out_b": _normal(g, T, std)}
    n = 4 * case["max_tokens"]  # rows of the transformer's output
    yc = _normal(g, (n, D), 2.0)
    yu = _normal(g, (n, D), 2.0)
    rc = torch.randperm(n, generator=g, device=DEV)[:R].to(torch.int32)
    x0 = _normal(g, (R, T))
    xi = _normal(g, (hd.steps, R, T))
    return hd, W, yc, yu, rc, x0, xi


def _kernel_inputs(case, seed):
    g, t = _gen(seed), TDT[case["dtype"]]
    if case["kind"] == "linear":
        m, n, k = case["m"], case["n"], case["k"]
        return _normal(g, (m, k), 1.0, t), _normal(g, (n, k), 0.02, t), _normal(g, n, 0.02)
    if case["kind"] == "attention":
        b, h, s, dh = case["slots"], case["heads"], case["seq"], case["d_head"]
        return (_normal(g, (b * case["per_slot"], h * dh), 1.0, t), _normal(g, (b, h, s, dh), 1.0, t),
                _normal(g, (b, h, s, dh), 1.0, t))
    b, h, s, dh = case["slots"], case["heads"], case["seq"], case["d_head"]
    ref = _normal(g, (b, h, s, dh), 1.0, t)
    # every row moves by its own amount, as between two decoding steps
    amount = torch.rand((b, 1, s, 1), generator=g, device=DEV)
    cur = (ref.float() + amount * _normal(g, (b, h, s, dh))).to(t)
    return cur, ref


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("decode", "blocks"):
        d, g = _dims(case), _gen(seed)
        weights = [_block_weights(d, g) for _ in range(d.n_layers)]
        x = _step_inputs(case, d, g)
        cache = B.MarCache(d, weights, device=DEV)
        torch.cuda.synchronize()  # the weights were copied: the program drops its own
        cache._blocks = None
        st = {"case": case, "dims": d, "cache": cache, "x": x, "out": cache.output()}
        if kind == "decode":
            n, shape = case["images"], (case["images"], d.seq_len, d.d_model)
            st["sel"] = [torch.empty((n if k % 2 else 2 * n, case["n"]), dtype=torch.int32, device=DEV)
                         for k in range(4)]
            st["guided"] = [torch.empty(shape, device=DEV) for _ in range(5)]
            st["uncond"] = torch.empty(shape, device=DEV)
        elif not case["full"]:
            cache.step(x[0], B.MAR_FULL)
            st["sel"] = [torch.empty((case["slots"], case["n"]), dtype=torch.int32, device=DEV) for _ in range(2)]
            st["y"] = [torch.empty(x[0].shape, dtype=torch.float32, device=DEV) for _ in range(2)]
        return st
    if kind == "head":
        hd, W, yc, yu, rc, x0, xi = _head_inputs(case, seed)
        head = B.MarHead(hd, W, device=DEV)
        return {"case": case, "head": head, "args": (yc, yu, rc, rc, x0, xi), "x": torch.empty_like(x0)}
    a = _kernel_inputs(case, seed)
    st = {"case": case, "args": a}
    if kind == "linear":
        st["out"] = torch.empty((case["m"], case["n"]), dtype=a[0].dtype, device=DEV)
    elif kind == "attention":
        st["out"] = torch.empty_like(a[0])
    else:
        st["scores"] = torch.empty((case["slots"], case["seq"]), dtype=torch.float64, device=DEV)
        st["idx"] = torch.empty((case["slots"], case["n"]), dtype=torch.int32, device=DEV)
    return st


# ---------------------------------------------------------------------------
# One pass
# ---------------------------------------------------------------------------

def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "decode":
        c, x, sel, n, b = state["cache"], state["x"], state["sel"], case["n"], case["images"]
        y, guided = state["out"], state["guided"]
        c.step(x[0], B.MAR_FULL)
        c.cfg_combine(B.MAR_CFG_STORE, y[:b], y[b:], SCALE, guided[0])
        for k in range(4):
            if k % 2:
                c.step(x[k + 1][:b], B.MAR_TOKEN_CACHED, n, sel_idx=sel[k])
                c.cfg_combine(B.MAR_CFG_REUSE, y[:b], None, SCALE, guided[k + 1], state["uncond"])
            else:
                c.step(x[k + 1], B.MAR_TOKEN_CACHED, n, sel_idx=sel[k])
                c.cfg_combine(B.MAR_CFG_STORE, y[:b], y[b:], SCALE, guided[k + 1])
        return {"y": y, "guided": guided, "uncond": state["uncond"], "sel": sel}
    if kind == "blocks":
        c, x = state["cache"], state["x"]
        if case["full"]:
            c.step(x[0], B.MAR_FULL)
            return {"y": state["out"]}
        # there and back: the second step restores what the first one changed
        for k in range(2):
            c.step(x[1 - k], B.MAR_TOKEN_CACHED, case["n"], y=state["y"][k], sel_idx=state["sel"][k])
        return {"y": state["y"], "sel": state["sel"]}
    if kind == "head":
        state["head"].sample(*state["args"], SCALE, state["x"])
        return {"x": state["x"]}
    if kind == "linear":
        B.k_linear(case["dtype"], *state["args"], state["out"], gelu=case["gelu"])
        return state["out"]
    if kind == "attention":
        q, k, v = state["args"]
        B.k_attention(case["dtype"], q, k, v, state["out"], case["slots"], case["heads"], case["seq"], case["d_head"],
                      case["per_slot"])
        return state["out"]
    B.k_scores(case["dtype"], *state["args"], state["scores"])
    B.k_select(state["scores"], case["n"], state["idx"])
    return {"scores": state["scores"], "idx": state["idx"]}


# ---------------------------------------------------------------------------
# What a pass cannot do without
# ---------------------------------------------------------------------------

def _stack_work(d, slots, n):
    """(bytes, flops) of one step: a full one (n None), or a cached one."""
    D, F, S, L, P = d.d_model, d.d_mlp, d.seq_len, d.n_layers, d.full_prefix
    es = 2 if d.dtype == "bf16" else 4
    per_row = 2 * (4 * D * D + 2 * F * D)
    rows = slots * S
    weights = (4 * D * D + 2 * F * D) * es
    dense = rows * per_row + 4 * rows * S * D
    if n is None:
        # weights, the input, the caches and the scoring reference, the output
        return L * weights + rows * D * (es + 2 * (L - P) * es + es + 4), L * dense
    sel = slots * n
    flops = P * dense + (L - P) * (sel * per_row + 4 * sel * S * D) + (2 * rows * D * D if P == 0 else 0)
    # the cached keys and values are read by every cached block; n rows of
    # them and of the output are written; the reference is read and replaced
    bytes_ = L * weights + rows * D * (es + 2 * es + 2 * (L - P) * es) + sel * D * (2 * (L - P) * es + 4)
    return bytes_, flops


def work(case):
    kind = case["kind"]
    if kind in ("decode", "blocks"):
        d = _dims(case)
        if kind == "decode":
            b = case["images"]
            parts = [_stack_work(d, 2 * b, None)]
            parts += [_stack_work(d, b if k % 2 else 2 * b, case["n"]) for k in range(4)]
            out = b * d.seq_len * d.d_model * 4
            parts += [(4 * out, 0)] * 5
        elif case["full"]:
            parts = [_stack_work(d, case["slots"], None)]
        else:
            parts = [_stack_work(d, case["slots"], case["n"])] * 2
        return {"bytes": sum(p[0] for p in parts), "flops": sum(p[1] for p in parts)}
    if kind == "head":
        hd = _head_dims(case)
        w, T, R = hd.width, hd.token_dim, case["tokens"]
        mats = hd.n_mod * w * w + 2 * hd.depth * w * w + 2 * T * w
        bytes_ = 2 * (mats + w * hd.cond_dim) + hd.steps * w * 4 + 2 * R * hd.cond_dim * 4 + (hd.steps + 2) * R * T * 4
        return {"bytes": bytes_, "flops": 2 * 2 * R * (hd.steps * mats + w * hd.cond_dim)}
    es = 2 if case["dtype"] == "bf16" else 4
    if kind == "linear":
        m, n, k = case["m"], case["n"], case["k"]
        return {"bytes": (m * k + n * k + m * n) * es + 4 * n, "flops": 2 * m * n * k}
    b, hd_, s = case["slots"], case["heads"] * case["d_head"], case["seq"]
    if kind == "attention":
        q = case["per_slot"]
        return {"bytes": b * hd_ * es * (2 * q + 2 * s), "flops": 4 * b * q * s * hd_}
    return {"bytes": 2 * b * s * hd_ * es + 16 * b * s + 4 * b * case["n"], "flops": 6 * b * s * hd_}


def tolerance(case):
    """About four times the error that was measured against exact()."""
    kind, bf = case["kind"], case.get("dtype", "bf16") == "bf16"
    if kind == "decode":  # 0.0041; 4e-7
        return {"rel": 1.6e-2, "differ": 2e-3} if bf else {"rel": 1.6e-6, "differ": 2e-3}
    if kind == "blocks":  # 0.0030
        return {"rel": 1.2e-2, "differ": 2e-3}
    if kind == "head":    # 0.0029
        return {"rel": 1.2e-2}
    if kind == "linear":  # 0.0017; fp32 sums over up to 4096 products
        return {"rel": 7e-3} if bf else {"rel": 4e-6}
    if kind == "attention":  # 0.0023
        return {"rel": 9e-3}
    return {"rel": 1e-14, "differ": 0.0}  # scores are correctly rounded, rows whole numbers


# ---------------------------------------------------------------------------
# The same in 64 bits, in plain torch
# ---------------------------------------------------------------------------

def _ln64(x, eps, w=None, b=None):
    m = x.mean(-1, keepdim=True)
    v = (x - m).square().mean(-1, keepdim=True)
    y = (x - m) / (v + eps).sqrt()
    return y if w is None else y * w + b


def _gelu64(x):
    return 0.5 * x * (1.0 + torch.erf(x / math.sqrt(2.0)))


def _attend64(q, k, v):
    """q [b, h, n, d], k and v [b, h, s, d], a few sequences at a time."""
    out = torch.empty_like(q)
    step = max(1, int(2e8 // (q.shape[1] * q.shape[2] * k.shape[2])))
    for i in range(0, q.shape[0], step):
        j = slice(i, i + step)
        p = torch.matmul(q[j], k[j].transpose(-1, -2).contiguous()) / math.sqrt(q.shape[-1])
        out[j] = torch.matmul(torch.softmax(p, -1), v[j])
    return out


class _Stack64:
    """The cached step in 64 bits: per block the keys and values of every
    token, the value rows of the scoring block and the output."""

    def __init__(self, d, weights):
        self.d, self.w = d, [{k: v.double() for k, v in b.items()} for b in weights]
        self.kv = [None] * d.n_layers
        self.ref = self.y = None

    def heads(self, t, slots):
        return t.reshape(slots, -1, self.d.n_heads, self.d.d_head).transpose(1, 2).contiguous()

    def block(self, l, h, at=None, b=0):
        """Block l on h [b, n, D]; `at`: these rows of the cached block."""
        w, d, n = self.w[l], self.d, h.shape[0]
        qkv = torch.addmm(w["qkv_b"], _ln64(h, d.ln_eps, w["ln1_w"], w["ln1_b"]).reshape(-1, d.d_model),
                          w["qkv_w"].t())
        q, k, v = (self.heads(t, n) for t in qkv.split(d.d_model, 1))
        if at is not None:
            kc, vc = self.kv[l]
            i = at[:, None, :, None].expand(-1, d.n_heads, -1, d.d_head)
            kc[:n].scatter_(2, i, k)
            vc[:n].scatter_(2, i, v)
            k, v = kc[:n], vc[:n]
        o = _attend64(q, k, v).transpose(1, 2).reshape(-1, d.d_model)
        h = h + torch.addmm(w["proj_b"], o, w["proj_w"].t()).view(h.shape)
        f = _gelu64(torch.addmm(w["fc1_b"], _ln64(h, d.ln_eps, w["ln2_w"], w["ln2_b"]).reshape(-1, d.d_model),
                                w["fc1_w"].t()))
        return h + torch.addmm(w["fc2_b"], f, w["fc2_w"].t()).view(h.shape), k, v

    def values(self, h):
        w, d = self.w[0], self.d
        v = torch.addmm(w["qkv_b"][2 * d.d_model:], _ln64(h, d.ln_eps, w["ln1_w"], w["ln1_b"]).reshape(-1, d.d_model),
                        w["qkv_w"][2 * d.d_model:].t())
        return self.heads(v, h.shape[0])

    def full(self, x):
        h, d = x.double(), self.d
        for l in range(d.n_layers):
            h, k, v = self.block(l, h)
            if l >= d.full_prefix:
                self.kv[l] = (k, v)
            if l == max(d.full_prefix - 1, 0):
                self.ref = v.clone()
        self.y = h
        return h

    def cached(self, x, n):
        h, d, b = x.double(), self.d, x.shape[0]
        cur = self.values(h) if d.full_prefix == 0 else None
        for l in range(d.full_prefix):
            h, _, cur = self.block(l, h)
        a, r = (t.transpose(1, 2).reshape(b, d.seq_len, -1) for t in (cur, self.ref[:b]))
        s = (a * r).sum(-1) / (a.square().sum(-1) * r.square().sum(-1)).sqrt()
        at = s.argsort(dim=1, stable=True)[:, :n].sort(1).values
        self.ref[:b] = cur
        rows = at[:, :, None].expand(-1, -1, d.d_model)
        c = h.gather(1, rows)
        for l in range(d.full_prefix, d.n_layers):
            c, _, _ = self.block(l, c, at)
        self.y[:b].scatter_(1, rows, c)
        return at.to(torch.int32)


def _exact_steps(case, seed):
    d, g = _dims(case), _gen(seed)
    stack = _Stack64(d, [_block_weights(d, g) for _ in range(d.n_layers)])
    x = _step_inputs(case, d, g)
    if case["kind"] == "blocks":
        y = stack.full(x[0])
        if case["full"]:
            return {"y": y}
        ys, sel = [], []
        for k in range(2):
            sel.append(stack.cached(x[1 - k], case["n"]))
            ys.append(stack.y.clone())
        return {"y": ys, "sel": sel}
    b, y, guided, sel, stored, unc = case["images"], stack.full(x[0]), [], [], None, None
    for k in range(5):
        if k:
            sel.append(stack.cached(x[k] if k % 2 else x[k][:b], case["n"]))
        if k in (0, 1, 3):
            u = y[b:]
            stored = u - y[:b]
        else:
            u = y[:b] + stored
            unc = u.clone()
        guided.append(u + SCALE * (y[:b] - u))
    return {"y": y, "guided": guided, "uncond": unc, "sel": sel}


def _exact_head(case, seed):
    hd, W, yc, yu, rc, x, xi = _head_inputs(case, seed)
    W = {k: v.double() for k, v in W.items()}
    w, R, S = hd.width, case["tokens"], hd.steps
    lin = torch.addmm
    silu = torch.nn.functional.silu
    f64 = {"dtype": torch.float64, "device": DEV}
    kept = torch.tensor([i * hd.train_steps // S for i in range(S)], device=DEV)
    f32 = torch.tensor([hd.beta_start, hd.beta_end], dtype=torch.float32).double().tolist()
    betas = torch.linspace(f32[0], f32[1], hd.train_steps, **f64)
    abar = torch.cumprod(1.0 - betas, 0)[kept]
    before = torch.cat([torch.ones(1, **f64), abar[:-1]])
    beta = 1.0 - abar / before
    sigma = (beta * (1.0 - before) / (1.0 - abar)).sqrt()
    half = hd.freq_dim // 2
    f = torch.exp(-math.log(10000.0) * torch.arange(half, **f64) / half)
    a = kept.double()[:, None] * f
    e = lin(W["t2_b"], silu(lin(W["t1_b"], torch.cat([a.cos(), a.sin()], 1), W["t1_w"].t())), W["t2_w"].t())
    i = rc.long()
    c = lin(W["z_b"], torch.cat([yc[i], yu[i]]).double(), W["z_w"].t())
    x = x.double()
    for t in reversed(range(S)):
        m = lin(W["ada_b"], silu(c + e[t]), W["ada_w"].t()).view(2 * R, hd.n_mod, w)
        h = lin(W["in_b"], x, W["in_w"].t()).repeat(2, 1)
        for k in range(hd.depth):
            u = _ln64(h, hd.ln_eps) * (1.0 + m[:, 3 * k + 1]) + m[:, 3 * k]
            u = silu(lin(W["fc1_b"][k], u, W["fc1_w"][k].t()))
            h = h + m[:, 3 * k + 2] * lin(W["fc2_b"][k], u, W["fc2_w"][k].t())
        u = _ln64(h, hd.ln_eps) * (1.0 + m[:, 3 * hd.depth + 1]) + m[:, 3 * hd.depth]
        eps = lin(W["out_b"], u, W["out_w"].t())
        eps = eps[R:] + SCALE * (eps[:R] - eps[R:])
        x = (x - beta[t] / (1.0 - abar[t]).sqrt() * eps) / (1.0 - beta[t]).sqrt()
        if t:
            x = x + sigma[t] * xi[t].double()
    return {"x": x}


def exact(case, seed):
    kind = case["kind"]
    if kind in ("decode", "blocks"):
        return _exact_steps(case, seed)
    if kind == "head":
        return _exact_head(case, seed)
    if kind == "linear":
        a, w, b = (t.double() for t in _kernel_inputs(case, seed))
        y = torch.addmm(b, a, w.t())
        return _gelu64(y) if case["gelu"] else y
    if kind == "attention":
        q, k, v = (t.double() for t in _kernel_inputs(case, seed))
        b, h, dh = case["slots"], case["heads"], case["d_head"]
        q = q.view(b, case["per_slot"], h, dh).transpose(1, 2).contiguous()
        return _attend64(q, k, v).transpose(1, 2).reshape(-1, h * dh)
    a, r = (t.double().transpose(1, 2).reshape(case["slots"], case["seq"], -1) for t in _kernel_inputs(case, seed))
    s = (a * r).sum(-1) / (a.square().sum(-1) * r.square().sum(-1)).sqrt()
    return {"scores": s, "idx": s.argsort(dim=1, stable=True)[:, :case["n"]].sort(1).values.to(torch.int32)}
