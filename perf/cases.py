"""The work that a user of this library has it do, as cases that can be measured: which calls, on which sizes, with what
inputs, what a pass cannot do without, and what a correct pass returns.

Every pass goes through the public Python entry points.  A state holds what a training program has in hand before the
call: parameters, gradients, the 4-bit optimizer state of a run in its hundredth step, the plan or the workspace.  The
initial states and the 64-bit expectations are written in plain torch from the definitions (block-wise normalization
with block 128, rank-1 normalization, the two 16-entry maps), with none of the library's code.

A case is one of five kinds:
  step      one optimizer step on one tensor (single-tensor entry points)
  plan      one optimizer step on a transformer's whole parameter set (multi-tensor plan)
  optim     one optimizer step on a small vision model through the torch.optim-style front end
  convert   both moments of one tensor compressed to 4 bits and decompressed again (checkpoints, conversion)
  ablation  a second moment through one map and rounding under every normalization (quantizer study)
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2309_01507_amd as lpmm

DEV = "cuda:0"
LR, BETA1, BETA2, EPS, WD, MOMENTUM = 1e-3, 0.9, 0.999, 1e-8, 0.01, 0.9
STEP0 = 100                       # the optimizer has taken this many steps when the pass begins
QUANT_MIN = 4096                  # tensors of at most this many elements, and vectors, keep fp32 states


# ---- the cases -------------------------------------------------------------------------------------------------------

def listed():
    return [
        # one projection matrix stepped on its own, as a program does that steps parameters one by one while the
        # backward pass still runs: latency and launches count
        {"name": "step_1024_f32", "kind": "step", "form": "rank1", "rows": 1024, "cols": 1024, "bf16": False},
        # an embedding matrix on its own, fp32 gradients, 9 of 10 rows without a gradient in this step
        {"name": "step_embed_f32", "kind": "step", "form": "rank1", "rows": 32000, "cols": 4096, "bf16": False,
         "sparse": True},
        # an output head stored (hidden, vocabulary): rows of an odd length, blocks that straddle rows
        {"name": "step_head_50257_bf16", "kind": "step", "form": "rank1", "rows": 1024, "cols": 50257, "bf16": True},
        # one rank's shard of a flattened transformer layer: block-wise second moment, a ragged last block
        {"name": "step_shard_b128_bf16", "kind": "step", "form": "b128", "rows": 1, "cols": 25298945, "bf16": True},
        # 108 M parameters, fp32 gradients: 197 tensors, from bias vectors to a 30522 x 768 embedding
        {"name": "plan_bert_base_f32", "kind": "plan", "form": "rank1", "style": "bert", "hidden": 768, "layers": 12,
         "vocab": 30522, "bf16": False},
        # 354 M parameters, bf16 gradients
        {"name": "plan_gpt2_medium_bf16", "kind": "plan", "form": "rank1", "style": "gpt", "hidden": 1024, "layers": 24,
         "vocab": 50257, "bf16": True},
        # the largest: 6.7 G parameters, bf16 gradients
        {"name": "plan_llama_7b_bf16", "kind": "plan", "form": "rank1", "style": "llama", "hidden": 4096, "layers": 32,
         "vocab": 32000, "bf16": True},
        # 4-bit Factor on the 354 M set
        {"name": "plan_gpt2_factor_bf16", "kind": "plan", "form": "factor", "style": "gpt", "hidden": 1024,
         "layers": 24, "vocab": 50257, "bf16": True},
        # SGD with 4-bit momentum on the 108 M set
        {"name": "plan_bert_sgdm_f32", "kind": "plan", "form": "sgdm", "style": "bert", "hidden": 768, "layers": 12,
         "vocab": 30522, "bf16": False},
        # convolutions (one statistic per dimension), narrow and ragged matrices, biases: the front end's step()
        {"name": "optim_vision_f32", "kind": "optim", "width": 96, "classes": 1000},
        # fp32 moments of one feed-forward matrix into 4-bit states and back
        {"name": "convert_11008x4096", "kind": "convert", "form": "rank1", "rows": 11008, "cols": 4096},
        # the quantizer study: the exponent map without its zero, stochastic rounding, all three normalizations
        {"name": "ablation_4096_de0", "kind": "ablation", "rows": 4096, "cols": 4096, "map": 1, "stochastic": True},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "plan", "plan", "optim", "convert", "ablation"])
    if kind == "step":
        form = rng.choice(["rank1", "rank1", "rank1", "b128", "factor", "sgdm"])
        if form in ("b128", "sgdm"):
            return {"kind": kind, "form": form, "rows": 1, "cols": _log_int(rng, 1 << 16, 1 << 27),
                    "bf16": rng.random() < 0.5}
        rows, cols = _log_int(rng, 128, 32768), _log_int(rng, 128, 51200)
        if rng.random() < 0.5:                       # half of the widths are what models commonly have
            cols = max(128, cols // 128 * 128)
        rows = max(64, min(rows, (1 << 27) // cols))
        return {"kind": kind, "form": form, "rows": rows, "cols": cols, "bf16": rng.random() < 0.5}
    if kind == "plan":
        hidden = 64 * rng.randint(4, 24)             # 256 .. 1536: half of them no multiple of 128
        return {"kind": kind, "form": rng.choice(["rank1", "rank1", "b128", "factor", "sgdm"]),
                "style": rng.choice(["bert", "gpt", "llama"]), "hidden": hidden, "layers": _log_int(rng, 2, 24),
                "vocab": _log_int(rng, 1000, 51200), "bf16": rng.random() < 0.5}
    if kind == "optim":
        return {"kind": kind, "width": 8 * rng.randint(4, 20), "classes": _log_int(rng, 10, 4000)}
    rows, cols = _log_int(rng, 64, 16384), _log_int(rng, 64, 16384)
    if kind == "convert":
        form = rng.choice(["rank1", "rank1", "b128"])
        return {"kind": kind, "form": form, "rows": rows, "cols": cols}
    return {"kind": kind, "rows": rows, "cols": min(cols, (1 << 25) // rows), "map": rng.randint(0, 2),
            "stochastic": rng.random() < 0.5}


# ---- shapes ----------------------------------------------------------------------------------------------------------

def _shapes(case):
    """The tensors of a step or plan case: matrices and vectors, in the order of the model."""
    if case["kind"] == "step":
        return [(case["rows"], case["cols"])]
    h, out = case["hidden"], [(case["vocab"], case["hidden"])]
    if case["style"] == "llama":
        f = (8 * h // 3 + 255) // 256 * 256
        for _ in range(case["layers"]):
            out += [(h, h)] * 4 + [(h, f)] * 2 + [(f, h)] + [(h,)] * 2
        return out + [(h,), (case["vocab"], h)]
    for _ in range(case["layers"]):
        out += [(h, 3 * h), (h, h), (h, 4 * h), (4 * h, h)]
        out += [(3 * h,), (h,), (4 * h,), (h,), (h,), (h,), (h,), (h,)]
    return out + ([(h,), (h,)] if case["style"] == "gpt" else [])


def _vision_shapes(case):
    w, c = case["width"], case["classes"]
    return [(w, 3, 7, 7), (2 * w, w, 3, 3), (4 * w, 2 * w, 3, 3), (8 * w, 4 * w, 3, 3), (3 * w, w), (6 * w, 2 * w),
            (4 * w, w), (16 * w, 4 * w), (8 * w, 32 * w), (c, 8 * w), (w,), (2 * w,), (4 * w,), (c,)]


def _numel(shape):
    return math.prod(shape)


def _form_of(case, shape):
    """How a tensor of the case keeps its state: the case's form, or fp32 for vectors and small tensors of a plan."""
    if case["kind"] != "step" and (len(shape) < 2 or _numel(shape) <= QUANT_MIN):
        return "sgdm32" if case.get("form") == "sgdm" else "fp32"
    if case["kind"] == "optim":
        return "nd" if len(shape) > 2 else "rank1"
    return case["form"]


# ---- the method's definitions in plain torch -------------------------------------------------------------------------

def _signed_map(dtype, dev):
    pos = [0.0055, 0.0325, 0.0775, 0.2125, 0.4375, 0.6625, 0.8875]
    return torch.tensor([-x for x in reversed(pos)] + [0.0] + pos + [1.0], device=dev).to(dtype)     # fp32 entries


def _unsigned_map(dtype, dev, zero=True):
    out = [0.0]
    for k, n in ((2, 2), (1, 4), (0, 8)):            # a decade's n bin midpoints
        p = [0.9 * j / n + 0.1 for j in range(n + 1)]
        out += [10.0 ** -k * (p[j] + p[j + 1]) / 2 for j in range(n)]
    out.append(1.0)
    return torch.tensor(out if zero else out[1:], device=dev).to(dtype)


def _pad_to(x, m):
    n = x.numel()
    return x if n % m == 0 else torch.nn.functional.pad(x, (0, m - n % m))


def _pack(codes):
    q = _pad_to(codes.to(torch.uint8).reshape(-1), 2).view(-1, 2)
    return q[:, 0] | (q[:, 1] << 4)


def _unpack(packed, n):
    return torch.stack((packed & 15, packed >> 4), 1).reshape(-1)[:n].long()


def _blocks(x, b=128):
    """The block maxima of |x| over its row-major flattening."""
    return _pad_to(x.reshape(-1).abs(), b).view(-1, b).amax(1)


def _spread(scale, n, b=128):
    return scale.repeat_interleave(b)[:n]


def _ratio(x, s):
    return torch.where(s > 0, x / s, torch.zeros_like(x))


def _encode_m(m):
    s = _blocks(m)
    T = _signed_map(m.dtype, m.device)
    n = _ratio(m.reshape(-1), _spread(s, m.numel()))
    return _pack(torch.bucketize(n, (T[:-1] + T[1:]) / 2, out_int32=True)), s


def _linear_codes(v, s):
    return torch.clamp(torch.ceil(16 * _ratio(v, s) - 1.5), 0, 15)


def _rank1_stats(v):
    """One maximum per index of every dimension."""
    return [v.amax([d for d in range(v.ndim) if d != k]) for k in range(v.ndim)]


def _rank1_scale(stats):
    p, out = len(stats), None
    for k, mu in enumerate(stats):
        x = mu.view([-1 if d == k else 1 for d in range(p)])
        out = x if out is None else torch.minimum(out, x)
    return out


# ---- states ----------------------------------------------------------------------------------------------------------

class _Slab:
    """Buffers of all tensors of a case in one allocation, each start a multiple of 1024 elements."""

    def __init__(self, sizes, dtype):
        self.at, n = [], 0
        for k in sizes:
            self.at.append((n, k))
            n += (k + 1023) // 1024 * 1024
        self.all = torch.zeros(max(n, 1), dtype=dtype, device=DEV)

    def __getitem__(self, i):
        a, k = self.at[i]
        return self.all[a:a + k]


def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _inputs(shape, gen, sparse=False):
    """Weights, gradient and both moments of one tensor in mid-training: a log-normal gradient scale per column (or,
    for vectors, per run of 1024 elements), a first moment of the same sign structure, a second moment around the
    square of the scale."""
    rows, cols = (shape[0], _numel(shape[1:])) if len(shape) > 1 else (1, shape[0])
    rnd = lambda *s: torch.randn(*s, generator=gen, device=DEV)
    if rows == 1:
        sig = (1e-3 * torch.exp(rnd((cols + 1023) // 1024))).repeat_interleave(1024)[None, :cols]
    else:
        sig = 1e-3 * torch.exp(rnd(cols))[None, :]
    w = 0.02 * rnd(rows, cols)
    g = rnd(rows, cols) * sig
    if sparse:
        g *= (torch.rand(rows, 1, generator=gen, device=DEV) < 0.1)
    m = 0.3 * rnd(rows, cols) * sig
    v = (0.4 + torch.rand(rows, cols, generator=gen, device=DEV)) * sig * sig
    return w, g, m, v


def _sizes(form, shape):
    """Elements of a tensor's state buffers, by name."""
    n = _numel(shape)
    if form in ("fp32", "sgdm32"):
        return {"m": n, "v": n} if form == "fp32" else {"m": n}
    nb, half = (n + 127) // 128, (n + 1) // 2
    d = {"m_codes": half, "m_scale": nb}
    if form == "b128":
        d.update(v_codes=half, v_scale=nb)
    elif form in ("rank1", "factor"):
        d.update(v_row=shape[0], v_col=_numel(shape[1:]))
        if form == "rank1":
            d["v_codes"] = half
    return d


def _fill_state(form, shape, get, m, v, g):
    """The 4-bit (or fp32) state of the moments m and v into the buffers get(name)."""
    if form in ("fp32", "sgdm32"):
        get("m").copy_(m.reshape(-1))
        if form == "fp32":
            get("v").copy_(v.reshape(-1))
        return
    q, s = _encode_m(m)
    get("m_codes").copy_(q)
    get("m_scale").copy_(s)
    if form == "b128":
        s = _blocks(v)
        get("v_scale").copy_(s)
        get("v_codes").copy_(_pack(_linear_codes(v.reshape(-1), _spread(s, v.numel()))))
    elif form == "rank1":
        r, c = _rank1_stats(v)
        get("v_row").copy_(r)
        get("v_col").copy_(c)
        get("v_codes").copy_(_pack(_linear_codes(v, _rank1_scale([r, c]))))
    elif form == "factor":
        get("v_row").copy_(v.sum(1))
        get("v_col").copy_(v.sum(0))


class _Set:
    """Parameters, gradients and states of a step or plan case."""

    def __init__(self, case, seed):
        self.shapes = _shapes(case)
        self.forms = [_form_of(case, s) for s in self.shapes]
        ns = [_numel(s) for s in self.shapes]
        self.param = _Slab(ns, torch.float32)
        self.grad = _Slab(ns, torch.bfloat16 if case["bf16"] else torch.float32)
        per = [_sizes(f, s) for f, s in zip(self.forms, self.shapes)]
        names = sorted({k for d in per for k in d})
        self.state = {k: _Slab([d.get(k, 0) for d in per], torch.uint8 if k.endswith("codes") else torch.float32)
                      for k in names}
        gen = _gen(seed)
        for i, (shape, form) in enumerate(zip(self.shapes, self.forms)):
            w, g, m, v = _inputs(shape, gen, case.get("sparse", False))
            self.param[i].copy_(w.reshape(-1))
            self.grad[i].copy_(g.reshape(-1))
            _fill_state(form, shape, lambda k: self.state[k][i], m, v, g)

    def lib_state(self, i):
        """The library's handle of tensor i's state buffers."""
        form, s = self.forms[i], lambda k: self.state[k][i]
        rows, cols = (self.shapes[i] if len(self.shapes[i]) == 2 else (1, self.shapes[i][0]))
        if form == "fp32":
            return s("m"), s("v")
        if form == "sgdm32":
            return s("m")
        if form == "sgdm":
            return lpmm.StateSgdm(rows * cols, s("m_codes"), s("m_scale"))
        if form == "b128":
            return lpmm.StateB128(rows * cols, s("m_codes"), s("m_scale"), s("v_codes"), s("v_scale"))
        if form == "factor":
            return lpmm.StateFactor(rows, cols, s("m_codes"), s("m_scale"), s("v_row"), s("v_col"))
        return lpmm.State4(rows, cols, s("m_codes"), s("m_scale"), s("v_codes"), s("v_row"), s("v_col"))

    def outputs(self):
        return {"param": self.param.all, **{k: v.all for k, v in self.state.items()}}


class _Plan:
    """A plan with the tensors it refers to; released with it."""

    def __init__(self, s, case):
        descs = []
        for i, form in enumerate(s.forms):
            st, n = s.lib_state(i), _numel(s.shapes[i])
            if form in ("sgdm", "sgdm32"):
                descs.append(lpmm.make_desc_sgdm(s.param[i], s.grad[i], st, n))
            elif form == "fp32":
                descs.append(lpmm.make_desc(s.param[i], s.grad[i], st, 1, n, no_decay=True))
            else:
                descs.append(lpmm.make_desc(s.param[i], s.grad[i], st))
        self.buffer = lpmm.new_plan(descs, lpmm.GRAD_BF16 if case["bf16"] else lpmm.GRAD_F32, DEV)

    def __del__(self):
        try:
            lpmm.lpmm_adamw4_plan_release(self.buffer)
        except Exception:
            pass


def _prepare_optim(case, seed):
    shapes, gen = _vision_shapes(case), _gen(seed)
    flat = _Slab([_numel(s) for s in shapes], torch.float32)
    params, states = [], []
    for i, shape in enumerate(shapes):
        w, g, m, v = _inputs(shape, gen)
        flat[i].copy_(w.reshape(-1))
        p = torch.nn.Parameter(flat[i].view(shape))
        p.grad = g.reshape(shape)
        params.append(p)
        if _form_of(case, shape) == "fp32":
            states.append({"m": m.reshape(-1), "v": v.reshape(-1)})
            continue
        q, s = _encode_m(m)
        v = v.view(shape)
        stats = _rank1_stats(v)
        d = {"m_codes": q, "m_blockscale": s, "v_codes": _pack(_linear_codes(v, _rank1_scale(stats)))}
        if len(shape) > 2:
            d["v_row"] = stats[0]
            d["v_col"] = torch.cat([_rank1_scale(stats[1:]).reshape(-1)] + stats[1:])
        else:
            d["v_rowmax"], d["v_colmax"] = stats
        states.append(d)
    opt = lpmm.AdamW4bit(params, lr=LR, betas=(BETA1, BETA2), eps=EPS, weight_decay=WD)
    opt.load_state_dict({"t": STEP0, "states": states})
    return {"opt": opt, "flat": flat, "params": params}


def _optim_outputs(s):
    out = []
    for st in s["opt"].state_buffers():
        d = {"m": st[0], "v": st[1]} if isinstance(st, tuple) else {k: v for k, v in vars(st).items()
                                                                     if torch.is_tensor(v)}
        out.append(d)
    return {"param": s["flat"].all, "state": out}


def prepare(case, seed):
    torch.cuda.set_device(0)
    kind = case["kind"]
    if kind == "optim":
        return {"kind": kind, **_prepare_optim(case, seed)}
    if kind in ("step", "plan"):
        s = _Set(case, seed)
        state = {"kind": kind, "set": s, "t": STEP0, "form": case["form"], "bf16": case["bf16"]}
        if kind == "plan":
            lpmm.ensure_init(4096)
            state["plan"] = _Plan(s, case)
        else:
            rows, cols = s.shapes[0]
            lpmm.ensure_init(rows + cols if case["form"] in ("rank1", "factor") else 4096)
            state["tensor"] = (s.param[0], s.grad[0], s.lib_state(0))
        return state
    rows, cols = case["rows"], case["cols"]
    lpmm.ensure_init(rows + cols)
    _, _, m, v = _inputs((rows, cols), _gen(seed))
    n = rows * cols
    codes = lambda: torch.zeros(((n + 1) // 2 + 3) // 4 * 4, dtype=torch.uint8, device=DEV)[:(n + 1) // 2]
    f = lambda k: torch.zeros(k, device=DEV)
    if kind == "convert":
        which = 1 if case["form"] == "rank1" else 2
        nv = rows if which == 1 else (n + 127) // 128
        return {"kind": kind, "which": which, "rows": rows, "cols": cols, "m": m, "v": v, "m_codes": codes(),
                "m_scale": f((n + 127) // 128), "v_codes": codes(), "v_scale": f(nv),
                "v_col": f(cols) if which == 1 else None, "m_out": f(n), "v_out": f(n)}
    sets = []
    for norm in (lpmm.NORM_B128, lpmm.NORM_B2048, lpmm.NORM_RANK1):
        a, b = lpmm.ablation_scale_sizes(norm, rows, cols)
        sets.append({"norm": norm, "codes": codes(), "scale": f(a), "col": f(b) if b else None, "out": f(n)})
    return {"kind": kind, "rows": rows, "cols": cols, "v": v, "sets": sets, "map": case["map"],
            "rounding": lpmm.ROUND_STOCHASTIC if case["stochastic"] else lpmm.ROUND_NEAREST, "seed": int(seed)}


# ---- one pass --------------------------------------------------------------------------------------------------------

_STEPS = {("rank1", False): lpmm.lpmm_adamw4_step, ("rank1", True): lpmm.lpmm_adamw4_step_bf16g,
          ("b128", False): lpmm.lpmm_adamw4_b128_step, ("b128", True): lpmm.lpmm_adamw4_b128_step_bf16g,
          ("factor", False): lpmm.lpmm_adamw4_factor_step, ("factor", True): lpmm.lpmm_adamw4_factor_step_bf16g,
          ("sgdm", False): lpmm.lpmm_sgdm4_step, ("sgdm", True): lpmm.lpmm_sgdm4_step_bf16g}


def run(s):
    if s["kind"] == "optim":
        s["opt"].step()
        return _optim_outputs(s)
    if s["kind"] == "step":
        s["t"] += 1
        fn = _STEPS[s["form"], s["bf16"]]
        if s["form"] == "sgdm":
            fn(*s["tensor"], LR, MOMENTUM)
        else:
            fn(*s["tensor"], LR, BETA1, BETA2, EPS, WD, s["t"])
        return s["set"].outputs()
    if s["kind"] == "plan":
        s["t"] += 1
        if s["form"] == "sgdm":
            lpmm.lpmm_sgdm4_step_multi(s["plan"].buffer, LR, MOMENTUM)
        else:
            lpmm.lpmm_adamw4_step_multi(s["plan"].buffer, LR, BETA1, BETA2, EPS, WD, s["t"])
        return s["set"].outputs()
    rows, cols = s["rows"], s["cols"]
    if s["kind"] == "convert":
        lpmm.lpmm_quant_state(0, s["m"], rows, cols, s["m_codes"], s["m_scale"], None)
        lpmm.lpmm_quant_state(s["which"], s["v"], rows, cols, s["v_codes"], s["v_scale"], s["v_col"])
        lpmm.lpmm_dequant_state(0, s["m_codes"], s["m_scale"], None, rows, cols, s["m_out"])
        lpmm.lpmm_dequant_state(s["which"], s["v_codes"], s["v_scale"], s["v_col"], rows, cols, s["v_out"])
        return {k: s[k] for k in ("m_codes", "m_scale", "v_codes", "v_scale", "v_col", "m_out", "v_out")}
    for d in s["sets"]:
        lpmm.lpmm_quant_ablation(d["norm"], s["map"], False, s["rounding"], s["seed"], s["v"], rows, cols, d["codes"],
                                 d["scale"], d["col"])
        lpmm.lpmm_dequant_ablation(d["norm"], s["map"], False, d["codes"], d["scale"], d["col"], rows, cols, d["out"])
    return [{k: d[k] for k in ("codes", "scale", "col", "out")} for d in s["sets"]]


# ---- what a pass cannot do without -----------------------------------------------------------------------------------

# operations of one element: decompress, rule and compress of each moment, the parameter update
_FLOPS = {"rank1": 40, "nd": 40, "b128": 40, "factor": 30, "sgdm": 15, "fp32": 15, "sgdm32": 4}


def work(case):
    kind = case["kind"]
    if kind in ("step", "plan", "optim"):
        total = flops = 0
        for shape in (_vision_shapes(case) if kind == "optim" else _shapes(case)):
            form, n = _form_of(case, shape), _numel(shape)
            b = n * (8 + (2 if case.get("bf16") else 4))                # parameters in and out, gradient in
            if form in ("fp32", "sgdm32"):
                b += n * (16 if form == "fp32" else 8)
            else:
                b += n + n // 16                                        # first moment's codes and scales, in and out
                if form in ("rank1", "nd", "b128"):
                    b += n                                              # second moment's codes, in and out
                b += n // 16 if form == "b128" else 0 if form == "sgdm" else 8 * sum(shape)
            total += b
            flops += n * _FLOPS[form]
        return {"bytes": total, "flops": flops}
    n = case["rows"] * case["cols"]
    if kind == "convert":
        stats = case["rows"] + case["cols"] if case["form"] == "rank1" else n // 128
        # each moment read, its codes written and read, its values written
        return {"bytes": 2 * (n * 8 + n) + 8 * (n // 128 + stats), "flops": 30 * n}
    return {"bytes": n * 4 + 3 * (n * 4 + n), "flops": 60 * n}          # the input once, three round trips


# ---- what a correct pass returns -------------------------------------------------------------------------------------

def tolerance(case):
    """Measured against the 64-bit values: parameters, scales and statistics 2e-8 to 4e-8 off (one or two fp32
    roundings); decompressed moments up to 7e-6 where a few values sit on a decision boundary and 64 bits round them
    the other way.  The row and column sums of the factorized form are 32-bit sums in any order."""
    if case["kind"] in ("convert", "ablation"):
        return {"rel": 3e-5, "max": 1e-1, "differ": 1e-6}
    if case.get("form") == "factor":
        return {"rel": 1e-6, "max": 4e-5, "differ": 1e-6}
    return {"rel": 2e-7, "max": 1e-5, "differ": 1e-6}


def _f32(x):
    return float(np.float32(x))


def _exact_tensor(form, shape, w, g, st, t):
    """One step of one tensor in 64 bits: the new parameters and the floating buffers of the new state."""
    b1, b2, lr, eps, wd = _f32(BETA1), _f32(BETA2), _f32(LR), _f32(EPS), _f32(WD)
    n = w.numel()
    w, g = w.double(), g.double()
    out = {}
    if form in ("fp32", "sgdm32"):
        m = st["m"].double()
    else:
        m = _signed_map(torch.float64, w.device)[_unpack(st["m_codes"], n)] * _spread(st["m_scale"].double(), n)
    if form in ("sgdm", "sgdm32"):
        m = _f32(MOMENTUM) * m + g
        out["param"] = w - lr * m
    else:
        m = b1 * m + (1 - b1) * g
        rows, cols = shape[0], n // shape[0]
        if form == "fp32":
            v = b2 * st["v"].double() + (1 - b2) * g * g
            out["v"], wd = v, 0.0 if st.get("no_decay", True) else wd
        elif form == "factor":
            sq = (g * g).view(rows, cols)
            r = b2 * st["v_row"].double() + (1 - b2) * sq.sum(1)
            c = b2 * st["v_col"].double() + (1 - b2) * sq.sum(0)
            v = (_ratio(r, r.sum())[:, None] * c[None, :]).reshape(-1)
            out["v_row"], out["v_col"] = r, c
        else:
            if form == "b128":
                s = _spread(st["v_scale"].double(), n)
            else:
                s = _rank1_scale([x.double() for x in st["stats"]]).expand(shape).reshape(-1)
            v = b2 * ((_unpack(st["v_codes"], n).double() + 1) / 16 * s) + (1 - b2) * g * g
            if form == "b128":
                out["v_scale"] = _blocks(v)
            else:
                out["stats"] = _rank1_stats(v.view(shape))
        bc1, bc2 = 1 - b1 ** t, 1 - b2 ** t
        out["param"] = w - lr * ((m / bc1) / (torch.sqrt(v / bc2) + eps) + wd * w)
    if form in ("fp32", "sgdm32"):
        out["m"] = m
    else:
        out["m_scale"] = _blocks(m)
    return out


def _exact_set(case, seed):
    s = _Set(case, seed)
    out = {"param": torch.zeros(s.param.all.numel(), dtype=torch.float64, device=DEV)}
    for k, v in s.state.items():
        out[k] = None if k.endswith("codes") else torch.zeros(v.all.numel(), dtype=torch.float64, device=DEV)
    for i, (shape, form) in enumerate(zip(s.shapes, s.forms)):
        st = {k: v[i] for k, v in s.state.items()}
        if form == "rank1":
            st["stats"] = [st["v_row"], st["v_col"]]
        new = _exact_tensor(form, shape, s.param[i], s.grad[i], st, STEP0 + 1)
        if form == "rank1":
            new["v_row"], new["v_col"] = new.pop("stats")
        for k, x in new.items():
            slab = s.param if k == "param" else s.state[k]
            a, n = slab.at[i]
            out[k][a:a + n] = x.reshape(-1)
    return out


def _exact_optim(case, seed):
    s = _prepare_optim(case, seed)
    out = {"param": torch.zeros(s["flat"].all.numel(), dtype=torch.float64, device=DEV), "state": []}
    for i, (p, buf) in enumerate(zip(s["params"], _optim_outputs(s)["state"])):
        shape, form = tuple(p.shape), _form_of(case, tuple(p.shape))
        st = dict(buf)
        if form != "fp32":
            st["m_scale"] = st["m_blockscale"]
            st["stats"] = [st["v_rowmax"], st["v_colmax"]] if form == "rank1" else (
                [st["v_row"]] + list(torch.split(st["v_col"][_numel(shape[1:]):], shape[1:])))
        st["no_decay"] = p.ndim <= 1
        new = _exact_tensor(form, shape, p.detach().reshape(-1), p.grad.reshape(-1), st, STEP0 + 1)
        a, n = s["flat"].at[i]
        out["param"][a:a + n] = new["param"]
        if form == "fp32":
            out["state"].append({"m": new["m"], "v": new["v"]})
            continue
        d = {"m_codes": None, "v_codes": None, "m_blockscale": new["m_scale"]}
        if form == "rank1":
            d["v_rowmax"], d["v_colmax"] = new["stats"]
        else:
            d["v_row"] = new["stats"][0]
            d["v_col"] = torch.cat([_rank1_scale(new["stats"][1:]).reshape(-1)] + new["stats"][1:])
        out["state"].append(d)
    return out


def _splitmix_uniform(seed, n):
    """The library's documented random number of each element: the top 24 bits of SplitMix64's output n + 1, in
    64-bit wrap-around arithmetic (a logical shift is an arithmetic one with the sign bits masked off)."""
    wrap = lambda x: x - (1 << 64) if x >= 1 << 63 else x
    shr = lambda z, k: (z >> k) & ((1 << (64 - k)) - 1)
    z = torch.arange(1, n + 1, device=DEV) * wrap(0x9E3779B97F4A7C15) + wrap(seed % (1 << 64))
    z = (z ^ shr(z, 30)) * wrap(0xBF58476D1CE4E5B9)
    z = (z ^ shr(z, 27)) * wrap(0x94D049BB133111EB)
    return shr(z ^ shr(z, 31), 40).double() * 2.0 ** -24


def exact(case, seed):
    kind = case["kind"]
    if kind in ("step", "plan"):
        return _exact_set(case, seed)
    if kind == "optim":
        return _exact_optim(case, seed)
    s = prepare(case, seed)
    n = s["rows"] * s["cols"]
    if kind == "convert":
        m, v = s["m"].double(), s["v"].double()
        ms, T = _blocks(m), _signed_map(torch.float64, DEV)
        mq = torch.bucketize(_ratio(m.reshape(-1), _spread(ms, n)), (T[:-1] + T[1:]) / 2)
        if s["which"] == 1:
            vs, vc = _rank1_stats(v)
            scale = _rank1_scale([vs, vc])
        else:
            vs, vc = _blocks(v), None
            scale = _spread(vs, n).view(v.shape)
        vq = _linear_codes(v, scale)
        return {"m_codes": None, "m_scale": ms, "v_codes": None, "v_scale": vs, "v_col": vc,
                "m_out": T[mq] * _spread(ms, n), "v_out": ((vq + 1) / 16 * scale).reshape(-1)}
    v, out = s["v"].double(), []
    T = ((_unsigned_map(torch.float64, DEV, zero=s["map"] == 0)) if s["map"] < 2 else
         torch.arange(1, 17, dtype=torch.float64, device=DEV) / 16)
    for d in s["sets"]:
        col = None
        if d["norm"] == lpmm.NORM_RANK1:
            scale, col = _rank1_stats(v)
            full = _rank1_scale([scale, col]).reshape(-1)
        else:
            b = 128 if d["norm"] == lpmm.NORM_B128 else 2048
            scale = _blocks(v, b)
            full = _spread(scale, n, b)
        x = _ratio(v.reshape(-1), full)
        if s["rounding"] == lpmm.ROUND_STOCHASTIC:
            hi = torch.bucketize(x, T).clamp(max=T.numel() - 1)                          # first entry >= x
            lo = (torch.bucketize(x, T, right=True) - 1).clamp(min=0)                    # last entry <= x
            p = _ratio(x - T[lo], T[hi] - T[lo])
            q = torch.where((hi > lo) & (_splitmix_uniform(s["seed"], n) < p), hi, torch.minimum(lo, hi))
        else:
            q = torch.bucketize(x, (T[:-1] + T[1:]) / 2)
        out.append({"codes": None, "scale": scale, "col": col, "out": T[q] * full})
    return out
