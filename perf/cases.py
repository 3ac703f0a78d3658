"""The work this package is measured on: chunk plans executed through the public binding.

A case names a model family with its sizes, the storage type and the chunk plan; one pass is one
``ac_execute`` of a plan whose weights are bound, on an input that is already in device memory, which is
how a program that serves or evaluates such a model calls the library.  The families and sizes are those
of ``paper_2401_10652_amd/inputs.py`` and ``bench.py`` (GPT prefill, ViT, pair stack, UNet stage) plus
ragged and small ones from the same ranges.  Activations are N(0, 1), weight matrices N(0, 0.02) or
N(0, 1 / sqrt(fan_in)) as in the workload recipes; biases and norm parameters are drawn too, as trained
ones are not zero.
"""
import math

import torch

from paper_2401_10652_amd import binding as B
from paper_2401_10652_amd import inputs as I

GIB = 1 << 30


def _transformer(name, dtype, layers, batch, seq, d_model, heads, d_ffn, causal, activation="gelu_erf", dim="seq",
                 chunk=(0, 0, 0, 0), budget=0, budget_share=0.0, in_flight=1, stored_scores=False):
    """chunk: rows (or batch elements) per segment of QKV, attention core, output projection, feed-forward (0: not
    cut, or sized from the budget).  budget: bytes; budget_share: the budget as a share of what the uncut plan needs."""
    return {"name": name, "family": "transformer", "dtype": dtype, "layers": layers, "batch": batch, "seq": seq,
            "d_model": d_model, "heads": heads, "d_ffn": d_ffn, "causal": causal, "activation": activation, "dim": dim,
            "c_qkv": chunk[0], "c_attn": chunk[1], "c_out": chunk[2], "c_ffn": chunk[3], "budget": budget,
            "budget_share": budget_share, "in_flight": in_flight, "stored_scores": stored_scores}


def _pair(name, n_res, c_z, c_hidden, heads, head_dim, factor, activation, chunk, dim):
    return {"name": name, "family": "pair", "dtype": "bf16", "n_res": n_res, "c_z": c_z, "c_hidden": c_hidden, "heads": heads,
            "head_dim": head_dim, "factor": factor, "activation": activation, "chunk": chunk, "dim": dim}


def _unet(name, layers, batch, height, width, channels, groups, chunk, heads=0, d_ffn=0, context_tokens=0, context_dim=0,
          gated=False):
    return {"name": name, "family": "unet", "dtype": "bf16", "layers": layers, "batch": batch, "height": height, "width": width,
            "channels": channels, "groups": groups, "chunk": chunk, "heads": heads, "d_ffn": d_ffn,
            "context_tokens": context_tokens, "context_dim": context_dim, "gated": gated}


def listed():
    return [
        # the smallest call: one fp32 block of 256 tokens (the validation model), latency and launches
        _transformer("block_f32_256", "f32", 1, 1, 256, 64, 4, 256, False, chunk=(64, 64, 64, 64)),
        # a small model evaluated in fp32, where the caller wants no bf16 rounding
        _transformer("gpt_f32_1k", "f32", 2, 1, 1024, 512, 8, 2048, True, chunk=(256, 256, 256, 256)),
        # prefill of a batch of four ordinary prompts whose length is no multiple of a tile
        _transformer("gpt_b4_s1000", "bf16", 2, 4, 1000, 1024, 16, 4096, True, activation="gelu_tanh"),
        # prefill of an 8k prompt with a budget that bites: the planner cuts what it has to
        _transformer("gpt_8k_tight", "bf16", 4, 1, 8192, 1024, 16, 4096, True, budget_share=0.8),
        # prefill of a 64k prompt under 4 GiB: the headline workload of bench.py
        _transformer("gpt_64k", "bf16", 2, 1, 65536, 2048, 16, 8192, True, budget=4 * GIB),
        # the paper's own setting: scores and probabilities stored, the attention core cut along the queries
        _transformer("gpt_4k_stored_scores", "bf16", 2, 1, 4096, 1024, 16, 4096, True, chunk=(0, 1024, 0, 0), stored_scores=True),
        # ViT of 4096 patches with every region cut into 512-token segments
        _transformer("vit_4k", "bf16", 12, 1, 4096, 768, 12, 3072, False, chunk=(512, 512, 512, 512)),
        # ViT on a batch of ordinary images (196 patches, padded to 200), eight images per segment, two segments in flight
        _transformer("vit_b32_s200", "bf16", 12, 32, 200, 768, 12, 3072, False, dim="batch", chunk=(8, 8, 8, 8), in_flight=2),
        # pair stack of a 1024-residue protein, every module in 64-row segments
        _pair("pair_1024", 1024, 128, 128, 4, 32, 4, "relu", 64, "row"),
        # pair stack of an ordinary protein of no round length, the ending node's attention along columns
        _pair("pair_200", 200, 128, 128, 4, 32, 4, "relu", 40, "natural"),
        # latent-diffusion stage: residual blocks on eight latents, two per segment
        _unet("unet_res_64x64", 2, 8, 64, 64, 320, 32, 2),
        # the same stage with its attention block: text context and gated feed-forward
        _unet("unet_attn_64x64", 1, 8, 64, 64, 320, 32, 2, heads=5, d_ffn=1280, context_tokens=77, context_dim=768, gated=True),
    ]


def _log_int(rng, lo, hi, step=1):
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return min(hi, max(lo, int(round(v / step)) * step))


def _draw_transformer(rng):
    dtype = "f32" if rng.random() < 0.2 else "bf16"
    if dtype == "f32":
        head_dim = rng.choice([16, 32, 64])
        heads = rng.choice([2, 4, 8])
        d = heads * head_dim
        seq, layers, batch = _log_int(rng, 96, 1536), rng.randint(1, 3), rng.choice([1, 1, 2])
        stored = False
    else:
        head_dim = rng.choice([64, 64, 128])
        heads = rng.choice([6, 8, 12, 16]) if head_dim == 64 else rng.choice([4, 8, 16])
        d = heads * head_dim
        seq = _log_int(rng, 128, 16384, 8)
        batch = max(1, min(16, int(8192 / seq * rng.uniform(0.5, 2.0))))
        layers = rng.randint(1, 4)
        stored = rng.random() < 0.12 and seq <= 4096
    causal = rng.random() < 0.6
    in_flight = 2 if rng.random() < 0.2 else 1
    plan = rng.choice(["whole", "cut", "tight"] + (["batch"] if batch > 1 else []))
    if stored:
        plan = "cut"
    dim, chunk, share = "seq", (0, 0, 0, 0), 0.0
    if plan == "cut":
        chunk = tuple(min(seq, _log_int(rng, max(64, seq // 12), seq, 8)) for _ in range(4))
    elif plan == "batch":
        dim, chunk = "batch", (rng.randint(1, batch),) * 4
    elif plan == "tight":
        share = rng.uniform(0.78, 0.95)
    return _transformer("", dtype, layers, batch, seq, d, heads, 4 * d, causal, rng.choice(["gelu_erf", "gelu_tanh", "relu"]),
                        dim, chunk, 0, share, in_flight, stored)


def _draw_pair(rng):
    n = _log_int(rng, 64, 768, 8)
    c = rng.choice([64, 128, 128])
    return _pair("", n, c, 128, rng.choice([2, 4]), 32, rng.choice([2, 4]), rng.choice(["relu", "gelu_erf"]),
                 _log_int(rng, max(8, n // 12), n), rng.choice(["row", "col", "natural"]))


def _draw_unet(rng):
    h, w = 8 * rng.randint(2, 10), 8 * rng.randint(2, 10)
    c, batch = rng.choice([128, 192, 256, 320, 320, 384, 512, 640]), rng.randint(1, 10)
    chunk = rng.randint(1, batch)
    if rng.random() < 0.5:
        return _unet("", rng.randint(1, 3), batch, h, w, c, 32, chunk)
    cross = rng.random() < 0.7
    return _unet("", 1, batch, h, w, c, 32, chunk, heads=c // 64, d_ffn=4 * c, context_tokens=rng.randint(16, 160) if cross else 0,
                 context_dim=768 if cross else 0, gated=rng.random() < 0.7)


def draw(rng):
    while True:
        case = rng.choice([_draw_transformer, _draw_transformer, _draw_pair, _draw_unet])(rng)
        # (a smaller job than the 64k prefill: fp32 and stored scores run at a fraction of the fused bf16 rate)
        limit = 2e11 if case["dtype"] == "f32" or case.get("stored_scores") else 8e12
        if work(case)["flops"] <= limit:
            del case["name"]
            return case


# ---- sizes ------------------------------------------------------------------------------------

def _config(case):
    name = case.get("name", "drawn")
    if case["family"] == "transformer":
        return I.TransformerConfig(name, 0, case["layers"], case["seq"], case["d_model"], case["heads"], case["d_ffn"],
                                   case["causal"], case["dtype"], None, batch=case["batch"], activation=case["activation"])
    if case["family"] == "pair":
        return I.PairConfig(name, 0, case["n_res"], case["c_z"], case["c_hidden"], case["heads"], case["head_dim"],
                            case["factor"], case["dtype"], activation=case["activation"])
    return I.ResStackConfig(name, 0, case["layers"], case["batch"], case["height"], case["width"], case["channels"],
                            case["groups"], heads=case["heads"], d_ffn=case["d_ffn"], context_tokens=case["context_tokens"],
                            context_dim=case["context_dim"], gated=case["gated"])


def _tensors(cfg):
    """[(name, shape)] of everything that is bound, in bind order."""
    if isinstance(cfg, I.TransformerConfig):
        shapes = I.transformer_layer_shapes(cfg)
        return [(n, shapes[n]) for _ in range(cfg.layers) for n in I.TRANSFORMER_LAYER_TENSORS]
    if isinstance(cfg, I.PairConfig):
        return I.pair_tensor_shapes(cfg)
    c, f, up = cfg.channels, cfg.d_ffn, 2 if cfg.gated else 1
    special = {"w1": (c, 9 * c), "w2": (c, 9 * c), "temb": (cfg.batch, c), "w_in": (c, c), "w_qkv": (3 * c, c), "b_qkv": (3 * c,),
               "w_o": (c, c), "w_1": (up * f, c), "b_1": (up * f,), "w_2": (c, f), "w_out": (c, c), "w_qc": (c, c),
               "w_kvc": (2 * c, cfg.context_dim), "w_oc": (c, c), "context": (cfg.batch * cfg.context_tokens, cfg.context_dim)}
    names = I.RES_BLOCK_TENSORS + I.attn_block_tensors(cfg)
    return [(n, special.get(n, (c,))) for _ in range(cfg.layers) for n in names]


def _input_shape(cfg):
    if isinstance(cfg, I.TransformerConfig):
        return (cfg.tokens, cfg.d_model)
    if isinstance(cfg, I.PairConfig):
        return (cfg.n_res, cfg.n_res, cfg.c_z)
    return (cfg.batch, cfg.height, cfg.width, cfg.channels)


def work(case):
    """Every input and weight read once and the output written once; the operations of the contractions (causal
    attention: the visible pairs only)."""
    cfg = _config(case)
    size = 2 if case["dtype"] == "bf16" else 4
    elems = 2 * math.prod(_input_shape(cfg)) + sum(math.prod(s) for _, s in _tensors(cfg))
    if case["family"] == "transformer":
        t, d, s = cfg.tokens, cfg.d_model, cfg.seq
        pairs = cfg.batch * (s * (s + 1) // 2 if cfg.causal else s * s)
        flops = cfg.layers * (2 * t * d * (4 * d + 2 * cfg.d_ffn) + 4 * pairs * d)
    elif case["family"] == "pair":
        n, z, h, hd = cfg.n_res, cfg.c_z, cfg.c_hidden, cfg.heads * cfg.head_dim
        mul = 2 * n * n * (4 * z * h + z * z + h * z) + 2 * n ** 3 * h
        att = 2 * n * n * (5 * z * hd + z * cfg.heads) + 4 * n ** 3 * hd
        flops = 2 * mul + 2 * att + 4 * n * n * cfg.transition_factor * z * z
    else:
        c, hw = cfg.channels, cfg.height * cfg.width
        t = cfg.batch * hw
        flops = 2 * 2 * t * 9 * c * c
        if cfg.heads:
            flops += 2 * t * c * (6 * c + (3 if cfg.gated else 2) * cfg.d_ffn) + 4 * t * hw * c
            if cfg.context_tokens:
                k = cfg.batch * cfg.context_tokens
                flops += 2 * t * c * 2 * c + 2 * k * cfg.context_dim * 2 * c + 4 * t * cfg.context_tokens * c
        flops *= cfg.layers
    return {"bytes": elems * size, "flops": flops}


# ---- the measured call ------------------------------------------------------------------------

def _values(name, shape, case, dtype, gen):
    leaf = name.split(".")[-1]
    std, mean = 1.0, 0.0
    if leaf.endswith("_g") and not leaf.startswith(("w", "b")):
        std, mean = 0.1, 1.0                                   # gain of a norm
    elif leaf == "temb":
        std = 0.5
    elif leaf == "context":
        std = 1.0
    elif leaf.startswith("w"):
        std = 0.02 if case["family"] == "transformer" and case["dtype"] == "bf16" else 1.0 / math.sqrt(shape[1])
    else:
        std = 0.1                                              # biases and shifts
    return torch.randn(shape, generator=gen, device="cuda").mul_(std).add_(mean).to(dtype)


def _regions(case):
    if case["family"] == "transformer":
        dim = B.AC_DIM_BATCH if case["dim"] == "batch" else B.AC_DIM_SEQ
        extent = case["batch"] if case["dim"] == "batch" else case["seq"]
        by_budget = case["budget"] > 0 or case["budget_share"] > 0
        kinds = (B.AC_REGION_QKV, B.AC_REGION_ATTENTION, B.AC_REGION_OUT_PROJ, B.AC_REGION_FFN)
        lens = (case["c_qkv"], case["c_attn"], case["c_out"], case["c_ffn"])
        return [(k, dim, 0 if by_budget else n or extent) for k, n in zip(kinds, lens)]
    if case["family"] == "pair":
        def dim(k):
            if case["dim"] == "natural":     # rows, except the ending node's attention, whose problems are columns
                return B.AC_DIM_COL if k == B.AC_REGION_TRIATT_END else B.AC_DIM_ROW
            return B.AC_DIM_COL if case["dim"] == "col" else B.AC_DIM_ROW
        return [(k, dim(k), case["chunk"]) for k in range(B.AC_REGION_TRIMUL_OUT, B.AC_REGION_PAIR_TRANSITION + 1)]
    kinds = (B.AC_REGION_RES_BLOCK, B.AC_REGION_UNET_ATTN) if case["heads"] else (B.AC_REGION_RES_BLOCK,)
    return [(k, B.AC_DIM_BATCH, case["chunk"]) for k in kinds]


def _plan(case, cfg):
    if case["family"] == "pair":
        return B.Plan(B.pair_desc(cfg), _regions(case), 0)
    if case["family"] == "unet":
        return B.Plan(B.res_stack_desc(cfg), _regions(case), 0)
    flags = B.AC_FLAG_TWO_SEGMENTS_IN_FLIGHT if case["in_flight"] == 2 else 0
    flags |= B.AC_FLAG_MATERIALIZED_SCORES if case["stored_scores"] else 0
    desc = B.transformer_desc(cfg, flags=flags)
    budget = case["budget"]
    if case["budget_share"] > 0:
        whole = B.Plan(desc, (), 0)
        budget = int(case["budget_share"] * whole.ac_plan_query().peak_bytes_planned)
        whole.close()
        try:
            return B.Plan(desc, _regions(case), budget)
        except B.AcError as err:
            # the tensors that no plan can cut take a larger share of this model: the least the planner can do
            if err.status != B.AC_ERR_BUDGET_INFEASIBLE:
                raise
            return B.Plan(desc, [(k, dim, 128) for k, dim, _ in _regions(case)], 0)
    return B.Plan(desc, _regions(case), budget)


def _inputs(case, cfg, seed):
    """The input and the weights in bind order."""
    dtype = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    gen = torch.Generator(device="cuda").manual_seed(seed)
    x = torch.randn(_input_shape(cfg), generator=gen, device="cuda").to(dtype)
    return x, [_values(n, s, case, dtype, gen) for n, s in _tensors(cfg)]


def prepare(case, seed):
    """Input, weights, the plan with its weights bound and its workspace: what such a program keeps."""
    cfg = _config(case)
    x, weights = _inputs(case, cfg, seed)
    plan = _plan(case, cfg)
    plan.ac_plan_bind_weights(weights)
    workspace = B.empty_workspace(plan.ac_plan_query().workspace_bytes)
    return {"plan": plan, "x": x, "y": torch.empty_like(x), "workspace": workspace}


def run(state):
    state["plan"].ac_execute(state["x"], state["y"], state["workspace"])
    return state["y"]


def tolerance(case):
    # Against the same stack in fp64 (relative 2-norm / largest element): fp32 2e-7 to 7e-7 / 5e-6; bf16 2.4e-3 to 5.0e-3 / 0.03
    # up to five modules deep and 8.0e-3 / 0.058 after twelve layers, the stored residual stream's roundings adding up as
    # the square root of the depth.
    if case["dtype"] == "f32":
        return {"rel": 4e-6, "max": 4e-5}
    rel = max(1e-2, 5e-3 * math.sqrt(case.get("layers", 1)))
    return {"rel": rel, "max": 15 * rel}


# ---- the same in 64 bits, plain torch -----------------------------------------------------------

def _norm(x, gain, shift):
    return torch.nn.functional.layer_norm(x, x.shape[-1:], gain, shift, 1e-5)


def _act(x, name):
    if name == "relu":
        return torch.relu(x)
    return torch.nn.functional.gelu(x, approximate="tanh" if name == "gelu_tanh" else "none")


def _attend(q, k, v, heads, causal, rows=2048):
    """q [s, heads * dh] against k, v [t, heads * dh] of one sequence, some query rows of one head at a time."""
    out, dh, at = torch.empty_like(q), q.shape[1] // heads, torch.arange(k.shape[0], device=q.device)
    for h in range(heads):
        c = slice(h * dh, (h + 1) * dh)
        for a in range(0, q.shape[0], rows):
            b = min(q.shape[0], a + rows)
            seen = b if causal else k.shape[0]
            p = q[a:b, c] @ k[:seen, c].T.contiguous()
            p *= 1.0 / math.sqrt(dh)
            if causal:
                p.masked_fill_(at[None, :seen] > at[a:b, None], -math.inf)
            out[a:b, c] = torch.softmax(p, -1) @ v[:seen, c]
    return out


def _layer(x, w, heads, causal, activation, sequences, context=None, gated=False):
    """One pre-LN layer on [tokens, d]; attention inside each of `sequences` equal runs of tokens."""
    d, s = x.shape[1], x.shape[0] // sequences
    qkv = _norm(x, w["ln1_g"], w["ln1_b"]) @ w["w_qkv"].T + w["b_qkv"]
    ctx = torch.cat([_attend(*t.split(d, -1), heads, causal) for t in qkv.split(s)])
    x = x + ctx @ w["w_o"].T + w["b_o"]
    if context is not None:
        q = _norm(x, w["lnc_g"], w["lnc_b"]) @ w["w_qc"].T
        kv = [(t @ w["w_kvc"].T).split(d, -1) for t in context]
        ctx = torch.cat([_attend(t, *kv[i], heads, False) for i, t in enumerate(q.split(s))])
        x = x + ctx @ w["w_oc"].T + w["b_oc"]
    hid = _norm(x, w["ln2_g"], w["ln2_b"]) @ w["w_1"].T + w["b_1"]
    if gated:
        value, gate = hid.chunk(2, -1)
        hid = value * _act(gate, activation)
    else:
        hid = _act(hid, activation)
    return x + hid @ w["w_2"].T + w["b_2"]


def _tri_mul(z, w, outgoing):
    t = _norm(z, w["ln_in_g"], w["ln_in_b"])
    a, b = (torch.sigmoid(t @ w[f"w_{n}g"].T + w[f"b_{n}g"]) * (t @ w[f"w_{n}p"].T + w[f"b_{n}p"]) for n in "ab")
    o = torch.empty_like(a)
    for c in range(a.shape[2]):     # o[i, j] = sum_k a[i, k] b[j, k], or a[k, i] b[k, j]
        ac, bc = a[:, :, c].contiguous(), b[:, :, c].contiguous()
        o[:, :, c] = ac @ bc.T.contiguous() if outgoing else ac.T.contiguous() @ bc
    g = torch.sigmoid(t @ w["w_g"].T + w["b_g"])
    return z + g * (_norm(o, w["ln_out_g"], w["ln_out_b"]) @ w["w_o"].T + w["b_o"])


def _tri_att(z, w, heads, starting):
    if not starting:                # the starting node's form on the transposed pair tensor
        return _tri_att(z.transpose(0, 1), w, heads, True).transpose(0, 1)
    t = _norm(z, w["ln_g"], w["ln_b"])
    bias = (t @ w["w_bias"].T).permute(2, 0, 1)
    out = torch.empty_like(t @ w["w_q"].T)
    dh = out.shape[2] // heads
    for a in range(0, z.shape[0], 64):
        q, k, v = ((t[a:a + 64] @ w[n].T).unflatten(-1, (heads, dh)).transpose(1, 2).contiguous() for n in ("w_q", "w_k", "w_v"))
        p = torch.softmax(torch.matmul(q, k.transpose(2, 3).contiguous()) / math.sqrt(dh) + bias, -1)
        out[a:a + 64] = torch.matmul(p, v).transpose(1, 2).flatten(2)
    return z + (torch.sigmoid(t @ w["w_g"].T + w["b_g"]) * out) @ w["w_o"].T + w["b_o"]


def _pair_block(z, w, heads, activation):
    def of(p):
        return {n[len(p):]: t for n, t in w.items() if n.startswith(p)}
    z = _tri_mul(_tri_mul(z, of("tmo."), True), of("tmi."), False)
    z = _tri_att(_tri_att(z, of("tas."), heads, True), of("tae."), heads, False)
    w = of("pt.")
    return z + _act(_norm(z, w["ln_g"], w["ln_b"]) @ w["w_1"].T + w["b_1"], activation) @ w["w_2"].T + w["b_2"]


def _group_norm(x, groups, gain, shift):
    return torch.nn.functional.group_norm(x.permute(0, 3, 1, 2), groups, gain, shift, 1e-5).permute(0, 2, 3, 1)


def _conv(x, w):
    b, h, wd, c = x.shape
    xp, w = torch.nn.functional.pad(x, (0, 0, 1, 1, 1, 1)), w.view(-1, 3, 3, c)
    return sum(xp[:, i:i + h, j:j + wd] @ w[:, i, j].T.contiguous() for i in range(3) for j in range(3))


def _res_block(x, w, groups):
    silu = torch.nn.functional.silu
    h = _conv(silu(_group_norm(x, groups, w["gn1_g"], w["gn1_b"])), w["w1"]) + (w["b1"] + w["temb"])[:, None, None, :]
    return x + _conv(silu(_group_norm(h, groups, w["gn2_g"], w["gn2_b"])), w["w2"]) + w["b2"]


def _attn_block(x, w, cfg):
    t = _group_norm(x, cfg.groups, w["gn_g"], w["gn_b"]).reshape(-1, cfg.channels) @ w["w_in"].T + w["b_in"]
    context = w["context"].split(cfg.context_tokens) if cfg.context_tokens else None
    t = _layer(t, w, cfg.heads, False, "gelu_erf", cfg.batch, context, cfg.gated)
    return x + (t @ w["w_out"].T + w["b_out"]).view_as(x)


def exact(case, seed):
    """What run() returns, in 64 bits."""
    cfg = _config(case)
    x, weights = _inputs(case, cfg, seed)
    x, names = x.double(), [n for n, _ in _tensors(cfg)]
    layers = 1 if case["family"] == "pair" else cfg.layers
    per = len(names) // layers
    for i in range(layers):
        w = {n: t.double() for n, t in zip(names[:per], weights[i * per:(i + 1) * per])}
        if case["family"] == "transformer":
            x = _layer(x, w, cfg.heads, cfg.causal, cfg.activation, cfg.batch)
        elif case["family"] == "pair":
            x = _pair_block(x, w, cfg.heads, cfg.activation)
        else:
            x = _res_block(x, w, cfg.groups)
            if cfg.heads:
                x = _attn_block(x, w, cfg)
    return x.contiguous()
