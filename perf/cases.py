"""The work that users of the library have it do, as cases that can be timed and whose outputs can be compared.

A case is one AGZO step (Alg. 2) through the public entry points, in one of four forms:
  set      agzo_step_many over the seven projections of one decoder layer, every projection with its own loss and scalar
           (the benchmark's workload; bf16 or fp32 storage; three forwards, one-sided, or f0/f+/f- from one pass)
  layer    agzo_step on a single linear layer (squared error, or token cross-entropy of an LM head)
  decoder  the whole-model step: decoder layers and an LM head composed from the per-layer calls and the glue kernels,
           one global scalar, bf16
  dense    the dense Gaussian estimator the paper compares with, over the seven projections: agzo_dense_perturb around
           plain forwards
Weights are updated in place, and every pass takes the next seed, as a training loop does.
"""
import math

import torch

from paper_2601_17261_amd import binding, synth

EPS = 1e-3
MODEL_EPS = 1e-2         # whole bf16 models: rounded activations put a floor under L+ - L-, which this stands clear of
POWER_STEPS = 3          # what the paper recommends and every configuration here uses
SETS = {"0.6b": synth.QWEN3_0P6B_LAYER, "4b": synth.QWEN3_4B_LAYER, "8b": synth.QWEN3_8B_LAYER}
SHARES_X = {"q": "attn", "k": "attn", "v": "attn", "gate": "mlp", "up": "mlp"}    # projections that read one tensor
SCHEDULES = {"central": 0, "one_sided": binding.ONE_SIDED, "shared": binding.SHARED_FORWARD}
# the decoder of the 28-layer configuration, at a depth that is quick to set up (every layer does the same work)
HIDDEN, HEADS, KV_HEADS, INTER, VOCAB = 2048, 16, 8, 6144, 32000


def listed():
    return [
        # the small fp32 configuration: one 256 x 256 layer, where launches and latency are all there is
        {"name": "layer_f32_256", "kind": "layer", "dtype": "f32", "d_in": 256, "d_out": 256, "tokens": 512, "rank": 4, "loss": "mse"},
        # a short batch (16 sentences of 27 tokens) through one narrow bf16 layer at the paper's rank
        {"name": "layer_short_batch", "kind": "layer", "dtype": "bf16", "d_in": 1024, "d_out": 1024, "tokens": 432, "rank": 1, "loss": "mse"},
        # the paper's own setting: 0.6B-sized projections held in fp32, rank 1, a batch of no round size
        {"name": "set_0p6b_f32", "kind": "set", "set": "0.6b", "dtype": "f32", "tokens": 1000, "rank": 1, "schedule": "central"},
        # the small bf16 layer set, 8 x 256 tokens
        {"name": "set_0p6b", "kind": "set", "set": "0.6b", "dtype": "bf16", "tokens": 2048, "rank": 8, "schedule": "central"},
        # few tokens on middle-sized projections: one column of the rank x tokens sweep
        {"name": "set_4b_512", "kind": "set", "set": "4b", "dtype": "bf16", "tokens": 512, "rank": 4, "schedule": "central"},
        # a batch packed without padding: a token count that no tile divides
        {"name": "set_4b_ragged", "kind": "set", "set": "4b", "dtype": "bf16", "tokens": 3001, "rank": 16, "schedule": "central"},
        # the largest rank, f0/f+/f- from one pass
        {"name": "set_4b_shared_r64", "kind": "set", "set": "4b", "dtype": "bf16", "tokens": 4096, "rank": 64, "schedule": "shared"},
        # the benchmark's layer set, 16 x 1024 tokens
        {"name": "set_8b", "kind": "set", "set": "8b", "dtype": "bf16", "tokens": 16384, "rank": 16, "schedule": "central"},
        # an LM head with token cross-entropy on a batch without padding
        {"name": "head_ce_ragged", "kind": "layer", "dtype": "bf16", "d_in": 2048, "d_out": 32000, "tokens": 3001, "rank": 16, "loss": "ce"},
        # whole-model step, the decoder configuration's widths and batch
        {"name": "decoder_16x512", "kind": "decoder", "layers": 4, "seqs": 16, "seq_len": 512, "rank": 16},
        # the same on a handful of short sentences
        {"name": "decoder_5x77", "kind": "decoder", "layers": 2, "seqs": 5, "seq_len": 77, "rank": 1},
        # the dense estimator on the small layer set
        {"name": "dense_0p6b", "kind": "dense", "set": "0.6b", "tokens": 2048},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: token counts, widths and ranks over the range the listed cases span, odd ones among them."""
    kind = rng.choice(("set", "set", "set", "layer", "layer", "decoder", "decoder", "dense"))
    rank = rng.choice((1, 4, 8, 16, rng.randint(2, 64)))
    if kind == "set":
        name = rng.choice(("0.6b", "4b", "8b"))
        f32 = name == "0.6b" and rng.random() < 0.5
        n = _log_int(rng, 128, 2048 if f32 else 16384)
        if rng.random() < 0.4:
            n = max(128, n // 256 * 256)
        return {"kind": "set", "set": name, "dtype": "f32" if f32 else "bf16", "tokens": n, "rank": rank,
                "schedule": rng.choice(("central", "central", "one_sided", "shared"))}
    if kind == "layer":
        loss = rng.choice(("mse", "mse", "ce"))
        f32 = loss == "mse" and rng.random() < 0.4
        top = 2048 if f32 else 8192
        d_in = 8 * _log_int(rng, 32, top // 8)
        d_out = _log_int(rng, 8000, 40000) if loss == "ce" else _log_int(rng, 256, top)
        return {"kind": "layer", "dtype": "f32" if f32 else "bf16", "d_in": d_in, "d_out": d_out, "tokens": _log_int(rng, 128, 2048 if f32 else 8192),
                "rank": rank, "loss": loss}
    if kind == "decoder":
        seq_len = _log_int(rng, 32, 2048)
        return {"kind": "decoder", "layers": rng.randint(1, 4), "seqs": max(1, min(64, _log_int(rng, 256, 8192) // seq_len)), "seq_len": seq_len, "rank": rank}
    return {"kind": "dense", "set": rng.choice(("0.6b", "4b")), "tokens": _log_int(rng, 128, 8192)}


# ---- inputs ------------------------------------------------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return dict(device="cuda", dtype=torch.float32, generator=g)


def _activations(seed, n, d_in, dtype):
    """bf16: power-law spectrum with outlier channels; fp32: a few planted directions and noise (the two recipes of the
    repository's configurations)."""
    if dtype == "bf16":
        return synth.device_powerlaw_x(seed, n, d_in)
    kw, k = _gen(seed), min(16, n, d_in)
    u = torch.linalg.qr(torch.randn(n, k, **kw))[0]
    v = torch.linalg.qr(torch.randn(d_in, k, **kw))[0]
    s = torch.logspace(1.0, -1.0, k, device="cuda")
    return ((u * s) @ v.T + 0.01 * torch.randn(n, d_in, **kw)).contiguous()


def _weights_and_target(seed, x, d_out, dtype):
    if dtype == "bf16":
        return synth.device_weights_and_target(seed, x, d_out)
    kw = _gen(seed)
    w = torch.randn(d_out, x.shape[1], **kw) * 0.02
    shift = 0.025 * (torch.randn(d_out, 4, **kw) @ torch.randn(x.shape[1], 4, **kw).T)
    return w, x @ (w + shift).T


def _set_layers(case, seed):
    """(W, X, target) per projection; projections that read the same activations share X."""
    xs, got = {}, []
    for i, (name, d_in, d_out) in enumerate(SETS[case["set"]]):
        key = SHARES_X.get(name, name)
        if key not in xs:
            xs[key] = _activations(1000 * seed + 100 + i, case["tokens"], d_in, case.get("dtype", "bf16"))
        w, t = _weights_and_target(1000 * seed + i, xs[key], d_out, case.get("dtype", "bf16"))
        got.append((w, xs[key], t))
    return got


def _learning_rate(case):
    return 1e-2 if case.get("dtype") == "f32" else 1e-4


def prepare(case, seed):
    kind = case["kind"]
    state = {"kind": kind, "ctx": binding.Context(), "step": 0, "lr": _learning_rate(case)}
    if kind == "set":
        r, layers = case["rank"], _set_layers(case, seed)
        out = torch.zeros(len(layers), 4, dtype=torch.float64, device="cuda")
        items = state["ctx"].make_step_items(
            [(binding.make_layer(w, x, r), w, x, binding.make_loss(t), 0, out[i], None) for i, (w, x, t) in enumerate(layers)])
        state.update(layers=layers, out=out, items=items, flags=SCHEDULES[case["schedule"]])
    elif kind == "layer":
        x = _activations(1000 * seed + 100, case["tokens"], case["d_in"], case["dtype"])
        if case["loss"] == "ce":
            kw = _gen(1000 * seed)
            w = (torch.randn(case["d_out"], case["d_in"], **kw) * 0.02).to(torch.bfloat16)
            t = torch.randint(0, case["d_out"], (case["tokens"],), device="cuda", generator=kw["generator"], dtype=torch.int32)
            loss = binding.make_loss(t, kind=binding.LOSS_CE)
        else:
            w, t = _weights_and_target(1000 * seed, x, case["d_out"], case["dtype"])
            loss = binding.make_loss(t)
        state.update(w=w, x=x, target=t, loss=loss, layer=binding.make_layer(w, x, case["rank"]),
                     out=torch.zeros(4, dtype=torch.float64, device="cuda"))
    elif kind == "decoder":
        params, ids = synth.device_decoder(seed, case["layers"], HIDDEN, HEADS, KV_HEADS, INTER, VOCAB, case["seqs"], case["seq_len"])
        state.update(model=_Decoder(state["ctx"], params, ids, case["rank"]))
    else:
        layers = _set_layers(case, seed)
        out = torch.zeros(len(layers), 4, dtype=torch.float64, device="cuda")
        state.update(layers=layers, out=out, desc=[(binding.make_layer(w, x, 1), binding.make_loss(t)) for w, x, t in layers])
    torch.cuda.synchronize()
    return state


# ---- one pass ----------------------------------------------------------------------------------------------------
class _Decoder:
    """Alg. 2 over decoder layers (grouped-query attention with per-head normalisation and rotary embedding, gated MLP)
    and an LM head with next-token cross-entropy: all linear layers perturbed at once, one scalar, one basis per layer."""

    def __init__(self, ctx, params, ids, r):
        self.ctx, self.r, self.n_layers = ctx, r, params["n_layers"]
        self.seqs, self.seq_len = ids.shape
        self.names = [(p, l) for l in range(self.n_layers) for p in synth.DECODER_PROJECTIONS] + [("head", 0)]
        self.index = {nm: i for i, nm in enumerate(self.names)}
        self.w = {nm: params[nm] for nm in self.names}
        self.embedding, self.ids = params["E"], ids.reshape(-1)
        target = torch.full(ids.shape, -1, dtype=torch.int32, device=ids.device)
        target[:, :-1] = ids[:, 1:].to(torch.int32)
        self.target = target.reshape(-1).contiguous()
        self.loss = binding.make_loss(self.target, kind=binding.LOSS_CE)
        n = self.ids.numel()
        self.y = {nm: torch.empty(n, w.shape[0], dtype=torch.bfloat16, device="cuda") for nm, w in self.w.items() if nm[0] != "head"}
        self.b = {nm: torch.empty(w.shape[1], r, dtype=torch.float32, device="cuda") for nm, w in self.w.items()}
        self.x = {}
        self.out = torch.zeros(4, dtype=torch.float64, device="cuda")

    def normed(self, h):
        y = torch.empty_like(h)
        self.ctx.glue_rmsnorm(h, y)
        return y

    def linear(self, nm, x, sign, seed0, loss_dev=None):
        w, y = self.w[nm], self.y.get(nm)
        desc = binding.make_layer(w, x, self.r, Y=y)
        loss = self.loss if nm[0] == "head" else None
        seed = seed0 + self.index[nm]
        if sign == 0:
            self.x[nm] = x
            self.ctx.layer_forward_sketch(desc, w, x, y, binding.SKETCH_NONE, None, seed, None, loss, loss_dev)
        else:
            self.ctx.perturbed_forward(desc, w, x, self.b[nm], seed, sign * MODEL_EPS, y, loss, loss_dev)
        return y

    def forward(self, sign, seed0, loss_dev):
        h = self.embedding[self.ids]
        for l in range(self.n_layers):
            n = self.normed(h)
            q, k, v = (self.linear((p, l), n, sign, seed0) for p in ("q", "k", "v"))
            a = torch.empty_like(q)
            self.ctx.glue_attention(q, k, v, a, self.seqs, self.seq_len)
            self.ctx.glue_add(h, self.linear(("o", l), a, sign, seed0))
            n = self.normed(h)
            g, u = self.linear(("gate", l), n, sign, seed0), self.linear(("up", l), n, sign, seed0)
            m = torch.empty_like(g)
            self.ctx.glue_swiglu(g, u, m)
            self.ctx.glue_add(h, self.linear(("down", l), m, sign, seed0))
        self.linear(("head", 0), self.normed(h), sign, seed0, loss_dev)

    def step(self, step, lr):
        seed0 = 100_000 * (step + 1)
        self.forward(0, seed0, self.out[0:1])
        self.ctx.basis_many([(binding.make_layer(self.w[nm], self.x[nm], self.r), self.x[nm], seed0 + i, None, self.b[nm])
                             for i, nm in enumerate(self.names)], POWER_STEPS)
        self.x.clear()
        self.forward(+1, seed0, self.out[1:2])
        self.forward(-1, seed0, self.out[2:3])
        self.ctx.two_point(self.out, MODEL_EPS)
        self.ctx.update_many([(self.w[nm], self.b[nm], seed0 + i, lr, self.out[3:4]) for i, nm in enumerate(self.names)])


def run(state):
    """One step; returns the losses with the scalar, {L0, L+, L-, g}, and the updated weights."""
    ctx, kind, step = state["ctx"], state["kind"], state["step"]
    state["step"] += 1
    if kind == "set":
        items, n = state["items"], len(state["layers"])
        for i in range(n):
            items[i].seed = 1000 * step + i
        ctx.step_many_raw(items, n, POWER_STEPS, EPS, state["lr"], state["flags"])
        return {"out": state["out"], "w": [w for w, _, _ in state["layers"]]}
    if kind == "layer":
        ctx.step(state["layer"], state["w"], state["x"], state["loss"], POWER_STEPS, EPS, state["lr"], step, 0, state["out"])
        return {"out": state["out"], "w": state["w"]}
    if kind == "decoder":
        model = state["model"]
        model.step(step, state["lr"])
        return {"out": model.out, "w": [model.w[nm] for nm in model.names]}
    out, seed0 = state["out"], 1000 * step
    for coef, column in ((EPS, 1), (-2.0 * EPS, 2)):
        for i, ((w, x, _), (desc, loss)) in enumerate(zip(state["layers"], state["desc"])):
            ctx.dense_perturb(w, seed0 + i, coef)
            ctx.layer_forward_sketch(desc, w, x, None, binding.SKETCH_NONE, None, 0, None, loss, out[i, column:column + 1])
    for i, (w, _, _) in enumerate(state["layers"]):
        ctx.dense_perturb(w, seed0 + i, EPS)
        ctx.two_point(out[i], EPS)
        ctx.dense_perturb(w, seed0 + i, -state["lr"], out[i, 3:4])
    return {"out": out, "w": [w for w, _, _ in state["layers"]]}


# ---- what a pass cannot do without -------------------------------------------------------------------------------
def _shapes(case):
    if case["kind"] in ("set", "dense"):
        return [(d_in, d_out) for _, d_in, d_out in SETS[case["set"]]]
    if case["kind"] == "layer":
        return [(case["d_in"], case["d_out"])]
    layer = synth.decoder_shapes(HIDDEN, HEADS, KV_HEADS, INTER)
    return [(layer[p][1], layer[p][0]) for p in synth.DECODER_PROJECTIONS] * case["layers"] + [(HIDDEN, VOCAB)]


def work(case):
    shapes, kind = _shapes(case), case["kind"]
    e = 4 if case.get("dtype") == "f32" else 2
    weights = sum(i * o for i, o in shapes)
    if kind == "decoder":
        n = case["seqs"] * case["seq_len"]
        read = 2 * n * HIDDEN + 12 * n                                    # embedding rows, ids and targets
    else:
        n = case["tokens"]
        if kind == "layer":
            read = e * n * case["d_in"] + (4 * n if case["loss"] == "ce" else e * n * case["d_out"])
        else:
            named = {SHARES_X.get(name, name): d_in for name, d_in, _ in SETS[case["set"]]}
            read = e * n * sum(named.values()) + e * n * sum(o for _, o in shapes)
    forwards = {"one_sided": 2, "shared": 1}.get(case.get("schedule"), 2 if kind == "dense" else 3)
    flops = 2.0 * n * weights * forwards
    if kind == "dense":
        flops += 4 * 2.0 * weights
    else:
        r = case["rank"]
        perturbed = 1 if case.get("schedule") == "one_sided" else 2
        flops += sum(2.0 * n * r * ((2 * POWER_STEPS + 2) * i + perturbed * o) + 2.0 * r * i * o for i, o in shapes)
    if kind == "decoder":                                                 # causal scores and values, three passes
        flops += 3 * case["layers"] * 2.0 * 2.0 * 128 * HEADS * case["seqs"] * case["seq_len"] * (case["seq_len"] + 1) / 2
    return {"bytes": float(read + 2 * e * weights), "flops": flops}


def tolerance(case):
    """Four times what a second implementation differed by, over the listed and drawn cases.  Single layers against Alg. 2
    in 64 bits (torch): fp32 storage 2e-9 (losses) and 1e-7 of one value (weights, one rounding); bf16 1e-6 (losses), 1e-5
    (weights: isolated one-ulp flips of the rounding, 2^-7 of one value).  Whole models against linear layers summed in
    another order: an ulp of a stored activation moves the losses by some 1e-5, and g by that over 2 eps, 3e-3 of the result
    for the fewest tokens."""
    if case["kind"] == "decoder":
        return {"rel": 1e-2, "max": 3e-2}
    return {"rel": 1e-7, "max": 1e-6} if case.get("dtype") == "f32" else {"rel": 1e-4, "max": 3e-2}
