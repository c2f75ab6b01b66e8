"""Timed cases of the AdaGC optimizer step: what a training program has this library do, through its public entry points.

A case names a parameter list (decoder-shaped or ragged), how the tensors lie in memory, the optimizer, the gradient
type, the clipping rule and the entry point.  ``prepare`` makes the state a training program holds in the middle of a
run (parameters, moments, moving averages of the norms, this step's gradients, the context); ``run`` is one optimizer
step; ``exact`` is the same step in 64 bits with plain torch.
"""
import ctypes
import math

import numpy as np
import torch

from paper_2502_11034_amd import binding as B
from paper_2502_11034_amd import workloads as W

DEV = "cuda:0"
STEP = 200                     # the step a state stands before: the moments' bias corrections are still alive
WARMUP = 1000                  # t_start of the cases that are still inside the warm-up
PAD = 256                      # "separate" layout: every tensor starts at a multiple of this many elements, as in an
                               # allocation of its own
MUON_NS = (3.4445, -4.7750, 2.0315)
MODES = {"adagc": B.ADAGC_MODE_ADAGC, "globalgc": B.ADAGC_MODE_GLOBALGC, "global_adagc": B.ADAGC_MODE_GLOBAL_ADAGC,
         "zclip": B.ADAGC_MODE_ZCLIP, "agc": B.ADAGC_MODE_AGC, "clippy": B.ADAGC_MODE_CLIPPY}


def _case(name=None, entry="step", shapes="gpt2", layout="separate", optimizer="adamw", grad="f32", copy=False,
          mode="adagc", warmup=False, report=False, **sizes):
    case = dict(entry=entry, shapes=shapes, layout=layout, optimizer=optimizer, grad=grad, copy=copy, mode=mode,
                warmup=warmup, report=report, **sizes)
    if name:
        case["name"] = name
    return case


def listed():
    return [
        # the smallest lists (a two-layer transformer of 0.5 M parameters): nothing but latency and launches
        _case("tiny_adamw", layers=2, d=128, ffn=512, vocab=1024, n_pos=0),
        # the same kind of program recorded once into a HIP graph and replayed for every step
        _case("small_graph_replay", entry="graph", layers=4, d=256, ffn=1024, vocab=4096, n_pos=256),
        # thousands of small tensors (adapters, biases, norms, per-channel scales): work per tensor counts, not bytes
        _case("many_small_tensors", shapes="ragged", tensors=5000, max_elems=32768, embed=0, list_seed=1),
        # GPT-2-small, fp32 throughout
        _case("gpt2_small_adamw", layers=12, d=768, ffn=3072, vocab=50257, n_pos=1024),
        # the first steps of a run: GlobalGC warm-up, with the per-tensor statistics read back for the log on each step
        _case("gpt2_small_warmup_logged", warmup=True, report=True, layers=12, d=768, ffn=3072, vocab=50257, n_pos=1024),
        # mixed precision (bf16 gradients, bf16 copies) through the entry point that allocates nothing
        _case("medium_static_bf16", entry="static", shapes="llama", grad="bf16", copy=True, layers=6, d=1024, heads=16,
              kv_heads=4, ffn=2816, vocab=32000),
        # update clipping (AGC), mixed precision
        _case("medium_agc", shapes="llama", mode="agc", grad="bf16", copy=True, layers=6, d=1024, heads=16, kv_heads=4,
              ffn=2816, vocab=32000),
        # a ragged list laid end to end in flat buffers, as flat-parameter and sharded optimizers keep it: odd sizes, odd
        # starting addresses
        _case("ragged_flat_buffers", shapes="ragged", layout="packed", tensors=1500, max_elems=4194304, embed=0, list_seed=2),
        # the large end: embedding, head and 4 layers of Llama-3-8B shapes, fp32 gradients and bf16 copies
        _case("llama3_8b_4_layers_adamw", shapes="llama", copy=True, layers=4, d=4096, heads=32, kv_heads=8, ffn=14336,
              vocab=128256),
        # the same with Lion on bf16 gradients
        _case("llama3_8b_4_layers_lion", shapes="llama", optimizer="lion", grad="bf16", copy=True, layers=4, d=4096, heads=32,
              kv_heads=8, ffn=14336, vocab=128256),
        # Muon on the hidden matrices of a small model: many matrices of a few hundred rows
        _case("muon_gpt2_small", entry="muon", optimizer="muon", grad="bf16", copy=True, layers=12, d=768, ffn=3072, vocab=50257,
              n_pos=1024),
        # Muon on the hidden matrices of 4 layers of Llama-3-8B shapes: the matrix products are everything
        _case("muon_llama3_8b_4_layers", entry="muon", shapes="llama", optimizer="muon", layers=4, d=4096, heads=32, kv_heads=8,
              ffn=14336, vocab=128256),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the listed ranges: any list shape, layout, optimizer, type, rule and entry point that go together."""
    if rng.random() < 0.25:
        options = dict(entry="muon", optimizer="muon", grad=rng.choice(["f32", "bf16"]), copy=rng.random() < 0.5,
                       layout=rng.choice(["separate", "separate", "packed"]), mode=rng.choice(["adagc", "adagc", "globalgc"]))
        if rng.random() < 0.5:                   # odd matrices, a few of each shape
            return _case(shapes="matrices", kinds=rng.randint(1, 3), per_kind=rng.randint(1, 8), rows=_log_uniform(rng, 65, 2500),
                         cols=_log_uniform(rng, 65, 5000), list_seed=rng.randint(1, 10 ** 6), **options)
        d = 64 * rng.randint(2, 16)
        return _case(shapes="gpt2", layers=rng.randint(1, 8), d=d, ffn=4 * d, vocab=1000, n_pos=0, **options)
    entry = rng.choice(["step", "step", "step", "graph", "static"])
    options = dict(entry=entry, optimizer=rng.choice(["adamw", "adamw", "lion"]), grad=rng.choice(["f32", "bf16"]),
                   copy=rng.random() < 0.5, layout=rng.choice(["separate", "separate", "packed"]),
                   mode=rng.choice(["adagc", "adagc", "adagc", "globalgc", "global_adagc", "zclip"] +
                                   (["agc", "clippy"] if entry == "step" else [])),
                   warmup=rng.random() < 0.2, report=entry == "step" and rng.random() < 0.2)
    shape = rng.choice(["gpt2", "llama", "ragged"])
    if shape == "ragged":
        return _case(shapes="ragged", tensors=_log_uniform(rng, 8, 4000), max_elems=_log_uniform(rng, 256, 2 ** 22),
                     embed=rng.choice([0, 0, _log_uniform(rng, 10 ** 4, 10 ** 8) | 1]), list_seed=rng.randint(1, 10 ** 6), **options)
    if shape == "gpt2":
        d = _log_uniform(rng, 60, 1600)
        return _case(shapes="gpt2", layers=rng.randint(1, 16), d=d, ffn=4 * d, vocab=_log_uniform(rng, 257, 50257),
                     n_pos=rng.choice([0, 256, 1024]), **options)
    heads = rng.choice([4, 8, 16, 32])
    d = heads * rng.choice([32, 64, 80, 96, 128])
    return _case(shapes="llama", layers=rng.randint(1, 4), d=d, heads=heads, kv_heads=heads // rng.choice([1, 2, 4]),
                 ffn=int(d * rng.uniform(2.5, 3.5)), vocab=_log_uniform(rng, 1000, 128256), **options)


# ------------------------------------------------------------------------------------------------ the list of a case

def _shapes(case):
    """Shapes of the case's tensors, in list order."""
    kind = case["shapes"]
    if kind == "gpt2":
        specs = W.gpt2_like_list(case["layers"], case["d"], case["ffn"], case["vocab"], case["n_pos"])
    elif kind == "llama":
        specs = W.llama_like_list(case["layers"], case["d"], case["heads"], case["kv_heads"], case["ffn"], case["vocab"])
    elif kind == "ragged":
        specs = W.ragged_stress_list(case["tensors"], case["max_elems"], None, seed=case["list_seed"])
        if case["embed"]:
            specs.append(W.TensorSpec("embed", (case["embed"],), "matrix"))
    else:
        rng = np.random.Generator(np.random.PCG64(case["list_seed"]))
        sides = [(case["rows"], case["cols"])]
        while len(sides) < case["kinds"]:
            sides.append((int(rng.integers(65, case["rows"] + 66)), int(rng.integers(65, case["cols"] + 66))))
        return [s for s in sides for _ in range(case["per_kind"])]
    if case["entry"] == "muon":                  # Muon is for the hidden matrices; the rest stays with AdamW
        specs = [s for s in specs if len(s.shape) == 2 and "." in s.name]
    return [s.shape for s in specs]


class _Layout:
    """Where the tensors of a list lie in flat buffers."""

    def __init__(self, case):
        self.shapes = _shapes(case)
        self.numels = [int(np.prod(s)) for s in self.shapes]
        pad = PAD if case["layout"] == "separate" else 1
        self.counts = [-(-n // pad) * pad for n in self.numels]
        self.starts = [0] + [int(x) for x in np.cumsum(self.counts)]
        self.total = self.starts.pop()
        self.n = len(self.numels)

    def views(self, flat):
        return [flat[s:s + n] for s, n in zip(self.starts, self.numels)]

    def per_element(self, per_tensor):
        return torch.repeat_interleave(torch.tensor(per_tensor, dtype=torch.float32, device=DEV),
                                       torch.tensor(self.counts, device=DEV), output_size=self.total)

    def inside(self):
        """1 in the tensors, 0 in the gaps between them."""
        runs = [x for n, c in zip(self.numels, self.counts) for x in (n, c - n)]
        values = torch.tensor([1.0, 0.0], device=DEV).repeat(self.n)
        return torch.repeat_interleave(values, torch.tensor(runs, device=DEV), output_size=self.total)


def _hyper(case):
    hp = dict(lr=3e-4, beta1=0.9, beta2=0.95, weight_decay=0.1, t_start=WARMUP if case["warmup"] else 100, lambda_abs=1.0,
              clip_mode=MODES[case["mode"]])
    if case["optimizer"] == "lion":
        hp.update(lr=1e-4, beta2=0.99)
    if case["optimizer"] == "muon":
        hp.update(lr=0.02)
    if case["mode"] == "zclip":
        hp.update(ema_beta=0.97, z_thres=2.0)
    elif case["mode"] == "agc":
        hp.update(lambda_rel=1e-3)
    elif case["mode"] == "clippy":
        hp.update(lambda_rel=1e-2, lambda_abs=0.5)
    return B.make_hyper(**hp)


def _inputs(case, seed, layout, into=None):
    """The buffers of one state, from the seed: gradients N(0, sigma_i^2) with sigma_i log-uniform in [1e-4, 1e-1] and one
    tensor in twenty spiking by 50, moments of that scale, gamma_i near the norm of an ordinary gradient.  `into`: refill
    these buffers."""
    rng = np.random.Generator(np.random.PCG64(int(seed)))
    gen = torch.Generator(device=DEV)
    gen.manual_seed(int(seed) * 2654435761 % (1 << 62) + 1)
    sigma = np.exp(rng.uniform(math.log(1e-4), math.log(1e-1), layout.n))
    spiked = sigma * np.where(rng.random(layout.n) < 0.05, 50.0, 1.0)
    norms = sigma * np.sqrt(np.asarray(layout.numels, dtype=np.float64)) * rng.uniform(0.9, 1.1, layout.n)
    inside = layout.inside()

    def normal():
        return torch.empty(layout.total, dtype=torch.float32, device=DEV).normal_(0.0, 1.0, generator=gen).mul_(inside)

    scale = layout.per_element(sigma)
    bufs = {"p": normal().mul_(0.02), "g": normal().mul_(layout.per_element(spiked))}
    if case["grad"] == "bf16":
        bufs["g"] = bufs["g"].to(torch.bfloat16)
    bufs["m"] = normal().mul_(scale).mul_(0.2)
    if case["optimizer"] == "adamw":
        bufs["v"] = normal().mul_(scale).square_().mul_(0.5).add_(scale.square_().mul_(0.5).mul_(inside))
    if case["copy"]:
        bufs["c"] = bufs["p"].to(torch.bfloat16)
    gamma = norms.copy()
    model = math.sqrt(float(np.sum(norms ** 2)))
    if case["mode"] == "global_adagc":
        gamma[:] = 0.0
        gamma[0] = model
    elif case["mode"] == "zclip":
        gamma = np.zeros(max(layout.n, 2))
        gamma[0], gamma[1] = model, (0.05 * model) ** 2
    bufs["ema"] = torch.tensor(gamma, dtype=torch.float32, device=DEV)
    if into is not None:
        for k, t in bufs.items():
            into[k].copy_(t)
        return into
    return bufs


# ------------------------------------------------------------------------------------------------ prepare and run

def prepare(case, seed):
    layout = _Layout(case)
    bufs = _inputs(case, seed, layout)
    state = {"case": case, "layout": layout, "bufs": bufs, "step": STEP, "hp": _hyper(case)}
    # a training loop keeps the pointer arrays of its tensors, which stay where they are
    for k in ("p", "g", "m", "v", "c"):
        state["ptr_" + k] = B.ptr_array(layout.views(bufs[k])) if k in bufs else None
    if case["entry"] == "static":
        state["norms"] = torch.zeros(layout.n, dtype=torch.float32, device=DEV)
        state["coefs"] = torch.zeros(layout.n, dtype=torch.float32, device=DEV)
        return state
    optimizer = {"adamw": B.ADAGC_OPT_ADAMW, "lion": B.ADAGC_OPT_LION, "muon": B.ADAGC_OPT_MUON}[case["optimizer"]]
    ctx = B.AdaGC(layout.numels, optimizer, B.ADAGC_GRAD_BF16 if case["grad"] == "bf16" else B.ADAGC_GRAD_F32, case["copy"],
                  telemetry=case["report"], update_clipping=case["mode"] in ("agc", "clippy"))
    state["ctx"] = ctx
    if case["copy"]:
        ctx.set_param_copies(state["ptr_c"])
    if case["entry"] == "muon":
        ctx.muon_attach(layout.shapes)
        state["mh"] = B.make_muon_hyper()
    if case["entry"] == "graph":
        _record(state, seed)
    return state


def _record(state, seed):
    """One eager step, then the step recorded; the eager step's effect is taken back by filling the buffers again."""
    state["sp"] = torch.frombuffer(bytearray(B.step_params_bytes(state["hp"], STEP)), dtype=torch.uint8).to(DEV)
    state["sp_step"] = state["sp"].view(torch.int64)[B.adagc_step_params.step.offset // 8:][:1]
    torch.cuda.synchronize()

    def call():
        state["ctx"].step_graph(state["ptr_p"], state["ptr_g"], state["ptr_m"], state["ptr_v"], state["bufs"]["ema"], state["sp"],
                                stream=torch.cuda.current_stream().cuda_stream)
    call()
    torch.cuda.synchronize()
    state["graph"] = torch.cuda.CUDAGraph()
    with torch.cuda.graph(state["graph"]):
        call()
    _inputs(state["case"], seed, state["layout"], state["bufs"])
    torch.cuda.synchronize()


def run(state):
    case, bufs = state["case"], state["bufs"]
    state["step"] += 1
    stream = torch.cuda.current_stream().cuda_stream
    if case["entry"] == "graph":
        state["sp_step"].add_(1)
        state["graph"].replay()
    elif case["entry"] == "static":
        B.adagc_step_static(state["layout"].numels, state["ptr_p"], state["ptr_g"], state["ptr_m"], state["ptr_v"], bufs["ema"],
                            state["hp"], state["step"],
                            optimizer=B.ADAGC_OPT_LION if case["optimizer"] == "lion" else B.ADAGC_OPT_ADAMW,
                            grad_dtype=B.ADAGC_GRAD_BF16 if case["grad"] == "bf16" else B.ADAGC_GRAD_F32,
                            params_bf16=state["ptr_c"], out_norms=state["norms"], out_coefs=state["coefs"], stream=stream)
    elif case["entry"] == "muon":
        state["ctx"].muon_step(state["ptr_p"], state["ptr_g"], state["ptr_m"], bufs["ema"], state["hp"], state["mh"], state["step"],
                               stream=stream)
    else:
        state["ctx"].step(state["ptr_p"], state["ptr_g"], state["ptr_m"], state["ptr_v"], bufs["ema"], state["hp"], state["step"],
                          stream=stream)
    out = {k: bufs[k] for k in ("p", "m", "v", "c", "ema") if k in bufs}
    if case["entry"] == "static":
        out.update(norms=state["norms"], coefs=state["coefs"])
    if case["report"]:
        out["norms"], out["coefs"], out["clipped"] = state["ctx"].get_norms(stream)
        out["m_norms"], out["v_norms"], out["update_norms"] = state["ctx"].get_state_norms(stream)
    return out


# ------------------------------------------------------------------------------------------------ work and tolerance

def work(case):
    """Each array once in and once out; Muon's products with the symmetric ones computed by half."""
    layout = _Layout(case)
    n = sum(layout.numels)
    grad = 2 if case["grad"] == "bf16" else 4
    state_arrays = 3 if case["optimizer"] == "adamw" else 2
    byts = n * (grad + 8 * state_arrays + (2 if case["copy"] else 0)) + 8 * layout.n
    flops = 20.0 * n
    if case["entry"] == "muon":
        for r, c in layout.shapes:
            a, b = min(r, c), max(r, c)
            flops += 5 * (3.0 * a * a * b + 1.0 * a * a * a)
    return {"bytes": float(byts), "flops": flops}


def tolerance(case):
    """Everything is stored once in fp32 from sums and formulas in 64 bits, so two implementations differ by an fp32
    rounding of single values; a bf16 copy then by one of its steps.  Muon's iteration is stored in bf16 between its
    products: see _MUON_TOLERANCE."""
    if case["entry"] == "muon":
        return dict(_MUON_TOLERANCE, max=0.016 if case["copy"] else _MUON_TOLERANCE["max"])
    return {"rel": 2.5e-7, "max": 0.016 if case["copy"] else 1e-6, "differ": 1e-3}


# theta after the step against theta after the same step with the products in 64 bits and no rounding of X between them
_MUON_TOLERANCE = {"rel": 1e-3, "max": 1e-2}


# ------------------------------------------------------------------------------------------------ the step in 64 bits

def _gradient_rule(case, hp, ema, norms, step):
    """(per-tensor coefficients, clipped flags, new ema) of the rules that act on the gradient."""
    n = norms.numel()
    model = norms.square().sum().sqrt()
    warm = step <= hp.t_start
    one = torch.ones_like(norms)
    mode = case["mode"]
    beta = float(hp.ema_beta)
    if mode == "adagc" and not warm:
        threshold = hp.lambda_rel * ema[:n]
        active = norms > threshold
        return torch.where(active, threshold / norms, one), active, beta * ema + (1 - beta) * torch.where(active, threshold, norms)
    new = ema.clone()
    if mode == "global_adagc" and not warm:
        threshold = hp.lambda_rel * ema[0]
        active = model > threshold
        h = torch.where(active, threshold / model, one[0])
        new[0] = beta * ema[0] + (1 - beta) * torch.where(active, threshold, model)
    elif mode == "zclip" and not warm:
        mu, var = ema[0], ema[1]
        z = (model - mu) / var.sqrt()
        active = z > hp.z_thres
        tau = mu + hp.z_thres ** 2 / z * var.sqrt()
        h = torch.where(active, tau / model, one[0])
        clipped = torch.where(active, tau, model)
        new[0] = beta * mu + (1 - beta) * clipped
        new[1] = beta * var + (1 - beta) * (clipped - new[0]) ** 2
    else:
        active = model > hp.lambda_abs
        h = torch.where(active, hp.lambda_abs / model, one[0])
        if mode == "adagc":
            new = torch.minimum(ema, h * norms)
        elif mode == "global_adagc":
            new[0] = torch.minimum(ema[0], h * model)
        elif mode == "zclip":
            new[0] = beta * ema[0] + (1 - beta) * h * model
            new[1] = beta * ema[1] + (1 - beta) * (h * model - new[0]) ** 2
    return h * one, active.expand(n), new


def _orthogonalise(u):
    a, b, c = MUON_NS
    tall = u.shape[0] > u.shape[1]
    x = u / (u.norm() + 1e-7)
    x = x.t().contiguous() if tall else x
    for _ in range(5):
        gram = x @ x.t()
        x = a * x + (b * gram + c * (gram @ gram)) @ x
    return x.t() if tall else x


def exact(case, seed):
    layout = _Layout(case)
    bufs = _inputs(case, seed, layout)
    hp, step = _hyper(case), STEP + 1
    ema = bufs["ema"].double()
    g, p, m = (layout.views(bufs[k]) for k in ("g", "p", "m"))
    v = layout.views(bufs["v"]) if "v" in bufs else None
    out = {k: torch.zeros(layout.total, dtype=torch.float64, device=DEV) for k in ("p", "m", "v") if k in bufs}
    new = {k: layout.views(t) for k, t in out.items()}
    lr, b1, b2, wd = float(hp.lr), float(hp.beta1), float(hp.beta2), float(hp.weight_decay)
    c1, c2 = 1 - b1 ** step, 1 - b2 ** step
    direction_norms = torch.zeros(layout.n, dtype=torch.float64, device=DEV)
    if case["mode"] in ("agc", "clippy"):
        coef, active, new_ema = torch.ones(layout.n, dtype=torch.float64, device=DEV), None, ema
        norms = direction_norms
    else:
        norms = torch.stack([x.double().square().sum() for x in g]).sqrt()
        coef, active, new_ema = _gradient_rule(case, hp, ema, norms, step)
    update_coef = []
    for i in range(layout.n):
        gh = g[i].double() * coef[i]
        pi, mi = p[i].double(), m[i].double()
        if case["entry"] == "muon":
            r, c = layout.shapes[i]
            new["m"][i].copy_(0.95 * mi + gh)
            o = _orthogonalise((gh + 0.95 * new["m"][i]).view(r, c)).reshape(-1)
            new["p"][i].copy_(pi - lr * (wd * pi + math.sqrt(max(1.0, r / c)) * o))
            continue
        if case["optimizer"] == "adamw":
            new["m"][i].copy_(b1 * mi + (1 - b1) * gh)
            new["v"][i].copy_(b2 * v[i].double() + (1 - b2) * gh * gh)
            delta = (new["m"][i] / c1) / ((new["v"][i] / c2).sqrt() + float(hp.eps))
        else:
            delta = torch.sign(b1 * mi + (1 - b1) * gh)
            new["m"][i].copy_(b2 * mi + (1 - b2) * gh)
        uc = torch.ones((), dtype=torch.float64, device=DEV)
        if case["mode"] == "agc":
            direction_norms[i] = delta.norm()
            uc = torch.minimum(uc, float(hp.lambda_rel) * pi.norm() / direction_norms[i])
        elif case["mode"] == "clippy":
            direction_norms[i] = delta.abs().max()
            uc = torch.minimum(uc, (float(hp.lambda_rel) * pi.abs().max() + float(hp.lambda_abs)) / (lr * direction_norms[i]))
        update_coef.append(uc)
        new["p"][i].copy_(pi - lr * (uc * delta + wd * pi))
    if "c" in bufs:
        out["c"] = out["p"]
    out["ema"] = new_ema
    if active is None:
        coef = torch.stack(update_coef)
        active = coef < 1.0
    if case["entry"] == "static" or case["report"]:
        out["norms"], out["coefs"] = norms, coef
    if case["report"]:
        out["clipped"] = active.to(torch.uint8)
        out["m_norms"] = torch.stack([x.norm() for x in new["m"]])
        out["v_norms"] = torch.stack([x.norm() for x in new["v"]]) if v is not None else torch.zeros_like(norms)
        out["update_norms"] = torch.stack([(x - y.double()).norm() for x, y in zip(new["p"], p)])
    return out
