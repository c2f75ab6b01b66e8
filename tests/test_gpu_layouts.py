"""The step on tensors of every size around the kernels' tiles and work items, laid end to end without gaps (every alignment to an
element, as in flat parameter buffers), must be bit for bit the step on the same tensors in allocations of their own: the kernels
take both through the same vectors, and neither the address nor the place in the visiting order enters a result.  The step on
separate allocations is held against the oracle elsewhere."""
import ctypes
import functools
from fractions import Fraction

import numpy as np
import pytest
import torch

from paper_2502_11034_amd import binding as B
from paper_2502_11034_amd import workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# one below, at and above: a vector, a round of a workgroup, the work items (2048, 4096), a chunk (16384) and its last item
SIZES = [1, 2, 3, 4, 5, 7, 255, 1023, 1024, 1025, 2047, 2048, 2049, 4095, 4096, 4097, 4101, 8191, 8193, 12287, 12289, 16383, 16384, 16385,
         16387, 18431, 18433, 20480, 20481, 32767, 49157, 6, 70001]


def _run(numels, flat, optimizer, grad_dtype, mode, entry, steps, seed=5):
    """State after `steps` steps: flat tensors p, m, v, copies, gamma, and the reported norms."""
    rng = np.random.default_rng(seed)
    starts = [0]
    for n in numels:
        starts.append(starts[-1] + n)
    total = starts[-1]
    host = {"p": rng.standard_normal(total) * 0.02, "g": rng.standard_normal(total) * 0.01, "m": rng.standard_normal(total) * 0.002,
            "v": rng.random(total) * 1e-4 + 1e-6}
    types = {"p": torch.float32, "g": torch.bfloat16 if grad_dtype == B.ADAGC_GRAD_BF16 else torch.float32, "m": torch.float32,
             "v": torch.float32, "c": torch.bfloat16}
    host["c"] = np.zeros(total)
    lists = {}
    for k, values in host.items():
        whole = torch.from_numpy(values).to(types[k]).to(DEV)
        views = [whole[a:b] for a, b in zip(starts, starts[1:])]
        lists[k] = views if flat else [x.clone() for x in views]
    lion = optimizer == B.ADAGC_OPT_LION
    gamma = torch.tensor([0.009 * n ** 0.5 for n in numels], dtype=torch.float32, device=DEV)
    hp = B.make_hyper(lr=1e-3, t_start=0, clip_mode=mode, lambda_rel=1e-3 if mode == B.ADAGC_MODE_AGC else 1.04)
    v = None if lion else lists["v"]
    extra = []
    if entry == "static":
        for t in range(7, 7 + steps):
            B.adagc_step_static(numels, lists["p"], lists["g"], lists["m"], v, gamma, hp, t, optimizer=optimizer, grad_dtype=grad_dtype,
                                params_bf16=lists["c"])
    else:
        ctx = B.AdaGC(numels, optimizer, grad_dtype, True, telemetry=True, update_clipping=mode == B.ADAGC_MODE_AGC)
        ctx.set_param_copies(lists["c"])
        for t in range(7, 7 + steps):
            ctx.step(lists["p"], lists["g"], lists["m"], v, gamma, hp, t)
        extra = [torch.from_numpy(x.copy()) for x in ctx.get_norms() + ctx.get_state_norms()]
        ctx.close()
    torch.cuda.synchronize()
    return [torch.cat(lists[k]) for k in ("p", "m", "v", "c")] + [gamma] + extra


@pytest.mark.parametrize("entry", ["step", "static"])
@pytest.mark.parametrize("grad_dtype", [B.ADAGC_GRAD_F32, B.ADAGC_GRAD_BF16])
@pytest.mark.parametrize("optimizer", [B.ADAGC_OPT_ADAMW, B.ADAGC_OPT_LION])
def test_flat_buffers_equal_separate_allocations(optimizer, grad_dtype, entry):
    a, b = (_run(SIZES, flat, optimizer, grad_dtype, B.ADAGC_MODE_ADAGC, entry, 2) for flat in (True, False))
    for k, (x, y) in enumerate(zip(a, b)):
        assert torch.equal(x, y), "array %d" % k


@pytest.mark.parametrize("optimizer", [B.ADAGC_OPT_ADAMW, B.ADAGC_OPT_LION])
def test_flat_buffers_equal_separate_allocations_with_update_clipping(optimizer):
    a, b = (_run(SIZES, flat, optimizer, B.ADAGC_GRAD_BF16, B.ADAGC_MODE_AGC, "step", 2) for flat in (True, False))
    for k, (x, y) in enumerate(zip(a, b)):
        assert torch.equal(x, y), "array %d" % k


def test_static_step_equals_step_on_many_small_tensors():
    """More tensors than one table launch takes, most of them shorter than a work item."""
    numels = [int(s.numel) for s in W.ragged_stress_list(700, 30000, None, seed=3)]
    a = _run(numels, True, B.ADAGC_OPT_ADAMW, B.ADAGC_GRAD_F32, B.ADAGC_MODE_ADAGC, "static", 2)
    b = _run(numels, False, B.ADAGC_OPT_ADAMW, B.ADAGC_GRAD_F32, B.ADAGC_MODE_ADAGC, "step", 2)
    for k, (x, y) in enumerate(zip(a, b)):
        assert torch.equal(x, y), "array %d" % k


@pytest.mark.parametrize("split,unroll", [(1, 4), (2, 2), (4, 1), (8, 2), (16, 1)])
@pytest.mark.parametrize("optimizer", [B.ADAGC_OPT_ADAMW, B.ADAGC_OPT_LION])
def test_update_clipping_with_every_size_of_work_item(optimizer, split, unroll):
    """The direction's norms are summed over the update's work items, which may be smaller than a round of its loads: the
    coefficients and the step must be the default's up to the order of summation (maxima: exactly)."""
    numels = SIZES
    gen = torch.Generator(device="cpu").manual_seed(9)
    make = lambda scale: [(torch.randn(n, generator=gen) * scale).to(DEV) for n in numels]
    p0, g, m0 = make(0.02), make(0.01), make(0.002)
    v0 = [x.square() + 1e-6 for x in m0]
    for mode in (B.ADAGC_MODE_AGC, B.ADAGC_MODE_CLIPPY):
        hp = B.make_hyper(lr=1e-3, t_start=0, clip_mode=mode, lambda_rel=1e-3 if mode == B.ADAGC_MODE_AGC else 1e-2,
                          lambda_abs=1e-5 if mode == B.ADAGC_MODE_CLIPPY else 1.0)
        results = []
        for kw in ({}, dict(update_split=split, unroll=unroll)):
            p, m, v = ([x.clone() for x in lst] for lst in (p0, m0, v0))
            gamma = torch.ones(len(numels), device=DEV)
            ctx = B.AdaGC(numels, optimizer, update_clipping=True, **kw)
            ctx.step(p, g, m, None if optimizer == B.ADAGC_OPT_LION else v, gamma, hp, 3)
            norms, coefs, flags = ctx.get_norms()
            ctx.close()
            results.append((torch.cat(p), norms, coefs, flags))
        a, b = results
        assert a[3].any()
        np.testing.assert_allclose(a[1], b[1], rtol=2e-7)            # two fp32 roundings of sums that differ by 1e-13
        np.testing.assert_allclose(a[2], b[2], rtol=2e-7)
        assert np.array_equal(a[3], b[3])
        assert ((a[0] - b[0]).abs() <= 2e-7 * a[0].abs() + 1e-12).all()


@pytest.mark.parametrize("entry", ["step", "graph", "static"])
@pytest.mark.parametrize("n", [1, 2, 191, 192, 193, 511, 512, 513, 1700])
def test_model_wide_rules_on_short_and_long_lists(n, entry):
    """Up to 192 tensors the last workgroup of the rules kernel evaluates a model-wide rule, beyond that a kernel of its own:
    the warm-up branch, the model's coefficient and its running minimum, and GlobalGC, on both sides of that line, several steps
    in a row (the count starts each at zero)."""
    rng = np.random.default_rng(n)
    numels = [int(x) for x in rng.integers(1, 40, n)]
    numels[-1] = 50000
    g = [torch.from_numpy(rng.standard_normal(k).astype(np.float32)).to(DEV) for k in numels]
    norms = np.array([float(x.double().norm()) for x in g])
    model = float(np.sqrt((norms ** 2).sum()))
    p, m = ([torch.zeros_like(x) for x in g] for _ in range(2))
    v = [torch.zeros_like(x) for x in g]
    gamma = torch.full((n,), 1e9, dtype=torch.float32, device=DEV)
    out_n, out_c = torch.zeros(n, device=DEV), torch.zeros(n, device=DEV)
    out_f = torch.zeros(n, dtype=torch.uint8, device=DEV)
    ctx = None if entry == "static" else B.AdaGC(numels)
    sp = torch.zeros(56, dtype=torch.uint8, device=DEV)
    least = np.full(n, 1e9)
    for step, (threshold, mode) in enumerate([(0.5 * model, B.ADAGC_MODE_ADAGC), (0.25 * model, B.ADAGC_MODE_ADAGC),
                                              (2.0 * model, B.ADAGC_MODE_GLOBALGC), (0.1 * model, B.ADAGC_MODE_GLOBALGC)], start=2):
        hp = B.make_hyper(t_start=100, lambda_abs=threshold, clip_mode=mode)
        if entry == "step":
            ctx.step(p, g, m, v, gamma, hp, step)
        elif entry == "graph":
            sp.copy_(torch.frombuffer(bytearray(B.step_params_bytes(hp, step)), dtype=torch.uint8))
            ctx.step_graph(p, g, m, v, gamma, sp)
        else:
            B.adagc_step_static(numels, p, g, m, v, gamma, hp, step, out_norms=out_n, out_coefs=out_c, out_clipped=out_f)
        got = ctx.get_norms() if ctx else tuple(x.cpu().numpy() for x in (out_n, out_c, out_f))
        h = min(1.0, float(np.float32(threshold)) / model)
        np.testing.assert_allclose(got[0], norms, rtol=2e-7)
        np.testing.assert_allclose(got[1], np.full(n, h), rtol=2e-7)
        assert (got[2] == (1 if h < 1.0 else 0)).all()
        if mode == B.ADAGC_MODE_ADAGC:
            least = np.minimum(least, h * norms)
        np.testing.assert_allclose(gamma.cpu().numpy(), least, rtol=2e-7)
    if ctx:
        ctx.close()


def test_steps_that_overlap_leave_nothing_behind():
    """Steps of one context share its scratch and have to be ordered by the caller.  Where that is missed the overlapping steps'
    own results mean nothing, but the next properly ordered step must be right again: the count by which the rules kernel finds
    its last workgroup starts every step at zero, whatever value it was left at."""
    n = 192
    rng = np.random.default_rng(4)
    numels = [int(x) for x in rng.integers(1, 3000, n)]
    state = lambda: [[torch.zeros(k, device=DEV) for k in numels] for _ in range(3)]
    g = [torch.from_numpy(rng.standard_normal(k).astype(np.float32)).to(DEV) for k in numels]
    norms = np.array([float(x.double().norm()) for x in g])
    model = float(np.sqrt((norms ** 2).sum()))
    gamma = torch.ones(n, device=DEV)
    ctx = B.AdaGC(numels)
    p, m, v = state()
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    lists = [B.ptr_array(x) for x in (p, g, m, v)]
    hp = B.make_hyper(t_start=0, lambda_abs=0.5 * model, clip_mode=B.ADAGC_MODE_GLOBALGC)
    ctx.step(*lists, gamma, hp, 2)               # the pointer table is uploaded once, before the steps that overlap
    torch.cuda.synchronize()
    for _ in range(50):
        for s in streams:
            ctx.step(*lists, gamma, hp, 2, stream=s.cuda_stream)
    torch.cuda.synchronize()
    for k, part in enumerate((0.25, 2.0, 0.125)):
        p, m, v = state()
        hp = B.make_hyper(t_start=0, lambda_abs=part * model, clip_mode=B.ADAGC_MODE_GLOBALGC)
        ctx.step(p, g, m, v, gamma, hp, 3 + k)
        got = ctx.get_norms()
        h = min(1.0, float(np.float32(part * model)) / model)
        np.testing.assert_allclose(got[0], norms, rtol=2e-7)
        np.testing.assert_allclose(got[1], np.full(n, h), rtol=2e-7)
        assert (got[2] == (1 if h < 1.0 else 0)).all()
    ctx.close()


# The rule's two limits, 64 chunks of a tensor and 16384 work items of 2048 elements with AdamW, 8192 with Lion: at them and one
# beyond, in whole chunks and in short ones.
FUSED = {"64_chunks": [64 * 16384, 5], "65_chunks": [64 * 16384 + 1, 5], "ragged_64th": [63 * 16384 + 1, 16385],
         "16384_long_adamw": [64 * 16384] * 32, "16385_long_adamw": [64 * 16384] * 32 + [1],
         "8192_long_lion": [64 * 16384] * 16, "8193_long_lion": [64 * 16384] * 16 + [1],
         "16384_short_adamw": [4096] * 8192, "16385_short_adamw": [4096] * 8192 + [1],
         "8192_short_lion": [4096] * 4096, "8193_short_lion": [4096] * 4096 + [1], "one": [1], "tiny_and_long": [1000] * 300 + [17000]}


@pytest.mark.parametrize("numels", FUSED.values(), ids=FUSED.keys())
@pytest.mark.parametrize("optimizer", [B.ADAGC_OPT_ADAMW, B.ADAGC_OPT_LION])
def test_rule_in_the_update_equals_the_rules_kernel(optimizer, numels):
    """Small lists evaluate the per-tensor rule in the update kernel (adagc_step and adagc_step_static, each by its own look at the
    list), adagc_step_graph always in the rules kernel: the same norms, coefficients, flags and gammas bit for bit on both sides
    of both limits, and the same step up to the last bit of the bias corrections (the device's pow against the host's), several
    steps in a row."""
    gen = torch.Generator(device="cpu").manual_seed(len(numels))
    g = [(torch.randn(n, generator=gen) * 0.01).to(DEV) for n in numels]
    lion = optimizer == B.ADAGC_OPT_LION
    sp = torch.zeros(56, dtype=torch.uint8, device=DEV)
    results = []
    for entry in ("graph", "step", "static"):
        p, m, v = ([torch.full_like(x, c) for x in g] for c in (0.02, 0.001, 1e-4))
        state = (p, g, m, None if lion else v)
        gamma = torch.tensor([(0.005 if i % 2 else 0.02) * n ** 0.5 for i, n in enumerate(numels)], dtype=torch.float32, device=DEV)
        outs = [torch.zeros(len(numels), dtype=t, device=DEV) for t in (torch.float32, torch.float32, torch.uint8)]
        ctx = None if entry == "static" else B.AdaGC(numels, optimizer)
        seen = []
        for step in (5, 6, 7):
            hp = B.make_hyper(lr=1e-3, t_start=0)
            if entry == "graph":
                sp.copy_(torch.frombuffer(bytearray(B.step_params_bytes(hp, step)), dtype=torch.uint8))
                ctx.step_graph(*state, gamma, sp)
            elif entry == "step":
                ctx.step(*state, gamma, hp, step)
            else:
                B.adagc_step_static(numels, *state, gamma, hp, step, optimizer=optimizer, out_norms=outs[0], out_coefs=outs[1],
                                    out_clipped=outs[2])
            seen += list(ctx.get_norms()) if ctx else [x.cpu().numpy() for x in outs]
            seen.append(gamma.cpu().numpy())
        if ctx:
            ctx.close()
        results.append((seen, torch.cat(p), torch.cat(m), torch.cat(v)))
    a, *sa = results[0]
    for b, *sb in results[1:]:
        for x, y in zip(a, b):
            assert np.array_equal(x, y)
        for x, y in zip(sa, sb):
            assert ((x - y).abs() <= 2e-7 * y.abs()).all()


# chunks of every number of work items, one element below, at and above it
ITEMS = [k * 2048 + d for k in range(1, 9) for d in (-1, 0, 1)]
MI = 1 << 20
ITEM_LISTS = {"a small list": ITEMS,                                      # short chunks: up to half of a chunk's items
              "a large list": ITEMS + [33 * MI],                          # one item
              "a large list of small tensors": ITEMS + [5600] * 6100,     # half again
              "the rule in the update kernel, AdamW": [64 * 16384] * 32, "one more": [64 * 16384] * 32 + [1],
              "the rule in the update kernel, Lion": [64 * 16384] * 16, "Lion, one more": [1] + [64 * 16384] * 16}


@pytest.mark.parametrize("optimizer", [B.ADAGC_OPT_ADAMW, B.ADAGC_OPT_LION])
@pytest.mark.parametrize("name", ITEM_LISTS)
def test_work_items_of_every_chunk(name, optimizer):
    """Which chunks are cut into items of a table, which are numbered with empty ones, and whether the rule is in the update kernel depends
    on the list; the results do not: the library's own choice, whole chunks, and the entry point that builds its tables on the GPU."""
    numels, results = ITEM_LISTS[name], []
    gen = torch.Generator(device=DEV).manual_seed(11)
    total = sum(numels)
    host = {"p": 0.02, "g": 0.01, "m": 0.002, "v": 1e-4}
    host = {k: torch.randn(total, generator=gen, device=DEV).mul_(x) for k, x in host.items()}
    host["v"].square_()
    hp = B.make_hyper(lr=1e-3, t_start=0)
    for kw in ({}, dict(update_split=1, unroll=4), None):
        lists = {k: [y.clone() for y in x.split(numels)] for k, x in host.items()}
        gamma = torch.tensor([(0.012, 0.009)[i % 2] * n ** 0.5 for i, n in enumerate(numels)], dtype=torch.float32, device=DEV)
        v = lists["v"] if optimizer == B.ADAGC_OPT_ADAMW else None
        norms, coefs = torch.zeros(len(numels), device=DEV), torch.zeros(len(numels), device=DEV)
        if kw is None:
            B.adagc_step_static(numels, lists["p"], lists["g"], lists["m"], v, gamma, hp, 7, optimizer=optimizer, out_norms=norms, out_coefs=coefs)
        else:
            ctx = B.AdaGC(numels, optimizer, **kw)
            ctx.step(lists["p"], lists["g"], lists["m"], v, gamma, hp, 7)
            norms, coefs = (torch.from_numpy(x).to(DEV) for x in ctx.get_norms()[:2])
            ctx.close()
        results.append([torch.cat(lists[k]) for k in ("p", "m", "v")] + [gamma, norms, coefs])
    assert (results[0][0] != host["p"]).float().mean() > 0.999 and (results[0][5] < 1).any() and (results[0][5] == 1).any()
    for other in results[1:]:
        for k, (x, y) in enumerate(zip(results[0], other)):
            assert torch.equal(x, y), "array %d" % k


# Up to 288 work items (2048 elements; a long chunk has eight, in groups of eight chunks) without telemetry a step is a single launch, whose
# workgroups tell each other their sums; one item more, and steps that are profiled, have the norm kernel.
ONE_LAUNCH = {"every size": [1, 5, 511, 512, 513, 1024, 2047, 2048, 2049, 4096, 16384, 16385, 16384 + 300, 40000, 5],
              "a chunk to a lane": [32 * 16384 - 5], "a transformer": [131072] + [16384, 65536, 128] * 2 + [300, 40000],
              "waves": [500] * 600 + [3000] * 60, "at the limit": [2048] * 288, "one more": [2048] * 289}


@pytest.mark.parametrize("optimizer,grad_dtype,copy", [(B.ADAGC_OPT_ADAMW, B.ADAGC_GRAD_F32, False), (B.ADAGC_OPT_ADAMW, B.ADAGC_GRAD_BF16, True),
                                                       (B.ADAGC_OPT_LION, B.ADAGC_GRAD_F32, True), (B.ADAGC_OPT_LION, B.ADAGC_GRAD_BF16, False)])
@pytest.mark.parametrize("name", ONE_LAUNCH)
def test_a_single_launch_equals_the_norm_kernel_and_the_update(name, optimizer, grad_dtype, copy):
    """Three steps each: profiled (two launches), as they are, without any waiting (every wave computes all that it was not told before it
    looked), a captured step replayed, from odd addresses, and the entry point that builds its tables on the GPU."""
    numels, results = ONE_LAUNCH[name], []
    total, lion = sum(numels), optimizer == B.ADAGC_OPT_LION
    set_polls = B.lib().adagc_internal_set_polls
    set_polls.argtypes = [ctypes.c_void_p, ctypes.c_uint32]
    hp = B.make_hyper(lr=1e-3, t_start=0)
    for kind in ("profiled", "one", "no waiting", "captured", "odd", "static"):
        gen = torch.Generator(device=DEV).manual_seed(3)
        flat = {k: torch.randn(total, generator=gen, device=DEV) * x for k, x in (("p", 0.02), ("g", 0.01), ("m", 0.002), ("v", 0.01))}
        flat["v"].square_()
        flat["c"] = torch.zeros(total, dtype=torch.bfloat16, device=DEV)
        if grad_dtype == B.ADAGC_GRAD_BF16:
            flat["g"] = flat["g"].to(torch.bfloat16)
        lists = {k: [y.clone() for y in x.split(numels)] for k, x in flat.items()}
        held = lists["m"]
        if kind == "odd":                          # the momentum at an odd byte
            held = [torch.zeros(4 * n + 8, dtype=torch.uint8, device=DEV) for n in numels]
            for buf, x in zip(held, lists["m"]):
                buf[3:3 + 4 * x.numel()] = x.view(torch.uint8)
        m = [buf.data_ptr() + 3 for buf in held] if kind == "odd" else held
        v = None if lion else lists["v"]
        gamma = torch.tensor([(0.009, 0.012)[i % 2] * n ** 0.5 for i, n in enumerate(numels)], dtype=torch.float32, device=DEV)
        norms, coefs, clipped = (torch.zeros(len(numels), dtype=t, device=DEV) for t in (torch.float32, torch.float32, torch.uint8))
        reports = []
        ctx = None if kind == "static" else B.AdaGC(numels, optimizer, grad_dtype, copy)
        if ctx:
            assert set_polls(ctx._ctx, 0 if kind == "no waiting" else 200) == (name != "one more")
            if copy:
                ctx.set_param_copies(lists["c"])
            if kind == "profiled":
                ctx.profile_begin(3)
        for step in range(3):
            if kind == "static":
                B.adagc_step_static(numels, lists["p"], lists["g"], m, v, gamma, hp, 7, optimizer=optimizer, grad_dtype=grad_dtype,
                                    params_bf16=lists["c"] if copy else None, out_norms=norms, out_coefs=coefs, out_clipped=clipped)
                reports += [norms.cpu(), coefs.cpu(), clipped.cpu()]
            elif kind == "captured" and step:
                if step == 1:
                    graph = torch.cuda.CUDAGraph()
                    torch.cuda.synchronize()
                    with torch.cuda.graph(graph):
                        ctx.step(lists["p"], lists["g"], m, v, gamma, hp, 7, stream=torch.cuda.current_stream().cuda_stream)
                graph.replay()
                torch.cuda.synchronize()
            else:
                ctx.step(lists["p"], lists["g"], m, v, gamma, hp, 7)
            if ctx:
                reports += [torch.from_numpy(x.copy()) for x in ctx.get_norms()]
            reports.append(gamma.cpu())
        torch.cuda.synchronize()
        if ctx:
            ctx.close()
        if kind == "odd":
            assert all((buf[:3] == 0).all() and (buf[3 + 4 * n:] == 0).all() for buf, n in zip(held, numels))
            held = [buf[3:3 + 4 * n].clone().view(torch.float32) for buf, n in zip(held, numels)]
        results.append(reports + [torch.cat(lists["p"]), torch.cat(held), torch.cat(lists["v"]), torch.cat(lists["c"])])
        if kind == "odd":                          # its sums run element by element, in another order: no bits to compare
            for x, y in zip(results.pop(), results[0]):
                assert torch.allclose(x.double(), y.double(), rtol=1e-5 if x.dtype != torch.bfloat16 else 2 ** -7, atol=0)
            continue
        for k, (x, y) in enumerate(zip(results[-1], results[0])):
            assert torch.equal(x, y), "%s: array %d" % (kind, k)
    assert (results[0][1] < 1).any() and (len(numels) == 1 or (results[0][1] == 1).any())


def test_single_launches_that_overlap_leave_nothing_behind():
    """Steps of one context on two streams at once, which is not allowed and leaves any state, hold nobody up and leave nothing that a later
    step on its own could take for its own sums."""
    numels = ONE_LAUNCH["a transformer"]
    gen = torch.Generator(device=DEV).manual_seed(4)
    hp = B.make_hyper(lr=1e-3, t_start=0)
    ctx, other = B.AdaGC(numels), B.AdaGC(numels)
    def state():
        s = {k: [torch.randn(n, generator=gen, device=DEV) * x for n in numels] for k, x in (("p", 0.02), ("g", 0.01), ("m", 0.002))}
        s["v"] = [torch.rand(n, generator=gen, device=DEV) * 1e-4 for n in numels]
        s["gamma"] = torch.tensor([0.009 * n ** 0.5 for n in numels], dtype=torch.float32, device=DEV)
        return s
    a = state()
    streams = [torch.cuda.Stream() for _ in range(2)]
    ctx.step(a["p"], a["g"], a["m"], a["v"], a["gamma"], hp, 7)          # the pointer table is uploaded once, before the steps that overlap
    torch.cuda.synchronize()
    for k in range(40):
        ctx.step(a["p"], a["g"], a["m"], a["v"], a["gamma"], hp, 7, stream=streams[k % 2].cuda_stream)
    torch.cuda.synchronize()
    b = state()
    c = {k: [x.clone() for x in y] if k != "gamma" else y.clone() for k, y in b.items()}
    for step in range(7, 12):
        ctx.step(b["p"], b["g"], b["m"], b["v"], b["gamma"], hp, step)
        other.step(c["p"], c["g"], c["m"], c["v"], c["gamma"], hp, step)
    torch.cuda.synchronize()
    for k in b:
        for x, y in zip(b[k], c[k]):
            assert torch.equal(x, y)
    ctx.close()
    other.close()


# Lists with more than 450 MiB of gradients, stepped in groups of up to 256 MiB of them: groups that are full to the byte, a tensor larger than
# a group, chunks of every kind and single tensors at the ends of groups.
GROUP = 256 * MI // 4
GROUPED = {"full groups": (B.ADAGC_GRAD_F32, [GROUP // 2] * 4 + [1]), "a tensor larger than a group": (B.ADAGC_GRAD_F32, [5, GROUP + 70001, 300, 40 * MI, 2049, 12 * MI, 7]),
           "small tensors": (B.ADAGC_GRAD_F32, ITEMS + [16384 * 3 + 511] * 2500), "bf16": (B.ADAGC_GRAD_BF16, [1000, 2 * GROUP - 1001, 2, 2 * GROUP - 2, 4099])}


@pytest.mark.parametrize("optimizer,copy,flat", [(B.ADAGC_OPT_ADAMW, False, True), (B.ADAGC_OPT_LION, True, False)])
@pytest.mark.parametrize("name", GROUPED)
def test_a_list_in_groups_equals_the_list_as_a_whole(name, optimizer, copy, flat):
    """Two steps, the second captured and replayed, against steps that are profiled, which take the list as a whole; end to end in flat buffers
    (whole lines) or each tensor on its own.  A step of a warm-up, which is not grouped, in between."""
    grad_dtype, numels = GROUPED[name]
    assert sum(numels) * (2 if grad_dtype == B.ADAGC_GRAD_BF16 else 4) > 450 * MI
    lion, total, results = optimizer == B.ADAGC_OPT_LION, sum(numels), []
    hp = B.make_hyper(lr=1e-3, t_start=0)
    for whole in (True, False):
        gen = torch.Generator(device=DEV).manual_seed(6)
        buf = {k: torch.randn(total, generator=gen, device=DEV).mul_(x) for k, x in (("p", 0.02), ("g", 0.01), ("m", 0.002)) + (() if lion else (("v", 0.01),))}
        if not lion:
            buf["v"].square_()
        if grad_dtype == B.ADAGC_GRAD_BF16:
            buf["g"] = buf["g"].to(torch.bfloat16)
        buf["c"] = torch.zeros(total if copy else 1, dtype=torch.bfloat16, device=DEV)
        lists = {k: list(x.split(numels)) if x.numel() == total else [] for k, x in buf.items()}
        if not flat:
            lists = {k: [y.clone() for y in x] for k, x in lists.items()}
            del buf
        gamma = torch.tensor([(0.009, 0.012)[i % 2] * n ** 0.5 for i, n in enumerate(numels)], dtype=torch.float32, device=DEV)
        ctx = B.AdaGC(numels, optimizer, grad_dtype, copy)
        if copy:
            ctx.set_param_copies(lists["c"])
        if whole:
            ctx.profile_begin(3)
        v, reports = None if lion else lists["v"], []
        for step, h in ((7, hp), (8, B.make_hyper(lr=1e-3, t_start=100, lambda_abs=1.0)), (9, hp)):
            if whole or step != 9:
                ctx.step(lists["p"], lists["g"], lists["m"], v, gamma, h, step)
            else:
                graph = torch.cuda.CUDAGraph()
                torch.cuda.synchronize()
                with torch.cuda.graph(graph):
                    ctx.step(lists["p"], lists["g"], lists["m"], v, gamma, h, step, stream=torch.cuda.current_stream().cuda_stream)
                graph.replay()
                torch.cuda.synchronize()
            reports += [torch.from_numpy(x.copy()) for x in ctx.get_norms()] + [gamma.cpu()]
        ctx.close()
        results.append((reports, {k: lists[k] for k in ("p", "m", "c") + (() if lion else ("v",))}))
    assert (results[0][0][1] < 1).any() and (results[0][0][1] == 1).any()
    for k, (x, y) in enumerate(zip(results[0][0], results[1][0])):
        assert torch.equal(x, y), "report %d" % k
    for k in results[0][1]:
        for i, (x, y) in enumerate(zip(results[0][1][k], results[1][1][k])):
            assert torch.equal(x, y), "%s of tensor %d" % (k, i)


# sizes around the ends of vectors, lines, tiles (512, 1024, 2048, 4096 elements) and chunks (16384); the last brings the list above
# what walk_lines.h asks for (8 Mi elements for Lion, and the mean of 16384)
LINES = [1, 2, 3, 4, 5, 31, 32, 33, 34, 63, 511, 513, 1023, 1024, 1025, 1056, 2047, 2049, 4064, 4095, 4096, 4097, 4128, 8190, 16353, 16383,
         16384, 16385, 16416, 20480, 32767, 32769, 49153, 8200003]
LEADS = [0, 1, 2, 3, 7, 15, 29, 31, 32]        # elements in front of the first tensor; with 16 the last one would start on a line
STEP, STATIC, GRAPH = "step", "static", "graph"
LINE_RUNS = [(B.ADAGC_OPT_ADAMW, B.ADAGC_GRAD_F32, True, STEP, B.ADAGC_MODE_ADAGC, {}, LEADS),
             (B.ADAGC_OPT_ADAMW, B.ADAGC_GRAD_F32, False, STEP, B.ADAGC_MODE_ADAGC, {}, LEADS),
             (B.ADAGC_OPT_ADAMW, B.ADAGC_GRAD_BF16, True, STATIC, B.ADAGC_MODE_ADAGC, {}, LEADS),
             (B.ADAGC_OPT_LION, B.ADAGC_GRAD_BF16, True, STEP, B.ADAGC_MODE_ADAGC, {}, LEADS),
             (B.ADAGC_OPT_ADAMW, B.ADAGC_GRAD_BF16, False, STATIC, B.ADAGC_MODE_ADAGC, {}, [1, 31]),
             (B.ADAGC_OPT_ADAMW, B.ADAGC_GRAD_BF16, False, GRAPH, B.ADAGC_MODE_ADAGC, {}, [1, 31]),
             (B.ADAGC_OPT_ADAMW, B.ADAGC_GRAD_F32, False, GRAPH, B.ADAGC_MODE_ZCLIP, {}, [0, 29]),
             (B.ADAGC_OPT_LION, B.ADAGC_GRAD_BF16, True, GRAPH, B.ADAGC_MODE_GLOBALGC, {}, [3, 15]),
             (B.ADAGC_OPT_LION, B.ADAGC_GRAD_BF16, True, STATIC, B.ADAGC_MODE_GLOBAL_ADAGC, {}, [2, 7]),
             (B.ADAGC_OPT_ADAMW, B.ADAGC_GRAD_BF16, False, STEP, B.ADAGC_MODE_AGC, {}, [3, 31]),
             (B.ADAGC_OPT_ADAMW, B.ADAGC_GRAD_F32, True, STEP, B.ADAGC_MODE_CLIPPY, {}, [1, 15]),
             (B.ADAGC_OPT_LION, B.ADAGC_GRAD_BF16, True, STEP, B.ADAGC_MODE_CLIPPY, {}, [29]),
             (B.ADAGC_OPT_ADAMW, B.ADAGC_GRAD_F32, False, STEP, B.ADAGC_MODE_ADAGC, {"grid_blocks": 400}, [7]),
             (B.ADAGC_OPT_LION, B.ADAGC_GRAD_BF16, True, STEP, B.ADAGC_MODE_ADAGC, {"update_split": 1}, [2]),
             (B.ADAGC_OPT_ADAMW, B.ADAGC_GRAD_F32, True, STEP, B.ADAGC_MODE_ADAGC, {"unroll": 4}, [1, 31]),
             (B.ADAGC_OPT_ADAMW, B.ADAGC_GRAD_BF16, False, GRAPH, B.ADAGC_MODE_ZCLIP, {"unroll": 4}, [7])]


class _Lines:
    """The list LINES in flat buffers, `lead` elements in: values from the seed, on the host."""

    def __init__(self, lead, grad_dtype):
        gen = torch.Generator().manual_seed(lead + 100)
        total = lead + sum(LINES) + 40
        randn = lambda scale: torch.randn(total, generator=gen) * scale
        self.lead, self.starts = lead, [lead]
        for n in LINES:
            self.starts.append(self.starts[-1] + n)
        self.host = {"p": randn(0.02), "g": randn(0.01).to(torch.bfloat16 if grad_dtype == B.ADAGC_GRAD_BF16 else torch.float32),
                     "m": randn(0.002), "v": torch.rand(total, generator=gen) * 1e-4 + 1e-6, "c": torch.full((total,), 7.0, dtype=torch.bfloat16)}

    def buffers(self, offset_m=0):
        """The flat buffers, and the list's views of them; m lies `offset_m` elements further on than the others."""
        whole = {k: (torch.cat([torch.zeros(offset_m), x]) if k == "m" else x).to(DEV) for k, x in self.host.items()}
        return whole, {k: [x[a:b] for a, b in zip(self.starts, self.starts[1:])] for k, x in
                       ((k, x[offset_m:] if k == "m" else x) for k, x in whole.items())}

    def check_gaps(self, whole, offset_m=0):
        for k, x in whole.items():
            at = offset_m if k == "m" else 0
            got = torch.cat([x[at:at + self.lead], x[at + self.starts[-1]:]]).cpu()
            want = torch.cat([self.host[k][:self.lead], self.host[k][self.starts[-1]:]])
            assert torch.equal(got, want) and (x[:at] == 0).all(), "elements outside the tensors (%s)" % k


def _step_in_lines(lists, optimizer, grad_dtype, copy, entry, mode, kw, warmup=False):
    gamma = torch.tensor([0.009 * n ** 0.5 for n in LINES], dtype=torch.float32, device=DEV)
    hp = B.make_hyper(lr=1e-3, t_start=100 if warmup else 0, clip_mode=mode, lambda_abs=1e-5 if mode == B.ADAGC_MODE_CLIPPY else float("inf"),
                      lambda_rel={B.ADAGC_MODE_AGC: 1e-3, B.ADAGC_MODE_CLIPPY: 1e-2}.get(mode, 1.04))
    v = None if optimizer == B.ADAGC_OPT_LION else lists["v"]
    if entry == STATIC:
        B.adagc_step_static(LINES, lists["p"], lists["g"], lists["m"], v, gamma, hp, 7, optimizer=optimizer, grad_dtype=grad_dtype,
                            params_bf16=lists["c"] if copy else None)
    else:
        ctx = B.AdaGC(LINES, optimizer, grad_dtype, copy, update_clipping=mode in (B.ADAGC_MODE_AGC, B.ADAGC_MODE_CLIPPY), **kw)
        if copy:
            ctx.set_param_copies(lists["c"])
        if entry == GRAPH:
            sp = torch.frombuffer(bytearray(B.step_params_bytes(hp, 7)), dtype=torch.uint8).to(DEV)
            ctx.step_graph(lists["p"], lists["g"], lists["m"], v, gamma, sp)
        else:
            ctx.step(lists["p"], lists["g"], lists["m"], v, gamma, hp, 7)
        torch.cuda.synchronize()
        ctx.close()
    torch.cuda.synchronize()
    return gamma


def _same_state(got, ref, lion):
    for k in ("p", "m", "c") + (() if lion else ("v",)):
        for i, n in enumerate(LINES):
            assert torch.equal(got[k][i], ref[k][i]), "%s of tensor %d (%d elements)" % (k, i, n)


@pytest.mark.parametrize("optimizer,grad_dtype,copy,entry,mode,kw,lead", [run[:6] + (lead,) for run in LINE_RUNS for lead in run[6]])
def test_tensors_that_start_anywhere_in_a_line(optimizer, grad_dtype, copy, entry, mode, kw, lead):
    """Where the arrays agree on their place in a 128-byte line, tiles start on lines (tests/test_walk_lines.py holds these lists against
    the rule): every element must be updated once, to the bits it gets in an allocation of its own, and the gaps in front of, between
    and behind the tensors must stay.  `lead` elements lie in front of the first tensor; once more with the moments elsewhere in a line
    than the parameters."""
    data, lion = _Lines(lead, grad_dtype), optimizer == B.ADAGC_OPT_LION
    ref = {k: [x.clone() for x in views] for k, views in data.buffers()[1].items()}
    before = [x.clone() for x in ref["p"]]
    gamma_ref = _step_in_lines(ref, optimizer, grad_dtype, copy, entry, mode, kw)
    assert all((x != y).any() for x, y in zip(ref["p"], before))
    for offset_m in (0, 3):
        whole, got = data.buffers(offset_m)
        gamma = _step_in_lines(got, optimizer, grad_dtype, copy, entry, mode, kw)
        _same_state(got, ref, lion)
        assert torch.equal(gamma, gamma_ref)
        data.check_gaps(whole, offset_m)


@pytest.mark.parametrize("optimizer,grad_dtype,copy", [(B.ADAGC_OPT_ADAMW, B.ADAGC_GRAD_F32, False), (B.ADAGC_OPT_ADAMW, B.ADAGC_GRAD_BF16, True),
                                                       (B.ADAGC_OPT_LION, B.ADAGC_GRAD_BF16, True)])
@pytest.mark.parametrize("entry", [STEP, STATIC, GRAPH])
def test_whole_lines_with_other_tensors_among_them(entry, optimizer, grad_dtype, copy):
    """A list that is walked in whole lines for the sake of most of its elements: some tensors' moments lie elsewhere in a line, some
    are in allocations of their own, and some have a momentum that is not even aligned to its elements and go element by element.  Inside
    the warm-up without a limit, so that the coefficient is 1 whatever the order of the norms' sums."""
    data, lion = _Lines(5, grad_dtype), optimizer == B.ADAGC_OPT_LION
    ref = {k: [x.clone() for x in views] for k, views in data.buffers()[1].items()}
    _step_in_lines(ref, optimizer, grad_dtype, copy, entry, B.ADAGC_MODE_ADAGC, {}, warmup=True)
    whole, got = data.buffers()
    shifted, elsewhere = data.buffers(3)
    packed = {}
    for i, n in enumerate(LINES[:-1]):
        if i % 4 == 1:
            got["m"][i] = elsewhere["m"][i]
        elif i % 4 == 2:
            for k in got:
                got[k][i] = got[k][i].clone()
        elif i % 4 == 3:
            packed[i] = torch.full((4 * n + 64,), 0xA5, dtype=torch.uint8, device=DEV)
            packed[i][33:33 + 4 * n] = got["m"][i].view(torch.uint8)
    lists = dict(got, m=[packed[i].data_ptr() + 33 if i in packed else x for i, x in enumerate(got["m"])])
    _step_in_lines(lists, optimizer, grad_dtype, copy, entry, B.ADAGC_MODE_ADAGC, {}, warmup=True)
    for i, buf in packed.items():
        n = 4 * LINES[i]
        assert (buf[:33] == 0xA5).all() and (buf[33 + n:] == 0xA5).all()
        got["m"][i] = buf[33:33 + n].clone().view(torch.float32)
    _same_state(got, ref, lion)
    data.check_gaps(whole)
    data.check_gaps(shifted, 3)
    for i in range(len(LINES) - 1):                       # momenta that lie elsewhere: what is at their usual place stays
        if i % 4 != 0:
            a, b = data.starts[i], data.starts[i + 1]
            assert torch.equal(whole["m"][a:b].cpu(), data.host["m"][a:b])


def test_a_context_whose_tensors_move_on_and_off_the_lines():
    """What a step derives from the tensors' places is kept until they move: steps on tensors laid end to end, twice in allocations of
    their own and end to end again, against a context for each of them."""
    data = _Lines(7, B.ADAGC_GRAD_F32)
    hp = B.make_hyper(lr=1e-3, t_start=0)
    results = []
    for separate_contexts in (False, True):
        _, flat = data.buffers()
        apart = {k: [x.clone() for x in views] for k, views in flat.items()}
        gamma = torch.tensor([0.009 * n ** 0.5 for n in LINES], dtype=torch.float32, device=DEV)
        ctxs = [B.AdaGC(LINES) for _ in range(2 if separate_contexts else 1)]
        for step, (lists, c) in enumerate(((flat, 0), (apart, 1), (apart, 1), (flat, 0)), start=7):
            ctxs[c % len(ctxs)].step(lists["p"], lists["g"], lists["m"], lists["v"], gamma, hp, step)
        torch.cuda.synchronize()
        for c in ctxs:
            c.close()
        results.append([torch.cat(x[k]) for x in (flat, apart) for k in "pmv"] + [gamma])
    for x, y in zip(*results):
        assert torch.equal(x, y)


def _state_next_to_a_tie(beta, t, exact):
    """An fp32 state x > 0 for which beta x + t and beta x + exact, each rounded to double and then to fp32, differ, `exact` (a Fraction)
    being the product that t rounds to double: which of the two a kernel computes is decided by the product that it fuses.  Searched among the
    x whose sum with t lies within a unit of its exact arithmetic of a tie between two fp32 values.  0 if there is none."""
    b, eb = int(beta * 2 ** 30), -30                                                # beta is an fp32 value
    while b % 2 == 0:
        b, eb = b // 2, eb + 1
    for e in range(int(np.floor(np.log2(t))) - 27, int(np.floor(np.log2(t))) - 18): # of x's unit: x is between t / 16 and 16 t
        units = int(round(t / 2.0 ** (eb + e)))
        for bits in range(b.bit_length() + 23, b.bit_length() + 29):                # of the sum, in units of 2^(eb + e)
            q = bits - 24                                                           # of its fp32 unit
            x = pow(b, -1, 2 ** q) * (2 ** (q - 1) - units) % 2 ** q
            x += -(-max(2 ** 23 - x, 0) // 2 ** q) * 2 ** q
            if x < 2 ** 24 and (b * x + units).bit_length() == bits:
                x = x * 2.0 ** e
                if np.float32(beta * x + t) != np.float32(float(Fraction(beta * x) + exact)):
                    return x
    return 0.0


TIES = [1, 5, 37, 1000, 1030] + [4099, 8191, 12289, 16385, 20001, 33001] * 5


@functools.lru_cache(maxsize=None)
def _ties(beta_m, beta_v):
    """Gradients (integers, so that the norms' sums of squares are exact), m and v next to ties where the coefficient of a clipped tensor
    with gamma 1 allows any, and m' and v' by the formulas in double without fusing."""
    rng = np.random.default_rng(12)
    b_m, b_v = float(np.float32(beta_m)), float(np.float32(beta_v))
    out, telling = [], [0, 0]
    for n in TIES:
        x = (2.0 * rng.integers(0, 128, n) + 1.0) * rng.choice([-1.0, 1.0], n)
        x[0] = 77.0
        h = float(np.float32(1.04)) / np.sqrt(np.sum(x * x))
        assert h < 1.0
        m, v = rng.random(n).astype(np.float32).astype(np.float64), rng.random(n).astype(np.float32).astype(np.float64)
        for a in np.unique(np.abs(x)):
            gh, at = h * a, np.abs(x) == a
            for q, (s, b, t, exact) in enumerate(((m, b_m, (1.0 - b_m) * gh, Fraction(1.0 - b_m) * Fraction(gh)),
                                                  (v, b_v, (1.0 - b_v) * gh * gh, Fraction((1.0 - b_v) * gh) * Fraction(gh)))):
                y = _state_next_to_a_tie(b, t, exact)
                if y:
                    s[at] = y
                    telling[q] += int(at.sum())
        m *= np.sign(x)
        gh = h * x
        out.append([y.astype(np.float32) for y in (x, m, v, b_m * m + (1.0 - b_m) * gh, b_v * v + (1.0 - b_v) * gh * gh)])
    return out, telling


@pytest.mark.parametrize("optimizer,grad_dtype,copy", [(o, g, c) for o in (B.ADAGC_OPT_ADAMW, B.ADAGC_OPT_LION)
                                                       for g in (B.ADAGC_GRAD_F32, B.ADAGC_GRAD_BF16) for c in (False, True)])
def test_moments_next_to_ties_have_the_bits_of_separately_rounded_sums(optimizer, grad_dtype, copy):
    """beta m + (1 - beta) h g and beta v + (1 - beta) (h g)^2 are sums of two products: which of them is fused decides the last bit of a
    value next to a tie.  It must not depend on the kernel or the place: short and long tensors, apart from each other and end to end
    (in whole lines, for the sake of a large tensor of zeros), against the formulas without fusing."""
    lion = optimizer == B.ADAGC_OPT_LION
    beta1, beta2 = (0.9, 0.99) if lion else (0.9, 0.95)
    data, telling = _ties(beta2 if lion else beta1, beta2)
    assert min(telling) >= 300, telling
    hp = B.make_hyper(lr=1e-3, beta1=beta1, beta2=beta2, t_start=0)
    for flat in (False, True):
        sizes = TIES + [8400001] if flat else TIES
        pad = 1 if flat else 128
        starts = [3 if flat else 0]
        for n in sizes:
            starts.append(starts[-1] + -(-n // pad) * pad)
        host = {k: np.zeros(starts[-1], dtype=np.float32) for k in "pgmv"}
        for a, n, rows in zip(starts, TIES, data):
            for k, x in zip("gmv", rows):
                host[k][a:a + n] = x
        buf = {k: torch.from_numpy(x).to(DEV) for k, x in host.items()}
        if grad_dtype == B.ADAGC_GRAD_BF16:
            buf["g"] = buf["g"].to(torch.bfloat16)
        buf["c"] = torch.zeros(starts[-1], dtype=torch.bfloat16, device=DEV)
        lists = {k: [x[a:a + n] for a, n in zip(starts, sizes)] for k, x in buf.items()}
        ctx = B.AdaGC(sizes, optimizer, grad_dtype, copy)
        if copy:
            ctx.set_param_copies(lists["c"])
        gamma = torch.ones(len(sizes), dtype=torch.float32, device=DEV)
        ctx.step(lists["p"], lists["g"], lists["m"], None if lion else lists["v"], gamma, hp, 7)
        torch.cuda.synchronize()
        ctx.close()
        for i, n in enumerate(TIES):
            for k, ref in zip("m" if lion else "mv", data[i][3:]):
                wrong = (lists[k][i].cpu().numpy() != ref).nonzero()[0]
                assert not len(wrong), "%s of tensor %d (%d elements), %s: %d values, first at %s" % (
                    k, i, n, "end to end" if flat else "apart", len(wrong), wrong[:5])


@pytest.mark.parametrize("entry", [STEP, GRAPH, STATIC])
@pytest.mark.parametrize("filler", [0, 6000001])
def test_gamma_next_to_ties_has_the_bits_of_separately_rounded_operations(filler, entry):
    """beta gamma + (1 - beta) norm next to ties, on a list whose rule is evaluated in the update kernel and on one with a rules kernel: the
    formula in double, without fusing.  (1 - beta) norm is rounded; integers as gradients, so that the norms are known."""
    rng = np.random.default_rng(5)
    beta = float(np.float32(0.9))
    grads, gammas = [], []
    while len(grads) < 40:
        x = (2.0 * rng.integers(0, 128, rng.integers(2, 60)) + 1.0) * rng.choice([-1.0, 1.0])
        norm = float(np.sqrt(np.sum(x * x)))
        gamma = _state_next_to_a_tie(beta, (1.0 - beta) * norm, Fraction(1.0 - beta) * Fraction(norm))
        if gamma:
            grads.append(x)
            gammas.append(gamma)
    want = [np.float32(beta * y + (1.0 - beta) * float(np.sqrt(np.sum(x * x)))) for x, y in zip(grads, gammas)]
    hp = B.make_hyper(lr=1e-3, ema_beta=0.9, lambda_rel=1e6, t_start=0)                 # nothing clipped
    g = [torch.from_numpy(x.astype(np.float32)).to(DEV) for x in grads] + ([torch.zeros(filler, device=DEV)] if filler else [])
    p, m, v = ([torch.zeros_like(x) for x in g] for _ in range(3))
    ema = torch.tensor(gammas + [1.0] * bool(filler), dtype=torch.float32, device=DEV)
    assert ema[:40].double().cpu().tolist() == gammas                                  # fp32 values
    numels = [x.numel() for x in g]
    if entry == STATIC:
        B.adagc_step_static(numels, p, g, m, v, ema, hp, 7)
    else:
        ctx = B.AdaGC(numels)
        if entry == GRAPH:
            ctx.step_graph(p, g, m, v, ema, torch.frombuffer(bytearray(B.step_params_bytes(hp, 7)), dtype=torch.uint8).to(DEV))
        else:
            ctx.step(p, g, m, v, ema, hp, 7)
        torch.cuda.synchronize()
        ctx.close()
    torch.cuda.synchronize()
    assert np.array_equal(ema[:40].cpu().numpy(), np.array(want))
