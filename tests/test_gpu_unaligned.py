"""Arrays that are not even aligned to their elements (records packed byte by byte, memory-mapped files): accepted by every entry
point and handled element by element.  The step must be the one on aligned arrays, up to the order in which the norms are summed:
that moves a coefficient by some 1e-13, and so a stored fp32 value by at most its last bit (2^-23).  Bytes beside the arrays must
stay as they are."""
import ctypes

import pytest
import torch

from paper_2502_11034_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
ULP = 2.0 ** -23

# tiny, short and long chunks: one below, at and above a wave, a round of a workgroup, the work items and a chunk
SIZES = [1, 2, 3, 5, 63, 64, 65, 255, 256, 257, 511, 512, 513, 1000, 1024, 1025, 2047, 2048, 2049, 4096, 4097, 8193, 16383, 16384, 16385,
         40000, 49157]
PAD = 64                        # bytes before and after every array


class Packed:
    """A tensor's values in a byte buffer, `offset` bytes past an aligned address."""

    def __init__(self, x, offset):
        self.dtype, self.n = x.dtype, x.numel() * x.element_size()
        self.at = PAD + offset
        self.buf = torch.full((self.n + 2 * PAD + 8,), 0xA5, dtype=torch.uint8, device=DEV)
        self.buf[self.at:self.at + self.n] = x.contiguous().view(torch.uint8)

    def data_ptr(self):
        return self.buf.data_ptr() + self.at

    def values(self):
        assert (self.buf[:self.at] == 0xA5).all() and (self.buf[self.at + self.n:] == 0xA5).all(), "bytes beside the array"
        return self.buf[self.at:self.at + self.n].clone().view(self.dtype)


def _lists(numels, grad_dtype, offsets, seed):
    """p, g, m, v, copies: from the seed alone, each array `offsets[name]` bytes off."""
    gen = torch.Generator(device="cpu").manual_seed(seed)
    rand = lambda n, scale: torch.randn(n, generator=gen) * scale
    out = {k: [] for k in "pgmvc"}
    for n in numels:
        p, g, m = rand(n, 0.02), rand(n, 0.01), rand(n, 0.002)
        v = m.square() + 1e-6
        g = g.to(torch.bfloat16) if grad_dtype == B.ADAGC_GRAD_BF16 else g
        for k, x in zip("pgmvc", (p, g, m, v, torch.zeros(n, dtype=torch.bfloat16))):
            out[k].append(Packed(x.to(DEV), offsets.get(k, 0)))
    return out


def _gamma(numels):
    return torch.tensor([(0.005 if i % 2 else 0.02) * n ** 0.5 for i, n in enumerate(numels)], dtype=torch.float32, device=DEV)


def _run(entry, optimizer, grad_dtype, mode, offsets):
    lists = _lists(SIZES, grad_dtype, offsets, 11)
    n = len(SIZES)
    lion = optimizer == B.ADAGC_OPT_LION
    clipping = mode in (B.ADAGC_MODE_AGC, B.ADAGC_MODE_CLIPPY)
    hp = B.make_hyper(lr=1e-3, t_start=0, clip_mode=mode,
                      lambda_rel={B.ADAGC_MODE_AGC: 1e-3, B.ADAGC_MODE_CLIPPY: 1e-2}.get(mode, 1.04),
                      lambda_abs=1e-5 if mode == B.ADAGC_MODE_CLIPPY else 1.0)
    gamma = _gamma(SIZES)
    p, g, m, c = (lists[k] for k in "pgmc")
    v = None if lion else lists["v"]
    if entry == "static":
        outs = (torch.zeros(n, device=DEV), torch.zeros(n, device=DEV), torch.zeros(n, dtype=torch.uint8, device=DEV))
        for step in (7, 8):
            B.adagc_step_static(SIZES, p, g, m, v, gamma, hp, step, optimizer=optimizer, grad_dtype=grad_dtype, params_bf16=c,
                                out_norms=outs[0], out_coefs=outs[1], out_clipped=outs[2])
        seen = [x.cpu() for x in outs]
    else:
        ctx = B.AdaGC(SIZES, optimizer, grad_dtype, True, telemetry=True, update_clipping=clipping)
        ctx.set_param_copies(c)
        sp = torch.zeros(ctypes.sizeof(B.adagc_step_params), dtype=torch.uint8, device=DEV)
        for step in (7, 8):
            if entry == "graph":
                sp.copy_(torch.frombuffer(bytearray(B.step_params_bytes(hp, step)), dtype=torch.uint8))
                ctx.step_graph(p, g, m, v, gamma, sp)
            else:
                ctx.step(p, g, m, v, gamma, hp, step)
        seen = [torch.from_numpy(x) for x in ctx.get_norms() + ctx.get_state_norms()]
        ctx.close()
    torch.cuda.synchronize()
    state = {k: torch.cat([x.values() for x in lists[k]]) for k in "pgmvc"}
    return state, gamma, seen


def _compare(a, b):
    (sa, ga, xa), (sb, gb, xb) = a, b
    assert torch.equal(sa["g"], sb["g"])
    for k in "pmv":
        assert ((sa[k] - sb[k]).abs() <= ULP * sb[k].abs()).all(), k
    assert torch.equal(sa["c"], sa["p"].to(torch.bfloat16))               # round to nearest even of what is stored
    assert ((ga - gb).abs() <= ULP * gb.abs()).all()
    assert torch.equal(xa[2], xb[2]) and xa[2].any()                      # the decisions
    for k, (x, y) in enumerate(zip(xa, xb)):
        # norms of values that differ by their last bits, and their own rounding; the norm of theta's change (the last of the
        # state's norms) takes the last bits of theta
        theta = torch.stack([t.norm() for t in sb["p"].cpu().split(SIZES)]) if k == 5 else 0.0
        assert ((x - y).abs() <= 2 * ULP * y.abs() + ULP * theta).all(), k


ALL = dict(p=2, g=2, m=1, v=3, c=1)          # bytes past an aligned address


@pytest.mark.parametrize("entry", ["step", "graph", "static"])
@pytest.mark.parametrize("grad_dtype", [B.ADAGC_GRAD_F32, B.ADAGC_GRAD_BF16])
@pytest.mark.parametrize("optimizer", [B.ADAGC_OPT_ADAMW, B.ADAGC_OPT_LION])
def test_arrays_at_any_byte(optimizer, grad_dtype, entry):
    offsets = dict(ALL, g=1) if grad_dtype == B.ADAGC_GRAD_BF16 else ALL
    _compare(_run(entry, optimizer, grad_dtype, B.ADAGC_MODE_ADAGC, offsets),
             _run(entry, optimizer, grad_dtype, B.ADAGC_MODE_ADAGC, {}))


@pytest.mark.parametrize("mode", [B.ADAGC_MODE_AGC, B.ADAGC_MODE_CLIPPY])
@pytest.mark.parametrize("optimizer", [B.ADAGC_OPT_ADAMW, B.ADAGC_OPT_LION])
def test_arrays_at_any_byte_with_update_clipping(optimizer, mode):
    _compare(_run("step", optimizer, B.ADAGC_GRAD_F32, mode, ALL), _run("step", optimizer, B.ADAGC_GRAD_F32, mode, {}))


@pytest.mark.parametrize("entry", ["step", "static"])
@pytest.mark.parametrize("which", list("pgmvc"))
def test_one_array_off_is_enough(which, entry):
    off = {which: 1 if which == "c" else 2}
    _compare(_run(entry, B.ADAGC_OPT_ADAMW, B.ADAGC_GRAD_F32, B.ADAGC_MODE_ADAGC, off),
             _run(entry, B.ADAGC_OPT_ADAMW, B.ADAGC_GRAD_F32, B.ADAGC_MODE_ADAGC, {}))


@pytest.mark.parametrize("grad_dtype", [B.ADAGC_GRAD_F32, B.ADAGC_GRAD_BF16])
def test_muon_arrays_at_any_byte(grad_dtype):
    """Columns that are a multiple of 4 (vectors, where the arrays allow them) and others, wide and tall matrices."""
    shapes = [(96, 128), (128, 64), (33, 50), (7, 7), (200, 300), (4, 5000), (257, 129)]
    numels = [r * c for r, c in shapes]
    results = []
    for offsets in (dict(p=2, g=1, m=3, c=1), {}):
        lists = _lists(numels, grad_dtype, offsets, 12)
        gamma = _gamma(numels)
        ctx = B.AdaGC(numels, B.ADAGC_OPT_MUON, grad_dtype, True)
        ctx.muon_attach(shapes)
        ctx.set_param_copies(lists["c"])
        for step in (7, 8):
            ctx.muon_step(lists["p"], lists["g"], lists["m"], gamma, B.make_hyper(lr=1e-3, t_start=0), B.make_muon_hyper(), step)
        seen = [torch.from_numpy(x) for x in ctx.get_norms()]
        ctx.close()
        torch.cuda.synchronize()
        results.append(({k: torch.cat([x.values() for x in lists[k]]) for k in "pgmvc"}, gamma, seen))
    _compare(*results)
