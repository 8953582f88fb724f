"""GPU parity of the SSD chunk functions (ssd_chunk_state, ssd_state_passing,
ssd_bmm_chunk, ssd_chunk_scan) through the C ABI against the float64 oracle
(oracle/ssd.py), on the same seeded inputs.

Tolerances, from the arithmetic of the kernels:
  * chunk state / chunk scan: each product has one operand rounded to bf16
    (the weighted x, the weighted cb entry, the entering state), a relative
    error of at most 2^-8 per term; the decays come from an fp32 prefix sum
    and exp2 (relative error ~1e-4 on the terms that matter) and the sums are
    fp32.  So |out - ref| <= 2^-7 * (the same sums over |terms|), which the
    oracle computes (``chunk_state_abs`` / ``chunk_scan_abs``).  A single
    round-to-nearest-even has a relative error of root mean square ~1.5e-3
    (uniform over half an ulp); a sum of several rounded terms averages it
    down, and the decay often leaves one or two terms dominant, so the root
    mean square of err / |terms| over all outputs must stay below 2^-9
    (1.95e-3); a wrong decay index or a lost dt shifts it by far more.
  * chunk matrix: exact bf16 products, fp32 sums of 128 terms:
    1e-5 * sum_n |Cm_l[n]| |Bm_s[n]|.
  * state passing: fp32 multiply-adds over the chunks, 1e-5 of the same
    recurrence over |states|.
  * the four chained: each stage's bound carried through, 2^-6 of the chained
    |terms| sums.
"""
import numpy as np
import pytest

import oracle.ssd as ossd
from paper_2504_17577_amd import gen

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

Q = 256
BOUND = 2.0 ** -7
RMS = 2.0 ** -9


@pytest.fixture(scope="module")
def ta():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2504_17577_amd import tileattn
    tileattn.lib()
    return tileattn


def dev_bf16(x):
    return torch.from_numpy(np.ascontiguousarray(x).view(np.int16)).view(torch.bfloat16).cuda()


def dev_f32(x):
    return torch.from_numpy(np.ascontiguousarray(x, dtype=np.float32)).cuda()


def check(tag, got, ref, scale, bound=BOUND, rms=RMS):
    got = np.asarray(got, dtype=np.float64)
    assert np.isfinite(got).all(), f"{tag}: non-finite output"
    r = np.abs(got - ref) / np.maximum(scale, 1e-30)
    worst, mean_sq = float(r.max()), float(np.sqrt(np.mean(r ** 2)))
    print(f"{tag}: max|d|={np.abs(got - ref).max():.3e} worst err/scale={worst:.3e} "
          f"rms={mean_sq:.3e}", flush=True)
    assert worst <= bound, f"{tag}: worst err/scale {worst} > {bound}"
    if rms is not None:
        assert mean_sq <= rms, f"{tag}: rms err/scale {mean_sq} > {rms}"


SHAPES = [  # (B, L, H, G)
    (2, 300, 4, 2),      # ragged last chunk, two groups
    (1, 1, 2, 1),        # a single position
    (1, 37, 2, 2),       # one short chunk, one head per group
    (1, 512, 4, 1),      # exact multiple of the chunk
    (2, 1000, 8, 2),     # four chunks, ragged
]


def problem(shape, seed):
    B, L, H, G = shape
    w, inp = gen.random_ssd_problem(B, L, H, G, seed=seed)
    return w, inp


@pytest.mark.parametrize("shape", SHAPES, ids=[str(s) for s in SHAPES])
def test_chunk_state(ta, shape):
    print(f"ssd_chunk_state {shape}", flush=True)
    w, inp = problem(shape, seed=sum(shape))
    out = torch.full((w.B, w.nc, w.H, w.P, w.N), float("nan"), device="cuda")
    ta.ssd_chunk_state(dev_bf16(inp["x"]), dev_bf16(inp["Bm"]), dev_f32(inp["dt"]),
                       dev_f32(inp["A"]), out=out)
    torch.cuda.synchronize()
    ref = ossd.chunk_state(inp["x"], inp["Bm"], inp["dt"], inp["A"], Q)
    scale = ossd.chunk_state_abs(inp["x"], inp["Bm"], inp["dt"], inp["A"], Q)
    check(f"chunk_state {shape}", out.cpu().numpy(), ref, scale)


@pytest.mark.parametrize("shape", SHAPES, ids=[str(s) for s in SHAPES])
def test_chunk_scan(ta, shape):
    print(f"ssd_chunk_scan {shape}", flush=True)
    w, inp = problem(shape, seed=7 + sum(shape))
    cb, prev = gen.make_ssd_scan_extras(w, seed=3)
    out = torch.full((w.B, w.L, w.H, w.P), float("nan"), device="cuda")
    ta.ssd_chunk_scan(dev_bf16(inp["x"]), dev_bf16(inp["Cm"]), dev_f32(cb), dev_f32(inp["dt"]),
                      dev_f32(inp["A"]), dev_f32(prev), dev_f32(inp["D"]), out=out)
    torch.cuda.synchronize()
    args = (inp["x"], inp["Cm"], cb, inp["dt"], inp["A"], prev, inp["D"], Q)
    check(f"chunk_scan {shape}", out.cpu().numpy(), ossd.chunk_scan(*args), ossd.chunk_scan_abs(*args))


def test_chunk_scan_without_skip_term(ta):
    w, inp = problem((1, 300, 2, 1), seed=21)
    cb, prev = gen.make_ssd_scan_extras(w, seed=4)
    y = ta.ssd_chunk_scan(dev_bf16(inp["x"]), dev_bf16(inp["Cm"]), dev_f32(cb), dev_f32(inp["dt"]),
                          dev_f32(inp["A"]), dev_f32(prev), None)
    torch.cuda.synchronize()
    zero = np.zeros_like(inp["D"])
    args = (inp["x"], inp["Cm"], cb, inp["dt"], inp["A"], prev, zero, Q)
    check("chunk_scan D=None", y.cpu().numpy(), ossd.chunk_scan(*args), ossd.chunk_scan_abs(*args))


@pytest.mark.parametrize("shape", SHAPES, ids=[str(s) for s in SHAPES])
def test_bmm_chunk(ta, shape):
    print(f"ssd_bmm_chunk {shape}", flush=True)
    w, inp = problem(shape, seed=11 + sum(shape))
    out = torch.full((w.B, w.nc, w.G, Q, Q), float("nan"), device="cuda")
    ta.ssd_bmm_chunk(dev_bf16(inp["Cm"]), dev_bf16(inp["Bm"]), out=out)
    torch.cuda.synchronize()
    ref = ossd.bmm_chunk(inp["Cm"], inp["Bm"], Q)
    ab = lambda u: np.ascontiguousarray(u) & np.uint16(0x7FFF)
    scale = ossd.bmm_chunk(ab(inp["Cm"]), ab(inp["Bm"]), Q)
    got = out.cpu().numpy()
    # rows and columns of padded positions (past L) are written as exact zeros
    pos = np.arange(w.nc * Q).reshape(w.nc, Q) >= w.L
    pad = pos[None, :, None, :, None] | pos[None, :, None, None, :]
    pad = np.broadcast_to(pad, got.shape)
    assert (got[pad] == 0).all(), "padded rows/columns of cb must be zero"
    check(f"bmm_chunk {shape}", got, ref, np.maximum(scale, 1e-30), bound=1e-5, rms=None)


@pytest.mark.parametrize("shape", SHAPES, ids=[str(s) for s in SHAPES])
def test_state_passing(ta, shape):
    print(f"ssd_state_passing {shape}", flush=True)
    w, inp = problem(shape, seed=13 + sum(shape))
    _, states = gen.make_ssd_scan_extras(w, seed=5)
    prev, final = ta.ssd_state_passing(dev_f32(states), dev_f32(inp["dt"]), dev_f32(inp["A"]))
    torch.cuda.synchronize()
    rp, rf = ossd.state_passing(states, inp["dt"], inp["A"], Q)
    sp, sf = ossd.state_passing(np.abs(states), inp["dt"], inp["A"], Q)
    check(f"state_passing prev {shape}", prev.cpu().numpy(), rp, np.maximum(sp, 1e-30), bound=1e-5,
          rms=None)
    check(f"state_passing final {shape}", final.cpu().numpy(), rf, sf, bound=1e-5, rms=None)


def chained(ta, dx, ddt, dA, dB, dC, dD=None):
    prev, final = ta.ssd_state_passing(ta.ssd_chunk_state(dx, dB, ddt, dA), ddt, dA)
    return ta.ssd_chunk_scan(dx, dC, ta.ssd_bmm_chunk(dC, dB), ddt, dA, prev, dD), final


def chained_scale(inp):
    """The chained sums with every term replaced by its magnitude."""
    ab = lambda u: np.ascontiguousarray(u) & np.uint16(0x7FFF)
    s_abs = ossd.chunk_state_abs(inp["x"], inp["Bm"], inp["dt"], inp["A"], Q)
    p_abs, _ = ossd.state_passing(s_abs, inp["dt"], inp["A"], Q)
    cb_abs = ossd.bmm_chunk(ab(inp["Cm"]), ab(inp["Bm"]), Q)
    return ossd.chunk_scan_abs(inp["x"], inp["Cm"], cb_abs, inp["dt"], inp["A"], p_abs, inp["D"], Q)


@pytest.mark.parametrize("shape", [(2, 300, 4, 2), (2, 1000, 8, 2), (1, 2048, 4, 1)],
                         ids=["s300", "s1000", "s2048"])
def test_chained_forward_matches_oracle(ta, shape):
    """ssd_forward, and the four kernels chained on the GPU, reproduce the
    oracle's chained result (pinned to the step-by-step recurrence)."""
    print(f"ssd chained {shape}", flush=True)
    w, inp = problem(shape, seed=17 + sum(shape))
    args = (dev_bf16(inp["x"]), dev_f32(inp["dt"]), dev_f32(inp["A"]),
            dev_bf16(inp["Bm"]), dev_bf16(inp["Cm"]), dev_f32(inp["D"]))
    y, final = ta.ssd_forward(*args)
    cy, cfinal = chained(ta, *args)
    torch.cuda.synchronize()
    ry, rf = ossd.ssd_forward(inp["x"], inp["dt"], inp["A"], inp["Bm"], inp["Cm"], inp["D"], Q)
    scale = chained_scale(inp)
    fs = ossd.state_passing(ossd.chunk_state_abs(inp["x"], inp["Bm"], inp["dt"], inp["A"], Q),
                            inp["dt"], inp["A"], Q)[1]
    for name, got, fin in (("one pass", y, final), ("chained", cy, cfinal)):
        check(f"{name} y {shape}", got.cpu().numpy(), ry, scale, bound=2.0 ** -6, rms=2.0 ** -8)
        check(f"{name} final {shape}", fin.cpu().numpy(), rf, np.maximum(fs, 1e-30))


def test_workload_b1_s8k_sampled(ta):
    """The paper's longest single-sequence shape (B=1, L=8192, 64 heads):
    chunk state and chunk scan on every chunk and head, checked on a sample of
    heads against the oracle run on those heads alone."""
    w = gen.SSD_WORKLOADS["ssd_b1_s8k"]
    print(f"ssd {w.name}", flush=True)
    inp = gen.make_ssd_inputs(w, seed=0)
    cb, prev = gen.make_ssd_scan_extras(w, seed=0)
    dx, dB, dC = dev_bf16(inp["x"]), dev_bf16(inp["Bm"]), dev_bf16(inp["Cm"])
    ddt, dA, dD = dev_f32(inp["dt"]), dev_f32(inp["A"]), dev_f32(inp["D"])
    st = ta.ssd_chunk_state(dx, dB, ddt, dA)
    y = ta.ssd_chunk_scan(dx, dC, dev_f32(cb), ddt, dA, dev_f32(prev), dD)
    torch.cuda.synchronize()
    heads = [0, 17, 63]
    sub = dict(x=inp["x"][:, :, heads], Bm=inp["Bm"], Cm=inp["Cm"], dt=inp["dt"][:, :, heads],
               A=inp["A"][heads], D=inp["D"][heads])
    ref_s = ossd.chunk_state(sub["x"], sub["Bm"], sub["dt"], sub["A"], Q)
    sc_s = ossd.chunk_state_abs(sub["x"], sub["Bm"], sub["dt"], sub["A"], Q)
    check("b1_s8k chunk_state", st[:, :, heads].cpu().numpy(), ref_s, sc_s)
    args = (sub["x"], sub["Cm"], cb, sub["dt"], sub["A"], prev[:, :, heads], sub["D"], Q)
    check("b1_s8k chunk_scan", y[:, :, heads].cpu().numpy(), ossd.chunk_scan(*args),
          ossd.chunk_scan_abs(*args))


def test_chunk_state_two_heads_per_workgroup(ta):
    """Grids of at least 1024 two-head workgroups run two heads of a group
    per workgroup: both heads of several pairs, both groups, a ragged last
    chunk, against the oracle on those heads alone."""
    shape = (2, 4000, 64, 2)
    print(f"ssd_chunk_state {shape} (two heads per workgroup)", flush=True)
    w, inp = problem(shape, seed=21)
    out = torch.full((w.B, w.nc, w.H, w.P, w.N), float("nan"), device="cuda")
    ta.ssd_chunk_state(dev_bf16(inp["x"]), dev_bf16(inp["Bm"]), dev_f32(inp["dt"]),
                       dev_f32(inp["A"]), out=out)
    torch.cuda.synchronize()
    assert bool(torch.isfinite(out).all())
    heads = [0, 1, 30, 31, 32, 33, 62, 63]
    groups = [h // (w.H // w.G) for h in heads]
    sub_x, sub_dt, sub_A = inp["x"][:, :, heads], inp["dt"][:, :, heads], inp["A"][heads]
    for i, (h, g) in enumerate(zip(heads, groups)):
        bm = inp["Bm"][:, :, [g]]
        ref = ossd.chunk_state(sub_x[:, :, [i]], bm, sub_dt[:, :, [i]], sub_A[[i]], Q)
        scale = ossd.chunk_state_abs(sub_x[:, :, [i]], bm, sub_dt[:, :, [i]], sub_A[[i]], Q)
        check(f"chunk_state {shape} head {h}", out[:, :, [h]].cpu().numpy(), ref, scale)


def test_repeatable_and_stream(ta):
    """Two runs are bitwise identical; a non-default stream gives the same."""
    w, inp = problem((1, 600, 4, 2), seed=31)
    cb, prev = gen.make_ssd_scan_extras(w, seed=6)
    a = [dev_bf16(inp["x"]), dev_bf16(inp["Cm"]), dev_f32(cb), dev_f32(inp["dt"]),
         dev_f32(inp["A"]), dev_f32(prev), dev_f32(inp["D"])]
    y1 = ta.ssd_chunk_scan(*a)
    y2 = ta.ssd_chunk_scan(*a)
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(s):
        y3 = ta.ssd_chunk_scan(*a, stream=s)
    s.synchronize()
    assert torch.equal(y1, y2) and torch.equal(y1, y3)


@pytest.mark.parametrize("shape,segments", [
    ((1, 1, 1, 1), 1),         # one position
    ((1, 64, 2, 2), 1),        # exactly one step
    ((2, 65, 3, 1), 2),        # one position into the second step, odd heads
    ((1, 300, 4, 2), 3),       # ragged last step, segments of two steps (the last short)
    ((1, 1000, 6, 3), 16),     # a segment per step
    ((2, 200, 256, 2), 1),     # two heads per workgroup
    ((2, 200, 256, 2), 2),     # ... with segments
    ((1, 70, 513, 171), 1),    # groups of three heads: one per workgroup
], ids=str)
def test_forward_one_pass(ta, shape, segments):
    """ssd_forward's kernel (steps of 64 positions, segments) against the
    oracle's chain and the four chained functions, with and without the skip
    term; the same bounds as the chain, whose roundings it has one of."""
    print(f"ssd_forward {shape} segments={segments}", flush=True)
    w, inp = problem(shape, seed=41 + sum(shape))
    dx, dB, dC = dev_bf16(inp["x"]), dev_bf16(inp["Bm"]), dev_bf16(inp["Cm"])
    ddt, dA, dD = dev_f32(inp["dt"]), dev_f32(inp["A"]), dev_f32(inp["D"])
    y, final = ta.ssd_forward(dx, ddt, dA, dB, dC, dD, num_segments=segments)
    y0, final0 = ta.ssd_forward(dx, ddt, dA, dB, dC, None, num_segments=segments)
    states = ta.ssd_chunk_state(dx, dB, ddt, dA)
    prev, cfinal = ta.ssd_state_passing(states, ddt, dA)
    cy = ta.ssd_chunk_scan(dx, dC, ta.ssd_bmm_chunk(dC, dB), ddt, dA, prev, dD)
    torch.cuda.synchronize()
    assert torch.equal(final, final0)
    ry, rf = ossd.ssd_forward(inp["x"], inp["dt"], inp["A"], inp["Bm"], inp["Cm"], inp["D"], Q)
    scale = chained_scale(inp)
    check(f"one pass y {shape}", y.cpu().numpy(), ry, scale, bound=2.0 ** -6, rms=2.0 ** -8)
    # without the skip term: y less D x, to fp32 rounding of that sum
    skip = dD[None, None, :, None] * dx.float()
    assert float((y - y0 - skip).abs().max()) <= 2.0 ** -20 * float(y.abs().max() + skip.abs().max())
    fs = ossd.state_passing(ossd.chunk_state_abs(inp["x"], inp["Bm"], inp["dt"], inp["A"], Q),
                            inp["dt"], inp["A"], Q)[1]
    check(f"one pass final {shape}", final.cpu().numpy(), rf, np.maximum(fs, 1e-30))
    # both paths are within the bound of the same value
    assert float(((y - cy).abs().cpu().numpy() / np.maximum(scale, 1e-30)).max()) <= 2.0 ** -5
    assert float(((final - cfinal).abs().cpu().numpy() / np.maximum(fs, 1e-30)).max()) <= 2.0 ** -6


@pytest.mark.parametrize("shape", [(1, 600, 2, 1), (2, 330, 256, 2)], ids=str)
def test_forward_infinite_state(ta, shape):
    """An infinite B makes one column of the state infinite: every later
    position is the infinity of the product's sign, as in the chained
    functions, not NaN (inf - inf in a split of the state)."""
    print(f"ssd_forward infinite state {shape}", flush=True)
    w, inp = problem(shape, seed=5)
    dx, dB, dC = dev_bf16(inp["x"]), dev_bf16(inp["Bm"]), dev_bf16(inp["Cm"])
    at, n = 10, 5
    dB[:, at, :, n] = float("inf")
    dx[:, at] = torch.where(dx[:, at] < 0, -1.0, 1.0).to(torch.bfloat16)
    dC[..., n] = torch.where(dC[..., n] < 0, -1.0, 1.0).to(torch.bfloat16)
    ddt = torch.full((w.B, w.L, w.H), 0.01, device="cuda")   # (no decay underflows)
    dA = torch.full((w.H,), -1.0, device="cuda")
    y, final = ta.ssd_forward(dx, ddt, dA, dB, dC)
    prev, cfinal = ta.ssd_state_passing(ta.ssd_chunk_state(dx, dB, ddt, dA), ddt, dA)
    cy = ta.ssd_chunk_scan(dx, dC, ta.ssd_bmm_chunk(dC, dB), ddt, dA, prev)
    sign = dx[:, at].float()[:, None] * dC[..., n].float().repeat_interleave(w.H // w.G, 2)[..., None]
    want = torch.where(sign > 0, float("inf"), float("-inf"))[:, at:]
    torch.cuda.synchronize()
    assert torch.equal(cy[:, at:], want)
    assert torch.equal(y[:, at:], want)
    assert torch.isfinite(y[:, :at]).all()
    assert torch.equal(torch.isinf(final), torch.isinf(cfinal))


def infinite_state_problem(shape, c, b, dt, A):
    """One column n of the state infinite from position 10 on, every x and C
    that meets it of size 1 and ``c``: y is the infinity of the product's sign
    from there on.  Returns the inputs of ssd_forward and those y."""
    w, inp = problem(shape, seed=7)
    dx, dB, dC = dev_bf16(inp["x"]), dev_bf16(inp["Bm"]), dev_bf16(inp["Cm"])
    at, n = 10, 5
    dB[:, at, :, n] = b
    dx[:, at] = torch.where(dx[:, at] < 0, -1.0, 1.0).to(torch.bfloat16)
    dC[..., n] = torch.where(dC[..., n] < 0, -c, c).to(torch.bfloat16)
    ddt = torch.full((w.B, w.L, w.H), dt, device="cuda")
    dA = torch.full((w.H,), A, device="cuda")
    sign = dx[:, at].float()[:, None] * dC[..., n].float().repeat_interleave(w.H // w.G, 2)[..., None] * b
    return (dx, ddt, dA, dB, dC), torch.where(sign > 0, float("inf"), float("-inf"))[:, at:], at


@pytest.mark.parametrize("b", [float("inf"), float("-inf")])
@pytest.mark.parametrize("shape", [(1, 600, 2, 1), (2, 330, 256, 2)], ids=str)
def test_forward_infinite_state_and_large_c(ta, shape, b):
    """The low part of an infinite state must not meet C at all: any finite
    stand-in of the other sign overflows against a large one, to NaN."""
    print(f"ssd_forward infinite state {shape} {b}, C = 512", flush=True)
    args, want, at = infinite_state_problem(shape, 512.0, b, 0.01, -1.0)
    y, final = ta.ssd_forward(*args)
    cy, cfinal = chained(ta, *args)
    torch.cuda.synchronize()
    assert torch.equal(cy[:, at:], want) and torch.equal(y[:, at:], want)
    assert torch.isfinite(y[:, :at]).all()
    assert torch.equal(torch.isinf(final), torch.isinf(cfinal)) and not torch.isnan(final).any()


@pytest.mark.parametrize("shape,segments", [((1, 1600, 2, 1), 5), ((2, 1000, 256, 2), 3)], ids=str)
def test_forward_infinite_state_over_segments(ta, shape, segments):
    """A segment of 320 or more positions whose decay underflows fp32, while that
    of a chunk of 256 does not (2^-124): the infinite state is carried past it,
    as in one walk and in the chained functions."""
    print(f"ssd_forward infinite state {shape} in {segments} segments", flush=True)
    args, want, at = infinite_state_problem(shape, 1.0, float("inf"), 0.0335, -10.0)
    y1, final1 = ta.ssd_forward(*args, num_segments=1)
    y, final = ta.ssd_forward(*args, num_segments=segments)
    cy, cfinal = chained(ta, *args)
    torch.cuda.synchronize()
    for v in (cy, y1, y):
        assert torch.equal(v[:, at:], want)
    assert torch.isfinite(y[:, :at]).all()
    for f in (final1, final):
        assert torch.equal(torch.isinf(f), torch.isinf(cfinal)) and not torch.isnan(f).any()


def large_problem(B, L, H, G, dt, A):
    """Inputs of ssd_forward drawn on the GPU: unit normals, dt and A uniform
    between the bounds given."""
    g = torch.Generator(device="cuda").manual_seed(B + L + H)
    r = lambda *s: torch.randn(s, generator=g, device="cuda").to(torch.bfloat16)
    u = lambda lo, hi, *s: torch.rand(s, generator=g, device="cuda") * (hi - lo) + lo
    return (r(B, L, H, 64), u(*dt, B, L, H), u(*A, H), r(B, L, G, 128), r(B, L, G, 128),
            u(0.5, 1.5, H))


def check_head(tag, args, y, final, b, h, lo=0, keep=0):
    """One head of one batch element against the oracle run on it alone, from
    position ``lo`` (its state there taken as zero) and compared from
    ``lo + keep`` on."""
    x, dt, A, Bm, Cm, D = args
    grp = h // (x.shape[2] // Bm.shape[2])
    bits = lambda a: a.contiguous().view(torch.int16).cpu().numpy().view(np.uint16)
    f32 = lambda a: a.contiguous().cpu().numpy()
    one = slice(b, b + 1)
    inp = dict(x=bits(x[one, lo:, h:h + 1]), Bm=bits(Bm[one, lo:, grp:grp + 1]),
               Cm=bits(Cm[one, lo:, grp:grp + 1]), dt=f32(dt[one, lo:, h:h + 1]),
               A=f32(A[h:h + 1]), D=f32(D[h:h + 1]))
    ry, rf = ossd.ssd_forward(inp["x"], inp["dt"], inp["A"], inp["Bm"], inp["Cm"], inp["D"], Q)
    got = f32(y[one, lo:, h:h + 1])
    check(f"{tag} y head {h} of {b}", got[:, keep:], ry[:, keep:], chained_scale(inp)[:, keep:],
          bound=2.0 ** -6, rms=2.0 ** -8)
    if final is not None:
        fs = ossd.state_passing(ossd.chunk_state_abs(inp["x"], inp["Bm"], inp["dt"], inp["A"], Q),
                                inp["dt"], inp["A"], Q)[1]
        check(f"{tag} final head {h} of {b}", f32(final[one, h:h + 1]), rf, np.maximum(fs, 1e-30))


@pytest.mark.parametrize("shape", [(23, 1001, 64, 1), (23, 1001, 63, 21), (1, 130, 1 << 17, 1),
                                   (1, 130, 1 << 17, 1 << 17), (1, 70, (1 << 17) + 1, 1)], ids=str)
def test_forward_streamed_x(ta, shape):
    """x and y past 512 MB together: x is read with the non-temporal policy, by
    two heads per workgroup and by one (three heads in a group); ragged L.
    The most heads, in one group and in as many: rows of x, y, B and C at
    their widest (64 rows of y span 2^31 bytes); one head more runs the
    functions chained."""
    print(f"ssd_forward streamed {shape}", flush=True)
    B, L, H, G = shape
    args = large_problem(B, L, H, G, (1e-3, 1e-1), (-16.0, -1.0))
    y, final = ta.ssd_forward(*args)
    torch.cuda.synchronize()
    assert torch.isfinite(y).all() and torch.isfinite(final).all()
    for b, h in ((0, 0), (0, H - 1), (B // 2, H // 2 - 1), (B - 1, H // 2), (B - 1, H - 1)):
        check_head(f"streamed {shape}", args, y, final, b, h)


@pytest.mark.parametrize("segments", [1, None])
def test_forward_past_4_gib_per_batch_element(ta, segments):
    """y of one batch element past 4 GiB, beyond what one 32-bit buffer range
    covers: both ends of the sequence and the middle.  With these decays a
    state is gone after 300 positions (e^-0.4 and less at each)."""
    B, L, H, G = 1, (1 << 18) + 333, 64, 1
    print(f"ssd_forward L={L} segments={segments}", flush=True)
    args = large_problem(B, L, H, G, (5e-2, 1e-1), (-16.0, -8.0))
    y, final = ta.ssd_forward(*args, num_segments=segments)
    torch.cuda.synchronize()
    assert torch.isfinite(y).all() and torch.isfinite(final).all()
    first = tuple(a[:, :1000] if a.dim() > 1 else a for a in args)
    mid = tuple(a[:, L // 2:L // 2 + 1000] if a.dim() > 1 else a for a in args)
    for h in (0, 63):
        check_head("first rows", first, y[:, :1000], None, 0, h)
        check_head("middle rows", mid, y[:, L // 2:L // 2 + 1000], None, 0, h, keep=300)
        check_head("last rows", args, y, final, 0, h, lo=L - 900, keep=300)


def test_forward_without_final_states_and_on_a_side_stream(ta):
    """final_states NULL through the C ABI, and a call on another stream while
    the current one has a write queued into a freed block of the workspace's
    size: the same y bit for bit, and the block is left alone."""
    B, L, H, G = 1, 1000, 64, 1
    args = large_problem(B, L, H, G, (1e-3, 1e-1), (-16.0, -1.0))
    x, dt, A, Bm, Cm, D = args
    y, final = ta.ssd_forward(*args)
    n = ta.ssd_segment_heuristic(B, L, H)
    assert n > 1
    need = ta.ssd_forward_workspace_bytes(B, L, H, n)
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    y2 = torch.full_like(y, float("nan"))
    rc = ta.lib().ssd_forward(x.data_ptr(), Bm.data_ptr(), Cm.data_ptr(), dt.data_ptr(), A.data_ptr(),
                              D.data_ptr(), y2.data_ptr(), None, B, L, H, G, 64, 128, n, ws.data_ptr(),
                              need, torch.cuda.current_stream().cuda_stream)
    assert rc == 0
    slow = torch.zeros(1 << 27, device="cuda")
    s = torch.cuda.Stream()
    torch.cuda.synchronize()
    assert torch.equal(y, y2)
    del ws, y2
    torch.cuda.empty_cache()
    outputs = [torch.empty_like(y), torch.empty_like(final)]   # (blocks for the call's outputs)
    block = torch.empty(need, dtype=torch.uint8, device="cuda")
    where = block.data_ptr()
    torch.cuda.synchronize()
    for _ in range(8):
        slow.add_(1.0)
    block.fill_(0xFF)            # queued behind them (fp32 NaN)
    del block, outputs
    y3, final3 = ta.ssd_forward(*args, stream=s)
    again = torch.empty(need, dtype=torch.uint8, device="cuda")
    assert again.data_ptr() == where, "the current stream's block went to the call"
    torch.cuda.synchronize()
    assert torch.equal(y, y3) and torch.equal(final, final3)
