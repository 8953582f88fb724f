"""GPU parity of attn_fwd_split (key range split over workgroups, partial
results merged by a second kernel) through the C ABI, against the fp64
oracle, at the stated tolerance: max |O - O_ref| <= 2e-2 and
max |LSE - LSE_ref| <= 1e-3.  Cases include splits that are empty for some
query tiles (causal), rows that see no key of a split, a split count above
the number of key tiles, bf16 output, and reuse of one workspace."""
import numpy as np
import pytest

import oracle
from paper_2504_17577_amd import gen

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

O_TOL, LSE_TOL = 2e-2, 1e-3


@pytest.fixture(scope="module")
def ta():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2504_17577_amd import tileattn
    tileattn.lib()
    return tileattn


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a).view(np.int16)).view(torch.bfloat16).cuda()


def run_split(ta, q, k, v, causal, scale, splits, out_dtype=torch.float32, workspace=None):
    B, Hq, Sq, D = q.shape
    o = torch.full((B, Hq, Sq, D), float("nan"), dtype=out_dtype, device="cuda")
    lse = torch.full((B, Hq, Sq), float("nan"), dtype=torch.float32, device="cuda")
    dq, dk, dv = dev(q), dev(k), dev(v)
    ta.attn_fwd_split(dq, dk, dv, causal=causal, scale=scale, num_splits=splits, out=o, lse=lse,
                      workspace=workspace, out_dtype=out_dtype)
    torch.cuda.synchronize()
    return o, lse


CASES = [
    # (B, Hq, Hkv, Sq, Sk, D, causal, splits)
    (1, 2, 2, 128, 128, 64, False, 2),
    (4, 16, 16, 1024, 1024, 64, True, 3),
    (4, 16, 16, 1024, 1024, 64, True, 5),
    (1, 8, 1, 200, 1000, 128, True, 7),     # some splits empty for early query tiles
    (2, 6, 3, 65, 63, 64, False, 4),        # one key tile: runs unsplit
    (1, 4, 4, 1, 1000, 128, True, 16),      # a single query row, 16 tiles
    (1, 4, 2, 300, 300, 128, True, 128),    # more splits than key tiles
    (1, 2, 2, 129, 4000, 128, False, 9),    # ragged last tile inside the last split
    # a wave whose rows partly see no key of the last split: lanes with no key
    # yet sit in a wave that raises its running max (regression: NaN weights)
    (1, 8, 2, 300, 2000, 128, True, 6),
]


@pytest.mark.parametrize("case", CASES, ids=[str(c) for c in CASES])
def test_split_against_oracle(ta, case):
    B, Hq, Hkv, Sq, Sk, D, causal, splits = case
    print(f"split case {case}", flush=True)
    q, k, v = gen.random_problem(B, Hq, Hkv, Sq, Sk, D, seed=11)
    scale = D ** -0.5
    o, lse = run_split(ta, q, k, v, causal, scale, splits)
    ro, rl = oracle.attn_fwd(q, k, v, causal, scale)
    o, lse = o.cpu().numpy(), lse.cpu().numpy()
    assert np.isfinite(o).all() and np.isfinite(lse).all()
    eo, el = float(np.abs(o - ro).max()), float(np.abs(lse - rl).max())
    print(f"  max|dO|={eo:.3e} max|dLSE|={el:.3e}", flush=True)
    assert eo <= O_TOL and el <= LSE_TOL


@pytest.mark.parametrize("name,splits", [("chunk_causal_d128_q1k_k8k", "auto"),
                                         ("cross_d128_q512_k4k", "auto"),
                                         ("paper_fa0_s512_causal", 4), ("paper_fa1_s512", 4)])
def test_split_workload_sampled(ta, name, splits):
    """Full-size workload with the heuristic split count (the bench's launch
    configuration for --splits auto) or a fixed one: sampled rows against the
    oracle."""
    w = gen.WORKLOADS[name]
    q, k, v = gen.make_inputs(w, seed=0)
    n = (ta.ta_split_heuristic(w.B, w.Hq, w.Hkv, w.Sq, w.Sk, w.D, w.causal)
         if splits == "auto" else splits)
    print(f"split workload {name}: {n} splits", flush=True)
    assert n > 1
    o, lse = run_split(ta, q, k, v, w.causal, w.scale, n)
    assert bool(torch.isfinite(o).all()) and bool(torch.isfinite(lse).all())
    rng = np.random.default_rng(3)
    rows = sorted({(int(rng.integers(w.B)), int(rng.integers(w.Hq)), int(rng.integers(w.Sq)))
                   for _ in range(300)} | {(0, 0, 0), (w.B - 1, w.Hq - 1, w.Sq - 1)})
    ro, rl = oracle.attn_rows(q, k, v, w.causal, w.scale, rows)
    idx = tuple(torch.tensor(c) for c in zip(*rows))
    eo = float(np.abs(o[idx].cpu().numpy() - ro).max())
    el = float(np.abs(lse[idx].cpu().numpy() - rl).max())
    print(f"  {len(rows)} rows: max|dO|={eo:.3e} max|dLSE|={el:.3e}", flush=True)
    assert eo <= O_TOL and el <= LSE_TOL


def test_split_bf16_out_is_rounded_fp32_and_deterministic(ta):
    q, k, v = gen.random_problem(1, 8, 2, 300, 2000, 128, seed=4)
    o32, l32 = run_split(ta, q, k, v, True, 128 ** -0.5, 6)
    o32b, l32b = run_split(ta, q, k, v, True, 128 ** -0.5, 6)
    o16, l16 = run_split(ta, q, k, v, True, 128 ** -0.5, 6, out_dtype=torch.bfloat16)
    assert bool(torch.isfinite(o32).all()) and bool(torch.isfinite(l32).all())
    assert torch.equal(o32.view(torch.int32), o32b.view(torch.int32))
    assert torch.equal(l32.view(torch.int32), l32b.view(torch.int32))
    assert torch.equal(o16.view(torch.int16), o32.to(torch.bfloat16).view(torch.int16))
    assert torch.equal(l16.view(torch.int32), l32.view(torch.int32))


def test_split_workspace_reused(ta):
    """One workspace for two calls in a row, the second smaller; stale
    partial results of the first must not leak into the second."""
    big = gen.random_problem(2, 8, 8, 256, 3000, 64, seed=21)
    small = gen.random_problem(1, 4, 4, 100, 700, 64, seed=22)
    need = ta.ta_split_workspace_bytes(2, 8, 256, 64, 8)
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    for (q, k, v), causal in ((big, False), (small, True)):
        o, lse = run_split(ta, q, k, v, causal, 0.125, 8, workspace=ws)
        ro, rl = oracle.attn_fwd(q, k, v, causal, 0.125)
        assert float(np.abs(o.cpu().numpy() - ro).max()) <= O_TOL
        assert float(np.abs(lse.cpu().numpy() - rl).max()) <= LSE_TOL


def test_split_rejects_small_workspace(ta):
    q, k, v = gen.random_problem(1, 2, 2, 64, 512, 64, seed=1)
    need = ta.ta_split_workspace_bytes(1, 2, 64, 64, 4)
    ws = torch.empty(need - 16, dtype=torch.uint8, device="cuda")
    with pytest.raises(ta.TileAttnError) as e:
        ta.attn_fwd_split(dev(q), dev(k), dev(v), num_splits=4, workspace=ws)
    assert e.value.status == 8


def test_split_side_stream_with_its_own_workspace(ta):
    """attn_fwd_split and mla_decode on a non-default stream, each allocating
    its workspace (on that stream): the same bits as on the default stream,
    while the default stream allocates and fills memory of the workspace's
    size right after the launch, which must not be the workspace's block."""
    q, k, v = (dev(a) for a in gen.random_problem(2, 8, 8, 512, 4000, 128, seed=31))
    o_ref, l_ref = ta.attn_fwd_split(q, k, v, num_splits=6)
    mq, mqp, mkv, mkp = (dev(a) for a in gen.random_mla_problem(4, 128, 1, 3000, seed=32))
    mo_ref, ml_ref = ta.mla_decode(mq, mqp, mkv, mkp, num_splits=5)
    need = max(ta.ta_split_workspace_bytes(2, 8, 512, 128, 6), ta.mla_workspace_bytes(4, 128, 5))
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    # launched on s from the default stream: the outputs are allocated on the
    # default stream, whose next allocation follows, the workspaces on s
    o, lse = ta.attn_fwd_split(q, k, v, num_splits=6, stream=s)
    mo, ml = ta.mla_decode(mq, mqp, mkv, mkp, num_splits=5, stream=s)
    junk = torch.full((need // 4 + 1,), float("nan"), dtype=torch.float32, device="cuda")
    torch.cuda.synchronize()
    del junk
    assert torch.equal(o, o_ref) and torch.equal(lse, l_ref)
    assert torch.equal(mo, mo_ref) and torch.equal(ml, ml_ref)


@pytest.mark.parametrize("case", [
    # (B, Hq, Hkv, Sq, Sk, D, causal, splits): up to 16 query rows per K/V head
    (1, 1, 1, 1, 1, 128, True, 1),          # one key
    (2, 2, 1, 1, 31, 64, False, 1),         # less than a tile
    (1, 16, 1, 1, 257, 128, False, 1),      # all 16 rows, one key past eight waves' tiles
    (2, 8, 4, 8, 300, 64, True, 1),         # 16 rows over two heads, diagonal in the last tile
    (1, 3, 3, 16, 16, 128, True, 1),        # square causal: rows see 1 .. 16 keys
    (1, 10, 2, 3, 1000, 128, True, 1),      # 15 rows
    (3, 8, 2, 1, 1000, 64, False, 3),       # splits of whole tiles, ragged end
    (1, 4, 1, 4, 130, 128, True, 3),        # last split seen by some rows only
    (2, 32, 8, 1, 4099, 128, False, 16),
], ids=str)
@pytest.mark.parametrize("out_dtype", [torch.float32, torch.bfloat16], ids=["fp32", "bf16"])
def test_decode_rows_against_oracle(ta, case, out_dtype):
    B, Hq, Hkv, Sq, Sk, D, causal, splits = case
    print(f"decode case {case} {out_dtype}", flush=True)
    q, k, v = gen.random_problem(B, Hq, Hkv, Sq, Sk, D, seed=17)
    o, lse = run_split(ta, q, k, v, causal, D ** -0.5, splits, out_dtype=out_dtype)
    ro, rl = oracle.attn_fwd(q, k, v, causal, D ** -0.5)
    o, lse = o.float().cpu().numpy(), lse.cpu().numpy()
    assert np.isfinite(o).all() and np.isfinite(lse).all()
    eo, el = float(np.abs(o - ro).max()), float(np.abs(lse - rl).max())
    print(f"  max|dO|={eo:.3e} max|dLSE|={el:.3e}", flush=True)
    assert eo <= O_TOL and el <= LSE_TOL
    # scale 0: every visible key weighs the same
    _, lse0 = run_split(ta, q, k, v, causal, 0.0, splits, out_dtype=out_dtype)
    seen = np.array([min(Sk, i + 1 + Sk - Sq) if causal else Sk for i in range(Sq)])
    assert float(np.abs(lse0.cpu().numpy() - np.log(seen)).max()) <= 1e-5


@pytest.mark.parametrize("case", [
    # (B, Hq, Hkv, Sq, Sk, D, causal): both sides of the choice between the
    # decode and the tiled kernel
    (4, 8, 8, 1, 64, 64, False), (5, 64, 64, 1, 65, 64, False), (75, 4, 4, 1, 447, 64, True),
    (75, 4, 4, 1, 448, 64, True), (80, 4, 4, 2, 640, 128, True), (79, 4, 4, 2, 640, 128, True),
    (150, 4, 2, 3, 64, 64, True), (150, 4, 2, 3, 65, 64, False), (100, 9, 3, 5, 16, 128, True),
], ids=str)
def test_decode_route_boundaries(ta, case):
    B, Hq, Hkv, Sq, Sk, D, causal = case
    print(f"decode route {case} decode={ta.ta_decode_route(B, Hq, Hkv, Sq, Sk, D, 1)}", flush=True)
    q, k, v = gen.random_problem(B, Hq, Hkv, Sq, Sk, D, seed=29)
    ro, rl = oracle.attn_fwd(q, k, v, causal, D ** -0.5)
    for f in (ta.attn_fwd, ta.attn_fwd_bf16out):
        o, lse = f(dev(q), dev(k), dev(v), causal=causal)
        torch.cuda.synchronize()
        assert float(np.abs(o.float().cpu().numpy() - ro).max()) <= O_TOL
        assert float(np.abs(lse.cpu().numpy() - rl).max()) <= LSE_TOL


@pytest.mark.parametrize("case", [
    # (B, Hq, Hkv, Sq, Sk, D, causal, splits): splits that take a call of few
    # query rows to the tiled kernel, and the same splits with longer keys
    (16, 4, 4, 1, 2048, 64, False, 8), (16, 4, 4, 3, 2000, 64, True, 8),
    (16, 4, 4, 3, 4096, 64, True, 8), (75, 2, 2, 1, 1200, 128, False, 2),
], ids=str)
def test_decode_route_boundaries_split(ta, case):
    B, Hq, Hkv, Sq, Sk, D, causal, splits = case
    print(f"decode route {case} decode={ta.ta_decode_route(B, Hq, Hkv, Sq, Sk, D, splits)}", flush=True)
    q, k, v = gen.random_problem(B, Hq, Hkv, Sq, Sk, D, seed=37)
    o, lse = run_split(ta, q, k, v, causal, D ** -0.5, splits)
    ro, rl = oracle.attn_fwd(q, k, v, causal, D ** -0.5)
    assert float(np.abs(o.cpu().numpy() - ro).max()) <= O_TOL
    assert float(np.abs(lse.cpu().numpy() - rl).max()) <= LSE_TOL
