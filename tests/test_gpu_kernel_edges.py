"""Kernels at the edges of their tiles and of the ranges their dispatch rules
cover, against the fp64 oracle (tolerance: TOL of the harness, the bound on
one output tensor's max error that the rounding of bf16 intermediates or of
the fp32 path's sums stays below)."""
import numpy as np
import pytest

import moe_workloads as mw
from gpu_harness import TOL, device_case, host, log, relerr, run_bwd, run_fwd, torch
from oracle import moe as om

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mf():
    t = torch()
    if not t.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2511_21431_amd as m
    m.lib()
    return m


def _check_bwd(mf, w, seed, C, accumulate, **opts):
    t = torch()
    case = mw.make_case(w, seed)
    dev = device_case(w, case)
    ref = om.moe_bwd(case["X"], case["idx"], case["gates"], case["W1"], case["W2"],
                     case["dY"], C)
    dW = None
    if accumulate:
        gen = t.Generator(device="cuda")
        gen.manual_seed(seed)
        dW = [t.randn(s, generator=gen, device="cuda") for s in
              ((w.E, 2 * w.F, w.h), (w.E, w.h, w.F))]
        base = [x.double().cpu().numpy() for x in dW]
    try:
        mf.memfine_set_launch_options(**opts)
        got = run_bwd(w, dev, C, dW=dW, accumulate=accumulate)
    finally:
        mf.memfine_set_launch_options()
    if accumulate:
        ref = dict(ref, dW1=ref["dW1"] + base[0], dW2=ref["dW2"] + base[1])
    for key in ("dX", "dgates", "dW1", "dW2"):
        err = relerr(host(got[key]), ref[key])
        log(f"  {key} {err:.2e}")
        assert err <= TOL[w.dtype], (key, err)


# Weight-gradient epilogue: a 32 x 32 block is stored whole or not at all, so
# every count of valid 64-row and 64-column pieces in a last tile of 256 or
# 128, with dW overwritten, added to by a second chunk and added to throughout.
# bf16, 160 experts of 320 x 320: 960 and 640 tiles of 256 x 256, the persistent launch
# with its tile counter, FC2's last half round in quarter tiles; fp32 there: 2400 and
# 1440 tiles of 128 x 128 (the smaller cases take 64 x 64).
@pytest.mark.parametrize("h,F,E,dtype", [
    (64, 64, 4, "bf16"), (128, 192, 3, "bf16"), (192, 64, 5, "bf16"), (320, 192, 80, "bf16"),
    (448, 320, 2, "bf16"), (320, 320, 160, "bf16"), (192, 320, 3, "f32"), (64, 64, 2, "f32"),
    (320, 320, 160, "f32")])
@pytest.mark.parametrize("accumulate", [False, True])
def test_wgrad_tile_edges(mf, h, F, E, dtype, accumulate):
    w = mw.Workload("edge", T=321, h=h, F=F, E=E, k=2, dtype=dtype, routing="dirichlet")
    log(f"wgrad edges h={h} F={F} E={E} {dtype} accumulate={accumulate}")
    for opts in ({}, {"tile": mf.TILE_256}) if dtype == "bf16" else ({},):
        _check_bwd(mf, w, 300 + h + F, 2, accumulate, **opts)


# Tile shape by rows per expert (48 and 320 of an average expert): both sides
# of each line, ragged and skewed loads, one row in all; and E = 80, where the
# tiles are located by walking the experts.  Every shape gives the same bits.
@pytest.mark.parametrize("T,E,h,F", [(1, 4, 192, 128), (96, 4, 320, 192), (97, 4, 320, 192),
                                     (639, 4, 192, 320), (640, 4, 192, 320), (37, 80, 128, 64),
                                     (2000, 80, 64, 128)])
def test_tile_shape_by_rows(mf, T, E, h, F):
    w = mw.Workload("rows", T=T, h=h, F=F, E=E, k=2, dtype="bf16", routing="dirichlet")
    log(f"tile shape T={T} E={E} h={h} F={F}")
    case = mw.make_case(w, 900 + T)
    dev = device_case(w, case)
    Y = host(run_fwd(w, dev, 1))
    assert relerr(Y, om.moe_fwd(case["X"], case["idx"], case["gates"], case["W1"], case["W2"],
                                1)) <= TOL["bf16"]
    _check_bwd(mf, w, 900 + T, 1, False)
    B = {k: host(v) for k, v in run_bwd(w, dev, 1).items()}
    for tile in (mf.TILE_128, mf.TILE_256):
        try:
            mf.memfine_set_launch_options(tile=tile)
            assert np.array_equal(host(run_fwd(w, dev, 1)), Y), tile
            other = {k: host(v) for k, v in run_bwd(w, dev, 1).items()}
        finally:
            mf.memfine_set_launch_options()
        for key in B:
            assert np.array_equal(other[key], B[key]), (tile, key)


# The same with enough experts for the other lines of the rule: 200 rows per expert
# with 160 tiles of 256 x 256 (32 experts; FC2 and FC1 dgrad), past 64 experts 40 and
# 129 rows (160 tiles; 80 for FC1 and FC2 dgrad) and a nearly full last round (240
# tiles, 60 rows); 256 and 160 tiles of 128 x 128 (64 x 128 then); and expert-ordered
# chunks, whose rows come from a few of the experts.
@pytest.mark.parametrize("T,E,h,F", [(3184, 32, 1024, 64), (3185, 32, 1024, 64), (2048, 32, 1024, 64),
                                     (2048, 32, 640, 64), (3184, 32, 128, 1024),
                                     (3185, 32, 128, 1024), (1600, 80, 320, 64),
                                     (1601, 80, 320, 64), (5120, 80, 320, 128),
                                     (5121, 80, 320, 128), (2400, 80, 576, 64),
                                     (2560, 32, 320, 192)])
def test_tile_shape_by_rows_and_grid(mf, T, E, h, F):
    test_tile_shape_by_rows(mf, T, E, h, F)
    w = mw.Workload("rows", T=T, h=h, F=F, E=E, k=2, dtype="bf16", routing="dirichlet")
    _check_bwd(mf, w, 900 + T, 5, True, chunk_order=mf.CHUNK_EXPERTS)


# Weight gradients: 128 x 128 tiles below a grid of 640 tiles of 256 x 256 (here
# one per expert), the larger ones from there; most experts have no row.
@pytest.mark.parametrize("E", [639, 640])
def test_wgrad_tile_shape_by_grid(mf, E):
    w = mw.Workload("wgrid", T=777, h=64, F=64, E=E, k=2, dtype="bf16", routing="dirichlet",
                    alpha=0.3)
    log(f"wgrad tile shape E={E}")
    for accumulate in (False, True):
        _check_bwd(mf, w, 70 + E, 2, accumulate)


# The rows at which fewer than 640 tiles of 256 x 256 take the larger shape: 4096 per
# expert from 448 tiles (512 here, FC1 wgrad), and one that hangs over dW's edges too
# much for it (495 tiles, dW1 of 1152 x 2112); with a tile option forcing the other shape
# the bits are the same.
@pytest.mark.parametrize("T,E,h,F", [(8191, 4, 2048, 2048), (8192, 4, 2048, 2048),
                                     (22600, 11, 2112, 576)])
def test_wgrad_tile_shape_by_rows(mf, T, E, h, F):
    w = mw.Workload("wrows", T=T, h=h, F=F, E=E, k=2, dtype="bf16", routing="dirichlet")
    log(f"wgrad tile shape T={T} E={E} h={h} F={F}")
    t = torch()
    rng = np.random.default_rng(T)
    dev = {"X": t.randn((T, h), device="cuda").bfloat16(), "dY": t.randn((T, h), device="cuda").bfloat16(),
           "W1": (t.randn((E, 2 * F, h), device="cuda") / 16).bfloat16(),
           "W2": (t.randn((E, h, F), device="cuda") / 16).bfloat16(),
           "idx": t.from_numpy(rng.integers(0, E, (T, 2)).astype(np.int32)).cuda(),
           "gates": t.rand((T, 2), device="cuda")}
    got = []
    for tile in (mf.TILE_AUTO, mf.TILE_128, mf.TILE_256):
        try:
            mf.memfine_set_launch_options(tile=tile)
            got.append(run_bwd(w, dev, 1))
        finally:
            mf.memfine_set_launch_options()
    for key in got[0]:
        assert t.equal(got[0][key], got[1][key]) and t.equal(got[0][key], got[2][key]), key
    # dW2 = (gate * dY)^T a, by expert in float64
    x, y, g = dev["X"].double(), dev["dY"].double(), dev["gates"].double()
    e = E - 1
    tok, slot = (dev["idx"] == e).nonzero(as_tuple=True)
    u = x[tok] @ dev["W1"][e].double().T
    a = t.nn.functional.silu(u[:, :F]) * u[:, F:]
    ref = (g[tok, slot][:, None] * y[tok]).T @ a
    assert float((got[0]["dW2"][e].double() - ref).abs().max() / ref.abs().max()) <= TOL["bf16"]


# fp32: 64-row tiles below 1280 tiles of 128 x 128, the larger ones from there
# (FC1: F / 64 = 256 column tiles x 4 and x 5 row tiles; FC2 dgrad: 319 and 320 x 4;
# FC2 and FC1 dgrad the same).
@pytest.mark.parametrize("T,h,F", [(512, 64, 16384), (640, 64, 16384), (512, 64, 40832),
                                   (512, 64, 40960), (512, 40832, 64), (512, 40960, 64)])
def test_f32_tile_shape_by_grid(mf, T, h, F):
    w = mw.Workload("grid", T=T, h=h, F=F, E=1, k=1, dtype="f32", routing="dirichlet")
    log(f"f32 tile shape T={T} h={h} F={F}")
    case = mw.make_case(w, 40 + T)
    dev = device_case(w, case)
    Y = host(run_fwd(w, dev, 1))
    assert relerr(Y, om.moe_fwd(case["X"], case["idx"], case["gates"], case["W1"], case["W2"],
                                1)) <= TOL["f32"]
    _check_bwd(mf, w, 40 + T, 1, False)


# Dispatch in one launch up to 2048 slots and 256 experts, and the count in one
# workgroup up to 8192 slots: both sides of each line, dropped ids among them,
# a chunk that starts inside the ids, and one expert taking every slot.
@pytest.mark.parametrize("T,k,E", [(1, 1, 1), (512, 4, 256), (512, 4, 257), (683, 3, 9),
                                   (1024, 8, 300), (2731, 3, 64), (4, 1, 1024),
                                   (4096, 6, 64), (6000, 5, 65), (3000, 1, 1), (3000, 2, 5)])
@pytest.mark.parametrize("hot", [False, True])
def test_dispatch_and_count_lines(mf, T, k, E, hot):
    t = torch()
    log(f"dispatch lines T={T} k={k} E={E} hot={hot}")
    rng = np.random.default_rng(T * k + E)
    idx = np.full((T, k), E - 1) if hot else rng.integers(0, E, size=(T, k))
    idx = idx.astype(np.int32)
    s = mf.make_shape(T, 64, 64, E, k, mf.BF16)
    work = t.full((E + 1,), -7, dtype=t.int32, device="cuda")
    assert mf.memfine_count(s, t.from_numpy(idx).cuda(), work).tolist() == \
        om.expert_counts(idx, E).tolist()
    assert work.cpu().numpy().tolist() == om.expert_counts(idx, E).tolist() + [0]
    if T * k > 2 and not hot:
        idx[0, 0], idx[-1, -1] = E, -1
        with pytest.raises(mf.MemfineError):
            mf.memfine_count(s, t.from_numpy(idx).cuda(), work)
        assert int(work[E]) == 2
    for t0, t1 in ((0, T), (T // 3, T)):
        n = (t1 - t0) * k
        out = [t.full((m,), -7, dtype=t.int32, device="cuda") for m in (E, E + 1, n, n)]
        mf.memfine_dispatch(s, t.from_numpy(idx).cuda(), t0, t1, *out)
        c, o, ss, rs = (x.cpu().numpy() for x in out)
        flat = idx.reshape(-1)[t0 * k:t1 * k]
        ok = (flat >= 0) & (flat < E)
        order = np.argsort(np.where(ok, flat, E), kind="stable")[:int(ok.sum())]
        assert c.tolist() == np.bincount(flat[ok], minlength=E).tolist()
        assert o.tolist() == np.concatenate(([0], np.cumsum(c))).tolist()
        assert ss[:order.size].tolist() == (order + t0 * k).tolist()
        want = np.full(n, -1)
        want[order] = np.arange(order.size)
        assert rs.tolist() == want.tolist()


# FC1 dgrad and both weight gradients in one launch for small problems: the
# line of each of its conditions (rows per expert 320, 160 with many experts, fp32 grids), the bits
# of the separate launches (forced by a tile option in bf16), both chunk orders.
@pytest.mark.parametrize("T,E,h,F,dtype", [(639, 4, 192, 320, "bf16"), (640, 4, 192, 320, "bf16"),
                                           (6360, 80, 320, 64, "bf16"), (6400, 80, 320, 64, "bf16"),
                                           (50, 5, 64, 64, "bf16"), (300, 3, 192, 128, "f32"),
                                           (200, 70, 64, 64, "f32")])
def test_bwd_in_one_launch(mf, T, E, h, F, dtype):
    w = mw.Workload("merge", T=T, h=h, F=F, E=E, k=2, dtype=dtype, routing="dirichlet")
    log(f"one launch T={T} E={E} {dtype}")
    for C, order in ((1, mf.CHUNK_TOKENS), (3, mf.CHUNK_TOKENS), (2, mf.CHUNK_EXPERTS)):
        for accumulate in (False, True):
            _check_bwd(mf, w, 50 + T + E, C, accumulate, chunk_order=order)
    if dtype == "bf16":
        dev = device_case(w, mw.make_case(w, 50 + T + E))
        one = {k: host(v) for k, v in run_bwd(w, dev, 1).items()}
        try:
            mf.memfine_set_launch_options(tile=mf.TILE_128)
            three = {k: host(v) for k, v in run_bwd(w, dev, 1).items()}
        finally:
            mf.memfine_set_launch_options()
        for key in one:
            assert np.array_equal(one[key], three[key]), key


# Router: both sides of the logits GEMM's tile rules (one round of 64-row, then
# of 128-row tiles), the dz rows' 64-token workgroups, and routers too small
# for a whole tile.  T = 1 and 65 also at 96 logits (dX from the dz kernel's
# per-token form).
@pytest.mark.parametrize("T,E,k", [(1, 256, 8), (65, 96, 3), (65, 128, 16), (16384, 256, 2),
                                   (16385, 256, 2), (32768, 256, 4), (32769, 256, 4)])
def test_router_tile_rules(mf, T, E, k):
    from oracle import router as orr
    t = torch()
    h = 64
    log(f"router rules T={T} E={E} k={k}")
    rng = np.random.default_rng(T + E)
    X = mw.round_to_bf16(rng.standard_normal((T, h)))
    Wr = mw.round_to_bf16(rng.standard_normal((E, h)) / 8)
    dg = rng.standard_normal((T, k)).astype(np.float32)
    Xd, Wd = (t.from_numpy(a).cuda().bfloat16() for a in (X, Wr))
    s = mf.make_shape(T, h, 64, E, k, mf.BF16)
    idx = t.full((T, k), -1, dtype=t.int32, device="cuda")
    gates, logits = t.empty((T, k), device="cuda"), t.empty((T, E), device="cuda")
    mf.memfine_router_fwd(s, Xd, Wd, idx, gates, logits)
    lg = host(logits)
    assert relerr(lg, orr.logits_of(X, Wr)) <= 1e-5      # fp32 sums of exact products
    ref = orr.router_fwd(X, Wr, k, logits=lg)
    assert np.array_equal(idx.cpu().numpy(), ref["idx"])
    assert np.max(np.abs(host(gates) - ref["gates"])) <= 1e-5
    dX, dWr = t.empty((T, h), device="cuda").bfloat16(), t.empty((E, h), device="cuda")
    mf.memfine_router_bwd(s, Xd, Wd, idx, gates, t.from_numpy(dg).cuda(), dX, dWr)
    R = orr.router_bwd(X, Wr, ref["idx"], lg, dg)
    assert relerr(host(dX), R["dX"]) <= TOL["bf16"]
    assert relerr(host(dWr), R["dWr"]) <= TOL["bf16"]


# Narrow routers on both sides of one workgroup of 32 tokens per CU, where the
# operands' depth in flight changes: the same sums.
@pytest.mark.parametrize("E,h", [(33, 64), (64, 448)])
def test_router_narrow_depth(mf, E, h):
    t = torch()
    T = 32 * t.cuda.get_device_properties(0).multi_processor_count
    log(f"router narrow depth E={E} h={h}")
    gen = t.Generator(device="cuda")
    gen.manual_seed(E)
    X = t.randn((T + 1, h), generator=gen, device="cuda").bfloat16()
    Wr = (t.randn((E, h), generator=gen, device="cuda") / 8).bfloat16()
    out = []
    for n in (T, T + 1):
        idx, gates = t.empty((n, 4), dtype=t.int32, device="cuda"), t.empty((n, 4), device="cuda")
        logits = t.empty((n, E), device="cuda")
        mf.memfine_router_fwd(mf.make_shape(n, h, 64, E, 4, mf.BF16), X[:n], Wr, idx, gates, logits)
        assert relerr(host(logits), (X[:n].double() @ Wr.double().T).cpu().numpy()) <= 1e-5
        out.append((idx[:T], gates[:T], logits[:T]))
    assert all(t.equal(a, b) for a, b in zip(*out))


# The top-k of wide routers on logits that tie (+0 and -0 among them), are
# infinite, or are not numbers (never selected): X is one-hot, so a token's
# logits are a column of Wr.
@pytest.mark.parametrize("E", [96, 100, 256])
def test_router_topk_special_logits(mf, E):
    t = torch()
    h, k = 64, 6
    log(f"router top-k special E={E}")
    rng = np.random.default_rng(E)
    cols = rng.integers(-2, 3, size=(h, E)).astype(np.float32)   # many ties
    cols[cols == 0] = np.where(rng.random((cols == 0).sum()) < 0.5, 0.0, -0.0)
    Wr = np.ascontiguousarray(cols.T)
    X = np.eye(h, dtype=np.float32)
    s = mf.make_shape(h, h, 64, E, k, mf.BF16)
    idx = t.empty((h, k), dtype=t.int32, device="cuda")
    gates, logits = t.empty((h, k), device="cuda"), t.empty((h, E), device="cuda")
    mf.memfine_router_fwd(s, t.from_numpy(X).cuda().bfloat16(),
                          t.from_numpy(Wr).cuda().bfloat16(), idx, gates, logits)
    lg, sel = host(logits).astype(np.float64), idx.cpu().numpy()
    assert np.array_equal(lg, cols.astype(np.float64))
    order = np.lexsort((np.broadcast_to(np.arange(E), lg.shape), -lg), axis=-1)[:, :k]
    assert np.array_equal(sel, order)
    # expert 1 at +inf, 2 not a number, 5 at -inf, the others falling with the id
    X2 = np.ones((4, h), np.float32)
    Wr2 = np.zeros((E, h), np.float32)
    Wr2[:, 0] = -np.arange(E) / 8.0
    Wr2[2, 1] = np.nan
    Wr2[5, 1] = -np.inf
    Wr2[1, 1] = np.inf
    s = mf.make_shape(4, h, 64, E, k, mf.BF16)
    idx, gates = t.empty((4, k), dtype=t.int32, device="cuda"), t.empty((4, k), device="cuda")
    mf.memfine_router_fwd(s, t.from_numpy(X2).cuda().bfloat16(),
                          t.from_numpy(Wr2).cuda().bfloat16(), idx, gates)
    assert idx.cpu().numpy().tolist() == [[1, 0, 3, 4, 6, 7]] * 4


# Router dX with the rows in registers (from 8192 tokens): a last row block of 1,
# 244 and 255 rows, half a column block, a result larger than the cache, every
# reduction length, adding to dX; at h = 4160 a workgroup walks four or more column
# blocks through its two LDS stages (all 33 at 33000 tokens, where the stores are
# streamed); the bits of the grouped GEMM (forced by a tile option).
@pytest.mark.parametrize("T,E,h", [(8191, 256, 64), (8192, 64, 64), (8193, 128, 192),
                                   (8436, 192, 320), (8447, 256, 448), (300001, 64, 512),
                                   (8193, 64, 4160), (8193, 128, 4160), (8193, 192, 4160),
                                   (8193, 256, 4160), (33000, 64, 4160)])
@pytest.mark.parametrize("accumulate", [False, True])
def test_router_dx_rows(mf, T, E, h, accumulate):
    t = torch()
    k = 4
    log(f"router dX rows T={T} E={E} h={h} accumulate={accumulate}")
    gen = t.Generator(device="cuda")
    gen.manual_seed(T + E)
    X = t.randn((T, h), generator=gen, device="cuda").bfloat16()
    Wr = (t.randn((E, h), generator=gen, device="cuda") / 8).bfloat16()
    idx = t.randn((T, E), generator=gen, device="cuda").topk(k, dim=1).indices.int().contiguous()
    gates = t.softmax(t.randn((T, k), generator=gen, device="cuda"), 1)
    dg = t.randn((T, k), generator=gen, device="cuda")
    old = t.randn((T, h), generator=gen, device="cuda").bfloat16()
    s = mf.make_shape(T, h, 64, E, k, mf.BF16)
    got = []
    for tile in (mf.TILE_AUTO, mf.TILE_256):
        dX = old.clone() if accumulate else t.full((T, h), float("nan"), device="cuda").bfloat16()
        dWr = t.empty((E, h), device="cuda")
        try:
            mf.memfine_set_launch_options(tile=tile)
            mf.memfine_router_bwd(s, X, Wr, idx, gates, dg, dX, dWr, accumulate_dX=accumulate)
        finally:
            mf.memfine_set_launch_options()
        got.append(dX)
    assert t.equal(got[0], got[1])
    if T > 100000:
        return
    g, d = gates.cpu().double(), dg.cpu().double()
    dz = g * (d - (g * d).sum(1, keepdim=True))
    D = t.zeros((T, E), dtype=t.float64).scatter_add_(1, idx.cpu().long(), dz)
    ref = D @ Wr.cpu().double() + (old.cpu().double() if accumulate else 0)
    assert relerr(host(got[0]), ref.numpy()) <= TOL["bf16"]


# Router with more bytes of dz rows (E > h) or logits than 32-bit offsets reach:
# T rows of 256 values, h = 64.  Rows sampled at the ends, around 2^31 and 2^32
# bytes and at random against float64; bf16 dX as the grouped GEMM (forced by a
# tile option) against the register-row kernel bit for bit.
@pytest.mark.parametrize("T,dtype,accumulate", [(2097300, "f32", False), (4194400, "f32", True),
                                                (4194400, "bf16", False), (8388650, "bf16", True)])
def test_router_rows_past_32_bit_offsets(mf, T, dtype, accumulate):
    t = torch()
    E, h, k = 256, 64, 2
    log(f"router rows past 32-bit offsets T={T} {dtype} accumulate={accumulate}")
    dt = t.bfloat16 if dtype == "bf16" else t.float32
    gen = t.Generator(device="cuda")
    gen.manual_seed(T)
    X = t.randn((T, h), generator=gen, device="cuda").to(dt)
    Wr = (t.randn((E, h), generator=gen, device="cuda") / 8).to(dt)
    dg = t.randn((T, k), generator=gen, device="cuda")
    old = t.randn((T, h), generator=gen, device="cuda").to(dt)
    s = mf.make_shape(T, h, 64, E, k, mf.BF16 if dtype == "bf16" else mf.F32)
    idx = t.full((T, k), -1, dtype=t.int32, device="cuda")
    gates, logits = t.empty((T, k), device="cuda"), t.full((T, E), float("nan"), device="cuda")
    mf.memfine_router_fwd(s, X, Wr, idx, gates, logits)
    per = 256 * (2 if dtype == "bf16" else 4)
    rows = t.cat([t.arange(300), t.arange(T - 300, T), t.randint(0, T, (2000,))] +
                 [t.arange(b // per - 300, min(b // per + 300, T)) for b in (1 << 31, 1 << 32)
                  if b // per - 300 < T]).cuda()
    z = X[rows].double() @ Wr.double().T
    assert relerr(logits[rows].double().cpu().numpy(), z.cpu().numpy()) <= 1e-5
    top = logits[rows].topk(k, dim=1)
    assert t.equal(logits[rows].gather(1, idx[rows].long()), top.values)
    del logits
    got = []
    for tile in (mf.TILE_AUTO, mf.TILE_256) if dtype == "bf16" else (mf.TILE_AUTO,):
        dX = old.clone() if accumulate else t.full((T, h), float("nan"), device="cuda").to(dt)
        dWr = t.full((E, h), float("nan"), device="cuda")
        try:
            mf.memfine_set_launch_options(tile=tile)
            mf.memfine_router_bwd(s, X, Wr, idx, gates, dg, dX, dWr, accumulate_dX=accumulate)
        finally:
            mf.memfine_set_launch_options()
        got.append(dX)
    assert all(t.equal(got[0], g) for g in got)
    g64, d64 = gates.double(), dg.double()
    dz = g64 * (d64 - (g64 * d64).sum(1, keepdim=True))
    D = t.zeros((len(rows), E), dtype=t.float64, device="cuda")
    D.scatter_add_(1, idx[rows].long(), dz[rows])
    ref = D @ Wr.double() + (old[rows].double() if accumulate else 0)
    assert relerr(got[0][rows].double().cpu().numpy(), ref.cpu().numpy()) <= TOL[dtype]
    ref = t.zeros((E, h), dtype=t.float64, device="cuda")
    for j in range(k):
        ref.index_add_(0, idx[:, j].long(), dz[:, j:j + 1] * X.double())
    assert relerr(host(dWr), ref.cpu().numpy()) <= TOL[dtype]


# An expert whose tile of 256 rows spans more than 2^31 bytes: of dW1 (256 rows of
# 2228224), of dW2 if all of its rows were there (64), of du (more than 240 of 300
# rows of 4456448 bf16 values), whatever the launch options; against float64 on the GPU.
@pytest.mark.parametrize("T,h,F,opts", [
    (5, 64, 2228224, {}), (5, 2228224, 128, {}), (300, 64, 2228224, {}),
    (300, 64, 2228224, {"tile": 2}), (300, 64, 2228224, {"pair": True})])
@pytest.mark.parametrize("accumulate", [False, True])
def test_very_long_rows(mf, T, h, F, opts, accumulate):
    t = torch()
    log(f"long rows T={T} h={h} F={F} {opts} accumulate={accumulate}")
    gen = t.Generator(device="cuda")
    gen.manual_seed(h)

    def rand(*shape, scale=1.0, dtype=t.bfloat16):
        return (t.randn(shape, generator=gen, device="cuda") * scale).to(dtype)
    X, dY = rand(T, h), rand(T, h)
    W1, W2 = rand(1, 2 * F, h, scale=h ** -0.5), rand(1, h, F, scale=h ** -0.5)
    idx = t.zeros((T, 1), dtype=t.int32, device="cuda")
    gates = t.rand((T, 1), generator=gen, device="cuda") + 0.5
    dX, dg = t.full((T, h), float("nan"), device="cuda").bfloat16(), t.empty((T, 1), device="cuda")
    if accumulate:
        dW = [rand(*W.shape, dtype=t.float32) for W in (W1, W2)]
    else:
        dW = [t.full(W.shape, float("nan"), device="cuda") for W in (W1, W2)]
    old = [x[0].clone() if accumulate else 0 for x in dW]
    try:
        mf.memfine_set_launch_options(**opts)
        mf.memfine_moe_bwd(mf.make_shape(T, h, F, 1, 1, mf.BF16), 1, X, idx, gates, W1, W2, dY, dX,
                           *dW, dg, accumulate_dW=accumulate)
    finally:
        mf.memfine_set_launch_options()
    x, y, g = X.double(), dY.double(), gates.double()
    u = x @ W1[0].double().T
    gate, up = u[:, :F], u[:, F:]
    s = t.sigmoid(gate)
    a, dA = gate * s * up, y @ W2[0].double()
    du = t.cat((g * dA * up * s * (1 + gate * (1 - s)), g * dA * gate * s), 1)

    def check(name, got, ref):
        err = float((got.double() - ref).abs().max() / ref.abs().max())
        log(f"  {name} {err:.2e}")
        assert err <= TOL["bf16"], name
    check("dgates", dg, (dA * a).sum(1, keepdim=True))
    check("dX", dX, du @ W1[0].double())
    check("dW2", dW[1][0], (g * y).T @ a + old[1])
    check("dW1", dW[0][0], du.T @ x + old[0])


# Router dz rows where dX is a product from them (E a multiple of 64): with Wr the
# identity dX is dz itself, so the bits are those of fp32 arithmetic with the sum
# over the slots as a pairwise tree of 16 - in fp32, with up to 64 KB of rows per
# workgroup, and rounded to bf16, below and from 8192 tokens.  Some ids are out
# of range (dropped) or repeated (added, in slot order).
@pytest.mark.parametrize("T,E,k,dtype", [(70, 64, 5, "f32"), (1, 128, 16, "f32"),
                                         (333, 192, 8, "f32"), (8200, 256, 8, "f32"),
                                         (129, 256, 16, "bf16"), (8200, 128, 3, "bf16")])
@pytest.mark.parametrize("accumulate", [False, True])
def test_router_dz_rows(mf, T, E, k, dtype, accumulate):
    t = torch()
    log(f"router dz rows T={T} E={E} k={k} {dtype} accumulate={accumulate}")
    rng = np.random.default_rng(T + E)
    f = np.float32
    idx = rng.permuted(np.tile(np.arange(E), (T, 1)), axis=1)[:, :k].astype(np.int32)
    idx[::3, 0] = np.array([E, -1, E + 7])[np.arange(T)[::3] % 3]
    idx[1::4, -1] = idx[1::4, 1]
    g = rng.random((T, k)).astype(f)
    d = rng.standard_normal((T, k)).astype(f)
    old = mw.round_to_bf16(rng.standard_normal((T, E))).astype(f)
    ok = (idx >= 0) & (idx < E)
    gk, dk = (np.zeros((T, 16), f) for _ in range(2))
    gk[:, :k], dk[:, :k] = np.where(ok, g, 0), np.where(ok, d, 0)
    s = gk * dk
    while s.shape[1] > 1:
        s = s[:, 0::2] + s[:, 1::2]
    dz = gk * (dk - s)
    ref = np.zeros((T, E), f)
    for j in range(k):
        rows = np.flatnonzero(ok[:, j])
        ref[rows, idx[rows, j]] += dz[rows, j]
    rnd = (lambda x: x) if dtype == "f32" else (lambda x: mw.round_to_bf16(x).astype(f))
    ref = rnd(ref)
    if accumulate:
        ref = rnd(old + ref)
    dt = t.float32 if dtype == "f32" else t.bfloat16
    dev = [t.from_numpy(a).cuda() for a in (idx, g, d)]
    Wr = t.eye(E, device="cuda", dtype=dt)
    X = t.from_numpy(old).cuda().to(dt)
    dX = X.clone() if accumulate else t.full((T, E), float("nan"), device="cuda").to(dt)
    dWr = t.empty((E, E), device="cuda")
    shape = mf.make_shape(T, E, 64, E, k, mf.F32 if dtype == "f32" else mf.BF16)
    mf.memfine_router_bwd(shape, X, Wr, *dev, dX, dWr, accumulate_dX=accumulate)
    assert np.array_equal(host(dX), ref)
