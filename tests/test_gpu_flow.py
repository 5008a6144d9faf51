"""The flowing GEMM kernel, every tile and mode, forced: ragged rows and columns, the fewest stages a tile takes, one tile per
workgroup and several, odd output views.  Reference: the oracle on sampled rows, and the DMA kernel's result everywhere.  Both
kernels add exact products in single precision; they differ in the order of at most 1 + K / 64 partial sums, so the
whole results agree to a few 2^-24 of the largest output (1e-5 is used)."""
import numpy as np
import pytest
import torch

import oracle
import workloads as wl

pytestmark = pytest.mark.gpu
TOL = 1e-3
TILES = {0: (128, 256, 3), 1: (128, 192, 3), 2: (128, 128, 4), 3: (64, 128, 4)}  # id: rows, columns, stages of lead


@pytest.fixture(scope="module")
def osc():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2604_12782_amd as m
    m.lib()
    return m


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def problem(osc, mode, M, N, K, r, seed):
    """(call(y_dtype, out), reference(rows))"""
    W = wl.weights(seed + 1, N, K)
    if mode == "dual":
        X, table = wl.activations_persistent(seed, M, K, r) if r else (wl.activations_diffuse(seed, M, K), None)
        oidx = oracle.table_to_index(table) if r else np.zeros(0, np.int32)
        d = dev(oidx) if r else None
        q, Wp = osc.osc_quantize_act(dev(X), d), osc.osc_pack_weight(dev(W), d)

        def ref(rows):
            a = oracle.quantize_mxfp4_osc(X[rows], oidx, ldb=q[2].shape[1] if r else 0)
            w = oracle.quantize_mxfp4_osc(W)
            return oracle.dual_gemm(a[0], a[1], a[2] if r else None, w[0], w[1], oracle.gather_wl(W, oidx))
        return lambda ydt, out=None: osc.osc_dual_gemm(*q, Wp, N, K, len(oidx), ydt, out=out), ref
    X = wl.activations_diffuse(seed, M, K)
    if mode == "fp8":
        q, Wp = osc.osc_quantize_act(dev(X), None, osc.OSC_FMT_FP8_E4M3_TOKEN), osc.osc_pack_weight_fp8(dev(W))
        return (lambda ydt, out=None: osc.osc_fp8_gemm(*q, Wp, N, K, y_dtype=ydt, out=out),
                lambda rows: oracle.fp8_gemm(*oracle.quantize_fp8_rows(X[rows]), *oracle.quantize_fp8_rows(W)))
    q, Wp = osc.osc_quantize_act(dev(X), None, osc.OSC_FMT_MXFP8), osc.osc_pack_weight_mxfp8(dev(W))
    return (lambda ydt, out=None: osc.osc_mxfp8_gemm(*q, Wp, N, K, y_dtype=ydt, out=out),
            lambda rows: oracle.mxfp8_gemm(*oracle.quantize_mxfp8(X[rows]), *oracle.quantize_mxfp8(W)))


def check(osc, tuning, tile, mode, M, N, K, r, seed):
    call, ref = problem(osc, mode, M, N, K, r, seed)
    bm = TILES[tile][0]
    rows = np.unique(np.clip(np.concatenate([np.arange(0, M, max(1, M // 5)), [bm - 1, bm, M - 1]]), 0, M - 1))
    tuning.gemm(f"{tile},7")
    Y, Yb = call(osc.OSC_DT_F32), call(osc.OSC_DT_BF16)
    wide = torch.full((M, N + 24), 7.0, dtype=torch.bfloat16, device="cuda")  # rows that keep 16-byte alignment, and a view that does not
    call(osc.OSC_DT_BF16, wide[:, 8:8 + N])
    call(osc.OSC_DT_BF16, Yb)
    odd = torch.full((M, N + 3), 7.0, dtype=torch.bfloat16, device="cuda")
    call(osc.OSC_DT_BF16, odd[:, 1:1 + N])
    assert osc.osc_tuning_last_gemm() == (7, tile)
    tuning.gemm("1,1")
    Y0 = call(osc.OSC_DT_F32)
    assert osc.osc_tuning_last_gemm() == (1, 1)
    want = ref(rows)
    got = Y[torch.from_numpy(rows).cuda()].cpu().numpy().astype(np.float64)
    assert np.abs(got - want).max() <= TOL * np.abs(want).max()
    assert float((Y - Y0).abs().max()) <= 1e-5 * float(Y0.abs().max())
    assert torch.equal(Yb, Y.to(torch.bfloat16))  # the same sums, rounded once
    assert torch.equal(wide[:, 8:8 + N], Yb) and bool((wide[:, :8] == 7).all()) and bool((wide[:, 8 + N:] == 7).all())
    assert torch.equal(odd[:, 1:1 + N], Yb) and bool((odd[:, :1] == 7).all()) and bool((odd[:, 1 + N:] == 7).all())


@pytest.mark.parametrize("mode", ["dual", "fp8", "mx8"])
@pytest.mark.parametrize("tile", sorted(TILES))
def test_flow_edges(osc, tuning, tile, mode):
    """One ragged tile with the fewest stages, one exact tile, a few ragged ones."""
    bm, bn, lead = TILES[tile]
    k1 = 256 if mode == "dual" else 128
    check(osc, tuning, tile, mode, 1, 8, k1 * (lead + 1), 0, 7600 + tile)
    check(osc, tuning, tile, mode, bm, bn, k1 * (lead + 2), 1 if mode == "dual" else 0, 7610 + tile)
    check(osc, tuning, tile, mode, 2 * bm + 5, bn + 13, 2560, 4 if mode == "dual" else 0, 7620 + tile)


@pytest.mark.parametrize("mode", ["dual", "fp8", "mx8"])
@pytest.mark.parametrize("tile", sorted(TILES))
def test_flow_several_tiles_per_workgroup(osc, tuning, tile, mode):
    """More tiles than CUs, a number that the eight dies do not divide: the load cursor crosses into the next tile while the
    current one is computed, both copies of the FP8 tile scales are used, and some workgroups have a tile more than others."""
    bm, bn, lead = TILES[tile]
    N = bn * 9 - 40
    M = bm * 31 - 17  # 279 tiles
    check(osc, tuning, tile, mode, M, N, 256 * (lead + 1) if mode == "dual" else 128 * (lead + 3), 2 if mode == "dual" else 0, 7700 + tile)


GUARD = 256  # rows behind a view: as many as the tallest tile


def into_views(call, osc, M, N, Y, Yb, what, rows=None):
    """The call's results written into views whose rows start at every residue of the store widths (16 bytes fp32, 8 bytes bf16), with
    columns on both sides and rows behind them: the values of a buffer of their own (of the first `rows`), and not a byte beside them."""
    n = M if rows is None else rows
    for dt, ydt, want in ((torch.float32, osc.OSC_DT_F32, Y), (torch.bfloat16, osc.OSC_DT_BF16, Yb)):
        for pad, col0 in ((0, 0), (4, 0), (4, 2), (8, 4), (2, 2), (3, 1), (1, 0)):
            wide = torch.full((M + GUARD, N + pad), 7.0, dtype=dt, device="cuda")
            call(ydt, wide[:M, col0:col0 + N])
            assert torch.equal(wide[:n, col0:col0 + N], want[:n]), (what, dt, pad, col0)
            wide[:n, col0:col0 + N] = 7
            assert bool((wide == 7).all()), (what, dt, pad, col0)


TILED = [(c, m) for c in ("0,7", "1,7", "2,7", "3,7", "4,2", "4,1", "2,1", "1,1") for m in ("dual", "fp8", "mx8")]
TILED += [("2,2", "dual"), ("4,4", "dual"), ("2,0", "dual"), ("1,0", "dual"), ("2,0", "fp8"), ("1,0", "fp8")]  # (not built for the others)


@pytest.mark.parametrize("cfg,mode", TILED)
def test_output_views(osc, tuning, cfg, mode):
    """The epilogue that all tiled kernels share, into views, for tiles inside the result, tiles with rows past it and tiles with columns
    past it; the values against the oracle."""
    tile, kern = map(int, cfg.split(","))
    for M, N in ((256, 512), (131, 512), (131, 395), (70, 1)) if kern != 2 else ((256, 512),):
        call, ref = problem(osc, mode, M, N, 1280, 1 if mode == "dual" else 0, 8100 + M)
        tuning.gemm(cfg)
        Y, Yb = call(osc.OSC_DT_F32), call(osc.OSC_DT_BF16)
        assert osc.osc_tuning_last_gemm() == (kern, tile)
        want = ref(np.arange(M))
        assert np.abs(Y.cpu().numpy().astype(np.float64) - want).max() <= TOL * np.abs(want).max()
        assert torch.equal(Yb, Y.to(torch.bfloat16))
        into_views(call, osc, M, N, Y, Yb, (cfg, mode, M, N))


@pytest.mark.parametrize("cfg", ["0,7", "4,1", "2,1", "1,1", "1,0"])
def test_output_views_of_experts(osc, tuning, cfg):
    """The same for experts, some of them empty, whose last tiles have rows of the next expert behind them, and with offsets that end before
    the output does."""
    sizes, N, K = [70, 0, 1, 129, 60, 0], 395, 1280
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    T, E = int(off[-1]), len(sizes)
    X = wl.activations_diffuse(8200, T, K)
    q, q8 = osc.osc_quantize_act(dev(X)), osc.osc_quantize_act(dev(X), None, osc.OSC_FMT_FP8_E4M3_TOKEN)
    W = [wl.weights(8210 + e, N, K) for e in range(E)]
    Wp, Wp8 = torch.cat([osc.osc_pack_weight(dev(w), None) for w in W]), torch.cat([osc.osc_pack_weight_fp8(dev(w)) for w in W])
    row_map = np.random.default_rng(8201).permutation(T).astype(np.int32)
    calls = {"dual": lambda d_off: lambda ydt, out=None: osc.osc_grouped_dual_gemm(*q, dev(row_map), d_off, T, Wp, N, K, 0, ydt, out=out),
             "fp8": lambda d_off: lambda ydt, out=None: osc.osc_fp8_gemm(*q8, Wp8, N, K, expert_offsets=d_off, y_dtype=ydt, out=out)}
    a, w = oracle.quantize_mxfp4_osc(X), [oracle.quantize_mxfp4_osc(x)[:2] for x in W]
    a8, w8 = oracle.quantize_fp8_rows(X), [oracle.quantize_fp8_rows(x) for x in W]
    refs = {"dual": oracle.grouped_dual_gemm(a[0], a[1], None, row_map, off, np.stack([x[0] for x in w]), np.stack([x[1] for x in w]), None),
            "fp8": oracle.grouped_fp8_gemm(*a8, off, np.stack([x[0] for x in w8]), np.stack([x[1] for x in w8]))}
    tuning.gemm(cfg)
    for name, make in calls.items():
        call = make(dev(off))
        Y, Yb = call(osc.OSC_DT_F32), call(osc.OSC_DT_BF16)
        assert osc.osc_tuning_last_gemm() == tuple(int(x) for x in reversed(cfg.split(","))), name
        assert np.abs(Y.cpu().numpy().astype(np.float64) - refs[name]).max() <= TOL * np.abs(refs[name]).max(), name
        assert torch.equal(Yb, Y.to(torch.bfloat16)), name
        into_views(call, osc, T, N, Y, Yb, (cfg, name))
        into_views(make(dev(np.minimum(off, 150).astype(np.int32))), osc, T, N, Y, Yb, (cfg, name, "short"), 150)


@pytest.mark.parametrize("stages,r", [(2, 0), (2, 1), (3, 4), (4, 0), (4, 2)])
def test_flow_no_more_stages_than_the_lead(osc, tuning, stages, r):
    """Dual path on 64 x 128 tiles, where the load cursor is up to three tiles ahead of the products: one tile, two, and six or seven
    a workgroup.  (Experts of few stages: below.)"""
    tile = 3
    bm, bn, _ = TILES[tile]
    K = 256 * (stages - (1 if r else 0))  # a branch of up to 64 channels is one stage
    check(osc, tuning, tile, "dual", bm - 3, bn, K, r, 8000 + tile)
    check(osc, tuning, tile, "dual", bm * 31, bn * 16 + 8, K, r, 8010 + tile)
    check(osc, tuning, tile, "dual", bm * 180 - 17, bn * 9 - 40, K, r, 8020 + tile)


def test_launcher_choice_agrees(osc, tuning):
    """The launcher's own choice (kernel, tile) over shapes on both sides of its rules, and its result against the DMA kernel."""
    for mode, M, N, K, r, chosen in [("dual", 1000, 1536, 4096, 1, (7, 3)), ("dual", 130, 4096, 1280, 2, (7, 3)), ("fp8", 300, 4104, 2048, 0, (7, 3)),
                                     ("mx8", 700, 1000, 1536, 0, (7, 3)), ("dual", 60, 33000, 1280, 0, (7, 3)), ("fp8", 40, 33000, 640, 0, (7, 3)),
                                     ("mx8", 2100, 2048, 640, 0, (7, 0)), ("dual", 4200, 4096, 1536, 1, (2, 4)),
                                     ("dual", 500, 4096, 768, 2, (7, 3)), ("dual", 1500, 1300, 768, 2, (1, 1)), ("dual", 300, 4096, 768, 0, (1, 1))]:
        call, _ = problem(osc, mode, M, N, K, r, 7800 + M)
        tuning.gemm(None)
        Y = call(osc.OSC_DT_F32)
        assert osc.osc_tuning_last_gemm() == chosen, (mode, M, N, K, r)
        tuning.gemm("1,1")
        Y0 = call(osc.OSC_DT_F32)
        assert float((Y - Y0).abs().max()) <= 1e-5 * float(Y0.abs().max()), (mode, M, N, K, r)


SIZES = [0, 1, 63, 64, 65, 127, 128, 129, 191, 192, 193, 256, 257, 385, 700, 0, 130, 0]


@pytest.mark.parametrize("N,K,K2,r", [(264, 1024, 512, 2), (5000, 1024, 512, 2), (264, 256, 128, 0), (13000, 256, 128, 0), (264, 256, 256, 2), (9000, 512, 256, 0),
                                      (264, 512, 384, 2), (9000, 512, 384, 2)])
def test_flow_experts(osc, tuning, N, K, K2, r):
    """Experts of every size around the tile's borders and the half tile that is skipped, empty ones at the ends: fewer tiles than CUs
    against the oracle; several per workgroup against the DMA kernel; one stage a tile (the row map's entries are needed as soon as
    they have been asked for), two, three and more than the lead.  Rows beyond the offsets stay untouched."""
    E, tokens = len(SIZES), 700
    off = np.concatenate([[0], np.cumsum(SIZES)]).astype(np.int32)
    T = int(off[-1])
    X, table = wl.activations_persistent(7900, tokens, K, r) if r else (wl.activations_diffuse(7900, tokens, K), None)
    oidx = oracle.table_to_index(table) if r else np.zeros(0, np.int32)
    d_oidx = dev(oidx) if r else None
    row_map = wl.rng(7901).integers(0, tokens, T).astype(np.int32)
    X2 = wl.activations_diffuse(7902, T, K2)
    q = osc.osc_quantize_act(dev(X), d_oidx)
    q8, qm = osc.osc_quantize_act(dev(X2), None, osc.OSC_FMT_FP8_E4M3_TOKEN), osc.osc_quantize_act(dev(X2), None, osc.OSC_FMT_MXFP8)
    W, W2 = [wl.weights(7910 + e, N, K) for e in range(E)], [wl.weights(7950 + e, N, K2) for e in range(E)]
    Wp = torch.cat([osc.osc_pack_weight(dev(w), d_oidx) for w in W])
    Wp8, Wpm = torch.cat([osc.osc_pack_weight_fp8(dev(w)) for w in W2]), torch.cat([osc.osc_pack_weight_mxfp8(dev(w)) for w in W2])
    d_off = dev(off)
    calls = {"dual": lambda ydt, out=None: osc.osc_grouped_dual_gemm(*q, dev(row_map), d_off, T, Wp, N, K, len(oidx), ydt, out=out),
             "fp8": lambda ydt, out=None: osc.osc_fp8_gemm(*q8, Wp8, N, K2, expert_offsets=d_off, y_dtype=ydt, out=out),
             "mx8": lambda ydt, out=None: osc.osc_mxfp8_gemm(*qm, Wpm, N, K2, expert_offsets=d_off, y_dtype=ydt, out=out)}
    refs = {}
    if N < 1000:
        a = oracle.quantize_mxfp4_osc(X, oidx, ldb=q[2].shape[1] if r else 0)
        w = [oracle.quantize_mxfp4_osc(x)[:2] for x in W]
        refs["dual"] = oracle.grouped_dual_gemm(a[0], a[1], a[2] if r else None, row_map, off, np.stack([x[0] for x in w]), np.stack([x[1] for x in w]),
                                                np.stack([oracle.gather_wl(x, oidx) for x in W]))
        w = [oracle.quantize_fp8_rows(x) for x in W2]
        refs["fp8"] = oracle.grouped_fp8_gemm(*oracle.quantize_fp8_rows(X2), off, np.stack([x[0] for x in w]), np.stack([x[1] for x in w]))
    for name, call in calls.items():
        tuning.gemm("0,7")
        Y, Yb = call(osc.OSC_DT_F32), call(osc.OSC_DT_BF16)
        assert osc.osc_tuning_last_gemm() == (7, 0), name
        tuning.gemm("1,1")
        Y0 = call(osc.OSC_DT_F32)
        assert osc.osc_tuning_last_gemm() == (1, 1), name
        assert float((Y - Y0).abs().max()) <= 1e-5 * float(Y0.abs().max()), name
        assert torch.equal(Yb, Y.to(torch.bfloat16)), name
        if name in refs:
            assert np.abs(Y.cpu().numpy().astype(np.float64) - refs[name]).max() <= TOL * np.abs(refs[name]).max(), name
    # offsets that end before the output does
    tuning.gemm("0,7")
    short = torch.from_numpy(np.minimum(off, 500)).cuda()
    out = torch.full((T, N), 7.0, dtype=torch.bfloat16, device="cuda")
    osc.osc_fp8_gemm(*q8, Wp8, N, K2, expert_offsets=short, y_dtype=osc.OSC_DT_BF16, out=out)
    assert bool((out[500:] == 7).all()) and not bool((out[:500] == 7).all())


@pytest.mark.parametrize("mode,E,rows,N,K,chosen", [("dual", 128, 270, 1536, 512, (7, 0)), ("fp8", 128, 270, 2048, 384, (7, 0)), ("mx8", 128, 270, 1024, 256, (7, 0)),
                                                    ("fp8", 128, 270, 1024, 128, (7, 0)), ("mx8", 128, 500, 2048, 384, (7, 0)), ("dual", 128, 150, 1536, 512, (1, 4)),
                                                    ("mx8", 64, 130, 2048, 384, (1, 4)), ("dual", 32, 270, 1536, 1024, (7, 0)), ("dual", 8, 160, 1024, 1024, (1, 1)),
                                                    ("mx8", 64, 80, 1024, 768, (1, 2)), ("fp8", 8, 330, 1024, 768, (1, 2)), ("fp8", 64, 160, 1024, 768, (7, 0))])
def test_launcher_choice_for_experts(osc, tuning, mode, E, rows, N, K, chosen):
    """Experts of one to three stages: 256-row tiles where those are ahead, the flowing kernel where they would start a few last rows
    of every expert on a tile of their own.  More stages: small tiles where those of the flowing kernel would leave CUs without
    one.  Same numbers as the DMA kernel's small tiles."""
    g = torch.Generator(device="cuda").manual_seed(8100 + rows)
    draw = lambda hi, *shape: torch.randint(0, hi, shape, dtype=torch.uint8, device="cuda", generator=g)  # noqa: E731
    sizes = torch.bincount(torch.randint(0, E, (E * rows,), device="cuda", generator=g), minlength=E)
    off = torch.cat([torch.zeros(1, dtype=torch.int64, device="cuda"), sizes.cumsum(0)]).to(torch.int32)
    T = E * rows
    if mode == "dual":
        Xq, W = draw(256, T, K // 2), draw(120, E * osc.osc_packed_weight_bytes(N, K, 0))
        Xs = torch.full((osc.osc_act_scale_bytes(T, K),), 127, dtype=torch.uint8, device="cuda")
        call = lambda: osc.osc_grouped_dual_gemm(Xq, Xs, None, None, off, T, W, N, K, 0, osc.OSC_DT_F32)  # noqa: E731
    elif mode == "fp8":
        Xq, Xs, W = draw(120, T, K), torch.ones(T, device="cuda"), draw(60, E * osc.osc_packed_weight_fp8_bytes(N, K))
        call = lambda: osc.osc_fp8_gemm(Xq, Xs, W, N, K, expert_offsets=off, y_dtype=osc.OSC_DT_F32)  # noqa: E731
    else:
        Xq, Xs, W = draw(120, T, K), torch.full((osc.osc_act_scale_bytes(T, K),), 127, dtype=torch.uint8, device="cuda"), draw(120, E * osc.osc_packed_weight_mxfp8_bytes(N, K))
        call = lambda: osc.osc_mxfp8_gemm(Xq, Xs, W, N, K, expert_offsets=off, y_dtype=osc.OSC_DT_F32)  # noqa: E731
    Y = call()
    assert osc.osc_tuning_last_gemm() == chosen
    tuning.gemm("1,1")
    Y0 = call()
    assert osc.osc_tuning_last_gemm() == (1, 1)
    rows_max = Y0.abs().amax(dim=1, keepdim=True)  # scale bytes drawn freely differ by many powers of two from channel to channel
    assert bool(torch.isfinite(Y).all()) and bool(((Y - Y0).abs() <= 1e-5 * rows_max).all())
