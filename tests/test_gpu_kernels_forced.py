"""Every GEMM kernel template on shapes it would not be chosen for: the launcher's tuning knobs
(include/osc_tuning.h) force the tile size and the kernel, the results must still meet the GEMM tolerance.  Also outputs
written into wider buffers (ldy > N) and through the unaligned bf16 store path."""
import numpy as np
import pytest
import torch

import oracle
import workloads as wl

pytestmark = pytest.mark.gpu
TOL = 1e-3


@pytest.fixture(scope="module")
def osc():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2604_12782_amd as m
    m.lib()
    return m


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def close(Y, ref, what, bf16=False):
    Y = Y.float().cpu().numpy().astype(np.float64)
    slack = TOL * np.abs(ref).max() + (2.0 ** -8 * np.abs(ref) if bf16 else 0.0)
    assert np.isfinite(Y).all() and (np.abs(Y - ref) <= slack).all(), what


# tile rows / 64, kernel id: 0 staged, 1 DMA (eight wavefronts at 256 rows), 2 persistent, 3 skinny,
# 4 ring (wavefront groups in anti-phase), 5 ring (in phase)
FORCED = ["4,1", "2,1", "1,1", "1,0", "2,0", "4,2", "2,2", "1,3", "4,4", "4,5"]  # (6, streaming: test_gpu_stream.py)


@pytest.mark.parametrize("cfg", FORCED)
@pytest.mark.parametrize("M,N,K,r", [(300, 200, 1024, 2), (513, 520, 512, 1), (256, 512, 768, 0), (70, 1000, 256, 4)])
def test_dual_forced(osc, tuning, cfg, M, N, K, r):
    tuning.gemm(cfg)
    X, table = wl.activations_persistent(7000 + M, M, K, r)
    W = wl.weights(7100 + N, N, K)
    oidx = oracle.table_to_index(table) if r else np.zeros(0, np.int32)
    d_oidx = dev(oidx) if r else None
    Xq, Xs, B = osc.osc_quantize_act(dev(X), d_oidx)
    Wp = osc.osc_pack_weight(dev(W), d_oidx)
    rq, rs, rb = oracle.quantize_mxfp4_osc(X, oidx, ldb=B.shape[1] if B is not None else 0)
    wq, ws, _ = oracle.quantize_mxfp4_osc(W)
    ref = oracle.dual_gemm(rq, rs, rb if r else None, wq, ws, oracle.gather_wl(W, oidx))
    for ydt, bf in ((osc.OSC_DT_F32, False), (osc.OSC_DT_BF16, True)):
        Y = osc.osc_dual_gemm(Xq, Xs, B, Wp, N, K, len(oidx), ydt)
        close(Y, ref, f"{cfg} {M}x{N}x{K} r={r} bf16={bf}", bf)


@pytest.mark.parametrize("M,N,K,r", [(300, 200, 1024, 2), (200, 300, 1280, 2), (64, 128, 2048, 1), (130, 260, 4096, 4),
                                     (513, 520, 1024, 0), (1, 40, 2304, 3), (2048, 1024, 4096, 2)])
@pytest.mark.parametrize("tile", ["1,1", "2,1"])
def test_dual_small_tiles(osc, tuning, tile, M, N, K, r):
    """64 x 128 and 128 x 128 tiles of the DMA kernel: even and odd numbers of stages, a branch of one to eight stages, ragged
    tiles in both directions."""
    tuning.gemm(tile)
    X, table = wl.activations_persistent(7060 + M, M, K, r) if r else (wl.activations_diffuse(7060 + M, M, K), None)
    W = wl.weights(7160 + N, N, K)
    oidx = oracle.table_to_index(table) if r else np.zeros(0, np.int32)
    d_oidx = dev(oidx) if r else None
    Xq, Xs, B = osc.osc_quantize_act(dev(X), d_oidx)
    Wp = osc.osc_pack_weight(dev(W), d_oidx)
    rows = np.arange(M) if M <= 600 else np.unique(np.concatenate([np.arange(0, M, 61), [63, 64, M - 1]]))
    rq, rs, rb = oracle.quantize_mxfp4_osc(X[rows], oidx, ldb=B.shape[1] if B is not None else 0)
    wq, ws, _ = oracle.quantize_mxfp4_osc(W)
    ref = oracle.dual_gemm(rq, rs, rb if r else None, wq, ws, oracle.gather_wl(W, oidx))
    sel = torch.from_numpy(rows).cuda()
    for ydt, bf in ((osc.OSC_DT_F32, False), (osc.OSC_DT_BF16, True)):
        Y = osc.osc_dual_gemm(Xq, Xs, B, Wp, N, K, len(oidx), ydt)
        assert osc.osc_tuning_last_gemm() == (1, int(tile[0]))
        close(Y[sel], ref, f"{tile} {M}x{N}x{K} r={r} bf16={bf}", bf)


@pytest.mark.parametrize("M,N,K", [(300, 200, 1024), (200, 300, 640), (64, 128, 2048), (513, 520, 896), (2048, 1024, 4096)])
@pytest.mark.parametrize("tile", ["1,1", "2,1"])
def test_fp8_small_tiles(osc, tuning, tile, M, N, K):
    """The per-token FP8 GEMM on 64 x 128 and 128 x 128 tiles of the DMA kernel: even and odd stage counts."""
    tuning.gemm(tile)
    X = wl.activations_diffuse(7250 + M, M, K)
    W = wl.weights(7251 + N, N, K)
    X8, xs = osc.osc_quantize_act(dev(X), None, osc.OSC_FMT_FP8_E4M3_TOKEN)
    rows = np.arange(M) if M <= 600 else np.unique(np.concatenate([np.arange(0, M, 61), [63, 64, M - 1]]))
    r8, rs = oracle.quantize_fp8_rows(X[rows])
    w8, ws = oracle.quantize_fp8_rows(W)
    sel = torch.from_numpy(rows).cuda()
    for ydt, bf in ((osc.OSC_DT_F32, False), (osc.OSC_DT_BF16, True)):
        Y = osc.osc_fp8_gemm(X8, xs, osc.osc_pack_weight_fp8(dev(W)), N, K, y_dtype=ydt)
        assert osc.osc_tuning_last_gemm() == (1, int(tile[0]))
        close(Y[sel], oracle.fp8_gemm(r8, rs, w8, ws), f"fp8 {tile} {M}x{N}x{K} bf16={bf}", bf)


def test_knobs_without_effect(osc, tuning):
    """The knobs that are accepted for kernels that are gone leave the choice and every bit of the results alone."""
    M, N, K = 300, 264, 1024
    X, W = dev(wl.activations_diffuse(7260, M, K)), dev(wl.weights(7261, N, K))
    d_oidx = torch.arange(0, K, 32, dtype=torch.int32, device="cuda")
    off = torch.tensor([0, 130, 130, M], dtype=torch.int32, device="cuda")
    rows = torch.arange(M, dtype=torch.int32, device="cuda")
    q, Wp = osc.osc_quantize_act(X, d_oidx), osc.osc_pack_weight(W, d_oidx)
    q8, W8 = osc.osc_quantize_act(X, None, osc.OSC_FMT_FP8_E4M3_TOKEN), osc.osc_pack_weight_fp8(W)
    calls = [lambda: osc.osc_dual_gemm(*q, Wp, N, K, K // 32), lambda: osc.osc_fp8_gemm(*q8, W8, N, K),
             lambda: osc.osc_grouped_dual_gemm(*q, rows, off, M, Wp.repeat(3), N, K, K // 32),
             lambda: osc.osc_fp8_gemm(*q8, W8.repeat(3), N, K, expert_offsets=off),
             lambda: osc.osc_swiglu_quantize_act(X, X)[0], lambda: osc.osc_swiglu_quantize_act_fp8(X, X)[0]]
    for call in calls:
        want, kernel = call(), osc.osc_tuning_last_gemm()
        for knob in (osc.OSC_TUNE_GROUPED_ONE_TILE, osc.OSC_TUNE_SWIGLU_TABLE, osc.OSC_TUNE_GEMM_KSPLIT):
            for value in (0, 1):
                osc.osc_tuning_set(knob, value)
                assert torch.equal(call(), want) and osc.osc_tuning_last_gemm() == kernel
            osc.osc_tuning_set(knob, -1)


@pytest.mark.parametrize("M,N,K", [(256, 512, 768), (300, 256, 384), (4392, 4096, 384), (2560, 7168, 640)])
def test_fp8_persistent_pipeline(osc, tuning, M, N, K):
    """The per-token FP8 GEMM (and, below, the MXFP8 GEMM) on the persistent kernel (forced; the launcher takes it from 257 tiles of 256 x 256 on):
    one tile, a ragged tail of rows (handled by a second launch), more tiles than workgroups (so that a workgroup
    walks several tiles and both copies of the tile scales in LDS are used), three (the minimum) and five stages."""
    tuning.gemm("4,2")
    X = wl.activations_diffuse(7300 + M, M, K)
    W = wl.weights(7301 + N, N, K)
    X8, xs = osc.osc_quantize_act(dev(X), None, osc.OSC_FMT_FP8_E4M3_TOKEN)
    rows = np.arange(M) if M <= 600 else np.unique(np.concatenate([np.arange(0, M, 37), [255, 256, 257, M - 41, M - 1]]))
    r8, rs = oracle.quantize_fp8_rows(X[rows])
    w8, ws = oracle.quantize_fp8_rows(W)
    ref = oracle.fp8_gemm(r8, rs, w8, ws)
    sel = torch.from_numpy(rows).cuda()
    Wp = osc.osc_pack_weight_fp8(dev(W))
    for ydt, bf in ((osc.OSC_DT_F32, False), (osc.OSC_DT_BF16, True)):
        Y = osc.osc_fp8_gemm(X8, xs, Wp, N, K, y_dtype=ydt)
        close(Y[sel], ref, f"fp8 persistent {M}x{N}x{K} bf16={bf}", bf)
    if M <= 600:
        # wide, shifted and odd output views: the 16-byte, 8-byte and element store paths of the epilogue
        for dt, ydt, bf in ((torch.float32, osc.OSC_DT_F32, False), (torch.bfloat16, osc.OSC_DT_BF16, True)):
            for width, col0 in ((N + 64, 0), (N + 64, 4), (N + 7, 3)):
                wide = torch.full((M, width), 7.0, dtype=dt, device="cuda")
                view = wide[:, col0:col0 + N]
                osc.osc_fp8_gemm(X8, xs, Wp, N, K, y_dtype=ydt, out=view)
                close(view, ref, f"fp8 persistent ldy={width} col0={col0} bf16={bf}", bf)
                assert (torch.cat([wide[:, :col0], wide[:, col0 + N:]], dim=1) == 7.0).all(), "wrote outside the output view"
    # every element against the DMA kernel (same products, same order inside a stage)
    Y2 = osc.osc_fp8_gemm(X8, xs, Wp, N, K)
    tuning.gemm("4,1")
    Y1 = osc.osc_fp8_gemm(X8, xs, Wp, N, K)
    assert float((Y1 - Y2).abs().max()) <= 1e-5 * float(Y1.abs().max())
    # the MXFP8 form of the same kernel: block scales travel with the stages
    tuning.gemm("4,2")
    Xm, Xms = osc.osc_quantize_act(dev(X), None, osc.OSC_FMT_MXFP8)
    q, sc = oracle.quantize_mxfp8(X[rows])
    wq, wsc = oracle.quantize_mxfp8(W)
    refm = oracle.mxfp8_gemm(q, sc, wq, wsc)
    Wm = osc.osc_pack_weight_mxfp8(dev(W))
    for ydt, bf in ((osc.OSC_DT_F32, False), (osc.OSC_DT_BF16, True)):
        Ym = osc.osc_mxfp8_gemm(Xm, Xms, Wm, N, K, y_dtype=ydt)
        close(Ym[sel], refm, f"mxfp8 persistent {M}x{N}x{K} bf16={bf}", bf)
    Y2 = osc.osc_mxfp8_gemm(Xm, Xms, Wm, N, K)
    tuning.gemm("4,1")
    Y1 = osc.osc_mxfp8_gemm(Xm, Xms, Wm, N, K)
    assert float((Y1 - Y2).abs().max()) <= 1e-5 * float(Y1.abs().max())


@pytest.mark.parametrize("cfg", ["1,0", "2,0"])
@pytest.mark.parametrize("M,N,K,r", [(70, 1000, 96, 2), (300, 200, 2080, 1), (513, 520, 1056, 4), (64, 130, 32, 0)])
def test_staged_rows_that_are_not_whole_lines(osc, tuning, cfg, M, N, K, r):
    """The staged kernel with rows (codes, and with ldb = K_o rounded up to 8 the branch) that end inside a 64-byte step, whose
    missing pieces come from the block of zeros: dual path, and per-token FP8 with K / 2 channels rounded to 16."""
    tuning.gemm(cfg)
    X, table = wl.activations_persistent(7700 + M, M, K, r) if r else (wl.activations_diffuse(7700 + M, M, K), None)
    W = wl.weights(7710 + N, N, K)
    oidx = oracle.table_to_index(table) if r else np.zeros(0, np.int32)
    d_oidx = dev(oidx) if r else None
    Wp = osc.osc_pack_weight(dev(W), d_oidx)
    wq, ws, _ = oracle.quantize_mxfp4_osc(W)
    for ldb in ((len(oidx) + 63) // 64 * 64, (len(oidx) + 7) // 8 * 8):
        Xq, Xs, B = osc.osc_quantize_act(dev(X), d_oidx, ldb=ldb)
        rq, rs, rb = oracle.quantize_mxfp4_osc(X, oidx, ldb=ldb)
        ref = oracle.dual_gemm(rq, rs, rb if r else None, wq, ws, oracle.gather_wl(W, oidx))
        for ydt, bf in ((osc.OSC_DT_F32, False), (osc.OSC_DT_BF16, True)):
            close(osc.osc_dual_gemm(Xq, Xs, B, Wp, N, K, len(oidx), ydt), ref, f"staged {cfg} {M}x{N}x{K} ldb={ldb} bf16={bf}", bf)
    K8 = K // 2 // 16 * 16
    X8 = wl.activations_diffuse(7720 + M, M, K8)
    W8 = wl.weights(7730 + N, N, K8)
    q8, s8 = osc.osc_quantize_act(dev(X8), None, osc.OSC_FMT_FP8_E4M3_TOKEN)
    Y = osc.osc_fp8_gemm(q8, s8, osc.osc_pack_weight_fp8(dev(W8)), N, K8)
    close(Y, oracle.fp8_gemm(*oracle.quantize_fp8_rows(X8), *oracle.quantize_fp8_rows(W8)), f"staged fp8 {cfg} {M}x{N}x{K8}")


def test_long_prompt_with_ragged_rows(osc):
    """500 x 2048 x 4128, where the launcher itself takes the staged kernel for rows that are not whole lines; sampled rows."""
    M, N, K = 500, 2048, 4128
    X, table = wl.activations_persistent(7740, M, K, 1)
    W = wl.weights(7741, N, K)
    oidx = oracle.table_to_index(table)
    Xq, Xs, B = osc.osc_quantize_act(dev(X), dev(oidx))
    Wp = osc.osc_pack_weight(dev(W), dev(oidx))
    rows = np.array([0, 63, 64, 127, 128, 300, 447, 448, 499])
    rq, rs, rb = oracle.quantize_mxfp4_osc(X[rows], oidx, ldb=B.shape[1])
    wq, ws, _ = oracle.quantize_mxfp4_osc(W)
    ref = oracle.dual_gemm(rq, rs, rb, wq, ws, oracle.gather_wl(W, oidx))
    Y = osc.osc_dual_gemm(Xq, Xs, B, Wp, N, K, len(oidx), osc.OSC_DT_F32)
    close(Y[torch.from_numpy(rows).cuda()], ref, "long ragged prompt")


@pytest.mark.parametrize("cfg", ["4,1", "2,1", "1,1", "1,0", "2,0", "1,3"])
def test_fp8_and_mxfp8_forced(osc, tuning, cfg):
    tuning.gemm(cfg)
    M, N, K = 300, 264, 768
    X = wl.activations_diffuse(7200, M, K)
    W = wl.weights(7201, N, K)
    X8, xs = osc.osc_quantize_act(dev(X), None, osc.OSC_FMT_FP8_E4M3_TOKEN)
    r8, rs = oracle.quantize_fp8_rows(X)
    w8, ws = oracle.quantize_fp8_rows(W)
    close(osc.osc_fp8_gemm(X8, xs, osc.osc_pack_weight_fp8(dev(W)), N, K), oracle.fp8_gemm(r8, rs, w8, ws), "fp8 " + cfg)
    if not cfg.endswith(",0"):  # the MXFP8 GEMM has no staged form
        Xm, Xms = osc.osc_quantize_act(dev(X), None, osc.OSC_FMT_MXFP8)
        q, s = oracle.quantize_mxfp8(X)
        wq, wsc = oracle.quantize_mxfp8(W)
        Y = osc.osc_mxfp8_gemm(Xm, Xms, osc.osc_pack_weight_mxfp8(dev(W)), N, K)
        close(Y, oracle.mxfp8_gemm(q, s, wq, wsc), "mxfp8 " + cfg)


@pytest.mark.parametrize("cfg", [None, "4,1", "1,1", "1,0"])
def test_output_into_wider_and_odd_buffers(osc, tuning, cfg):
    if cfg:
        tuning.gemm(cfg)
    M, N, K = 200, 320, 512
    X, table = wl.activations_persistent(7300, M, K, 2)
    W = wl.weights(7301, N, K)
    oidx = oracle.table_to_index(table)
    Xq, Xs, B = osc.osc_quantize_act(dev(X), dev(oidx))
    Wp = osc.osc_pack_weight(dev(W), dev(oidx))
    rq, rs, rb = oracle.quantize_mxfp4_osc(X, oidx, ldb=B.shape[1])
    wq, ws, _ = oracle.quantize_mxfp4_osc(W)
    ref = oracle.dual_gemm(rq, rs, rb, wq, ws, oracle.gather_wl(W, oidx))
    for dt, ydt, bf in ((torch.float32, osc.OSC_DT_F32, False), (torch.bfloat16, osc.OSC_DT_BF16, True)):
        # aligned wide buffer (16-byte stores); first column 4 elements in (8-byte stores for bf16);
        # odd stride and odd first column (element stores)
        for width, col0 in ((N + 64, 0), (N + 64, 4), (N + 7, 3)):
            wide = torch.full((M, width), 7.0, dtype=dt, device="cuda")
            view = wide[:, col0:col0 + N]
            osc.osc_dual_gemm(Xq, Xs, B, Wp, N, K, len(oidx), ydt, out=view)
            close(view, ref, f"ldy={width} col0={col0} bf16={bf}", bf)
            rest = torch.cat([wide[:, :col0], wide[:, col0 + N:]], dim=1)
            assert (rest == 7.0).all(), "wrote outside the output view"


@pytest.mark.parametrize("cfg,K,K2", [("4,1", 512, 384), ("2,1", 512, 384), ("1,1", 512, 384), ("1,0", 1056, 400), ("2,0", 1056, 400)])
def test_grouped_with_skewed_experts(osc, tuning, cfg, K, K2):
    """Experts of 0, 1, 63 ... 700 rows, sizes on both sides of every tile border, through the DMA
    kernel's 256-row tiles (4,1) and the smaller ones: dual path with a row map, per-token FP8 and
    MXFP8; staged (,0) with rows that are not whole lines."""
    tuning.gemm(cfg)
    sizes = [0, 1, 63, 64, 65, 127, 128, 129, 255, 256, 257, 383, 384, 385, 700, 0, 130]
    E = len(sizes)
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int32)
    T = int(off[-1])
    tokens, N, r = 900, 256, 2
    X, table = wl.activations_persistent(7500, tokens, K, r)
    oidx = oracle.table_to_index(table)
    row_map = wl.rng(7501).integers(0, tokens, T).astype(np.int32)
    Xq, Xs, B = osc.osc_quantize_act(dev(X), dev(oidx))
    rq, rs, rb = oracle.quantize_mxfp4_osc(X, oidx, ldb=B.shape[1])
    stride = osc.osc_packed_weight_bytes(N, K, len(oidx))
    Wp = torch.empty(E * stride, dtype=torch.uint8, device="cuda")
    wq, wsc, wlr = [], [], []
    for e in range(E):
        W = wl.weights(7510 + e, N, K)
        osc.osc_pack_weight(dev(W), dev(oidx), out=Wp[e * stride:(e + 1) * stride])
        a, b, _ = oracle.quantize_mxfp4_osc(W)
        wq.append(a), wsc.append(b), wlr.append(oracle.gather_wl(W, oidx))
    ref = oracle.grouped_dual_gemm(rq, rs, rb, row_map, off, np.stack(wq), np.stack(wsc), np.stack(wlr))
    for ydt, bf in ((osc.OSC_DT_F32, False), (osc.OSC_DT_BF16, True)):
        Y = osc.osc_grouped_dual_gemm(Xq, Xs, B, dev(row_map), dev(off), T, Wp, N, K, len(oidx), ydt)
        assert osc.osc_tuning_last_gemm() == (int(cfg[2]), int(cfg[0]))
        close(Y, ref, f"grouped dual {cfg} bf16={bf}", bf)
    # 8-bit forms: rows in expert order (no row map in these entry points); MXFP8 rows are whole lines
    mx = K2 % 128 == 0
    X2 = wl.activations_diffuse(7502, T, K2)
    X8, xs = osc.osc_quantize_act(dev(X2), None, osc.OSC_FMT_FP8_E4M3_TOKEN)
    Xm, Xms = osc.osc_quantize_act(dev(X2), None, osc.OSC_FMT_MXFP8) if mx else (None, None)
    r8, r8s = oracle.quantize_fp8_rows(X2)
    m8, m8s = oracle.quantize_mxfp8(X2) if mx else (None, None)
    s8, sm = osc.osc_packed_weight_fp8_bytes(N, K2), osc.osc_packed_weight_mxfp8_bytes(N, K2)
    Wp8 = torch.empty(E * s8, dtype=torch.uint8, device="cuda")
    Wpm = torch.empty(E * sm, dtype=torch.uint8, device="cuda")
    w8, w8s = [], []
    refm = np.zeros((T, N))
    for e in range(E):
        W = wl.weights(7530 + e, N, K2)
        osc.osc_pack_weight_fp8(dev(W), out=Wp8[e * s8:(e + 1) * s8])
        a, b = oracle.quantize_fp8_rows(W)
        w8.append(a), w8s.append(b)
        if mx:
            osc.osc_pack_weight_mxfp8(dev(W), out=Wpm[e * sm:(e + 1) * sm])
        if mx and off[e + 1] > off[e]:
            refm[off[e]:off[e + 1]] = oracle.mxfp8_gemm(m8[off[e]:off[e + 1]], m8s[off[e]:off[e + 1]], *oracle.quantize_mxfp8(W))
    ref8 = oracle.grouped_fp8_gemm(r8, r8s, off, np.stack(w8), np.stack(w8s))
    close(osc.osc_fp8_gemm(X8, xs, Wp8, N, K2, expert_offsets=dev(off), y_dtype=osc.OSC_DT_BF16), ref8, "grouped fp8 " + cfg, True)
    if mx:
        close(osc.osc_mxfp8_gemm(Xm, Xms, Wpm, N, K2, expert_offsets=dev(off), y_dtype=osc.OSC_DT_BF16), refm, "grouped mxfp8 " + cfg, True)


def test_launcher_takes_256_row_dma_tiles_for_few_stages(osc):
    """4100 x 2000 at three stages: the launcher's own choice is 256 x 256 tiles of the DMA kernel on eight wavefronts, with a ragged
    last tile in both directions; a row of every fourth 128 and the borders against the oracle."""
    M, N, K, r = 4100, 2000, 512, 2
    X, table = wl.activations_persistent(7600, M, K, r)
    W = wl.weights(7601, N, K)
    oidx = oracle.table_to_index(table)
    rows = np.unique(np.concatenate([np.arange(0, 32, 4) * 128 + 5, [0, 127, 128, 4095, 4096, 4099]]))
    Xq, Xs, B = osc.osc_quantize_act(dev(X), dev(oidx))
    Wp = osc.osc_pack_weight(dev(W), dev(oidx))
    rq, rs, rb = oracle.quantize_mxfp4_osc(X[rows], oidx, ldb=B.shape[1])
    wq, ws, _ = oracle.quantize_mxfp4_osc(W)
    ref = oracle.dual_gemm(rq, rs, rb, wq, ws, oracle.gather_wl(W, oidx))
    sel = torch.from_numpy(rows).cuda()
    for ydt, bf in ((osc.OSC_DT_BF16, True), (osc.OSC_DT_F32, False)):
        Y = osc.osc_dual_gemm(Xq, Xs, B, Wp, N, K, len(oidx), ydt)
        assert osc.osc_tuning_last_gemm() == (1, 4)
        close(Y[sel], ref, f"256-row tiles bf16={bf}", bf)


# a shape for each: one round of 256 x 256 tiles and more on the persistent kernel, the flowing kernel, few rows, few blocks
@pytest.mark.parametrize("cfg,M,N,K", [(None, 400, 4096, 1280), (None, 4400, 4096, 512), (None, 4096, 4096, 1536), (None, 16, 512, 1024), (None, 200, 600, 768),
                                       ("4,2", 600, 520, 1024), ("0,7", 600, 520, 1024), ("3,7", 600, 520, 1024), ("4,4", 600, 520, 1024),
                                       ("1,1", 600, 520, 1024), ("2,1", 600, 520, 1024), ("4,1", 600, 520, 1024)])
def test_activation_scales_at_any_word(osc, tuning, cfg, M, N, K):
    """Activation scales may start at any 4-byte address: same numbers (up to the order of the sums, where another kernel takes the
    call) as from a 16-byte address, and no kernel that fetches them 16 bytes at a time."""
    X, table = wl.activations_persistent(7800, M, K, 1)
    d_oidx = dev(oracle.table_to_index(table))
    W = dev(wl.weights(7801, N, K))
    q, Wp = osc.osc_quantize_act(dev(X), d_oidx), osc.osc_pack_weight(W, d_oidx)
    qm, Wm = osc.osc_quantize_act(dev(X), None, osc.OSC_FMT_MXFP8), osc.osc_pack_weight_mxfp8(W)
    calls = {"dual": (q[1], lambda s: osc.osc_dual_gemm(q[0], s, q[2], Wp, N, K, K // 32, osc.OSC_DT_F32)),
             "mxfp8": (qm[1], lambda s: osc.osc_mxfp8_gemm(qm[0], s, Wm, N, K, y_dtype=osc.OSC_DT_F32))}
    for name, (scales, call) in calls.items():
        tuning.gemm("1,1")
        Y0 = call(scales)
        tuning.gemm(cfg)
        for words in (1, 2, 3):
            buf = torch.full((scales.numel() + 16,), 0xff, dtype=torch.uint8, device="cuda")
            view = buf[4 * words:4 * words + scales.numel()]
            view.copy_(scales)
            assert view.data_ptr() % 16 == 4 * words
            Y = call(view)
            assert osc.osc_tuning_last_gemm()[0] not in (2, 4, 7), (name, osc.osc_tuning_last_gemm())
            assert float((Y - Y0).abs().max()) <= 1e-5 * float(Y0.abs().max()), (name, words)
