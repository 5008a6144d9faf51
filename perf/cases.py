"""The work that is timed: the linear layers of a transformer run through the library's public entry
points, from one decoded token to a full prefill, and the offline calibration that precedes them.

Shapes are those of the benchmark configurations (hidden 4096 with 4096 / 1024 / 12288 outputs, the
mixture-of-experts layer with hidden 2048, 128 experts of 768, top 8) and generic ones between
them.  Every path starts at bf16 activations and ends at what its caller uses; quantised
activations, scales and gathered outliers are the path's own intermediate results.

kind       one pass
linear     quantise the activations in the format `fmt`, one GEMM
attn       quantise + q, k, v projections; quantise + o projection
ffn        RMSNorm fused with the quantiser, gate|up projection, SwiGLU fused with the 8-bit quantiser of
           the `w2` format, down projection
moe        quantise, grouped gate|up projection over routed rows, SwiGLU + 8-bit quantiser, grouped down
           projection
dynamic    run-time protection: quantise with the outliers found per token, GEMM with the dense branch
calibrate  threshold, candidate counts and suppression table of a calibration set

`reuse` says whether the caller keeps its output buffers from call to call (a serving loop) or lets the
entry points allocate them.
"""
import math

import torch

import paper_2604_12782_amd as osc

DEV = "cuda"
BF16 = osc.OSC_DT_BF16
F32 = osc.OSC_DT_F32
LARGEST_MNK = 8192 * 12288 * 4096  # no drawn linear or dynamic layer is larger


def listed():
    return [
        # one token through an attention block's projections: launches and latency are all there is
        dict(name="attn_decode_1", kind="attn", M=1, K=4096, Nq=4096, Nkv=1024, r=2, reuse=True),
        # the step that the repository's benchmark times
        dict(name="attn_prefill_8192", kind="attn", M=8192, K=4096, Nq=4096, Nkv=1024, r=2, reuse=False),
        # a decode batch through a whole feed-forward block: the weights are streamed once
        dict(name="ffn_decode_16", kind="ffn", M=16, K=4096, inter=12288, r=2, w2="mxfp8", reuse=True),
        # the largest call: a full prefill through the same block
        dict(name="ffn_prefill_8192", kind="ffn", M=8192, K=4096, inter=12288, r=2, w2="mxfp8", reuse=False),
        # a prompt of ordinary, odd length, with the other 8-bit format for the down projection
        dict(name="ffn_prompt_1000_fp8", kind="ffn", M=1000, K=4096, inter=12288, r=1, w2="fp8", reuse=False),
        # experts with a few rows each (a decode batch) and with a few hundred (a prefill)
        dict(name="moe_decode_32", kind="moe", T=32, K=2048, inter=768, E=128, top=8, r=2, w2="fp8", reuse=True),
        dict(name="moe_prefill_4096", kind="moe", T=4096, K=2048, inter=768, E=128, top=8, r=2, w2="mxfp8", reuse=False),
        # a chunk of a prompt through one wide projection, four protected channels per group
        dict(name="linear_512_wide", kind="linear", fmt="mxfp4", M=512, N=12288, K=4096, r=4, y="bf16", reuse=False),
        # sizes that no tile divides, single-precision results
        dict(name="linear_ragged_333", kind="linear", fmt="mxfp4", M=333, N=1000, K=2080, r=1, y="f32", reuse=False),
        # the W8A8 fallback on a prompt
        dict(name="linear_fp8_2048", kind="linear", fmt="fp8", M=2048, N=4096, K=4096, r=0, y="bf16", reuse=False),
        # the format with scales per 16 channels, in the regime it is built for
        dict(name="linear_nvfp4_16", kind="linear", fmt="nvfp4", M=16, N=12288, K=4096, r=1, y="bf16", reuse=True),
        # calibrating one position of one layer
        dict(name="calibrate_8192", kind="calibrate", M=8192, K=4096, G=32, R=2, reuse=True),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _size(rng, lo, hi, *steps):
    """a size between lo and hi, spread over its logarithm, a multiple of one of `steps`"""
    step = rng.choice(steps)
    return max(step, _log_int(rng, lo, hi) // step * step)


def draw(rng):
    kind = rng.choice(["linear"] * 5 + ["attn"] * 2 + ["ffn"] * 2 + ["moe"] * 2 + ["dynamic", "calibrate"])
    reuse = rng.random() < 0.5
    r = rng.choice([0, 1, 1, 2, 2, 4])
    if kind == "linear":
        fmt = rng.choice(["mxfp4"] * 5 + ["mxfp4_g64", "fp8", "fp8", "mxfp8", "e8m0_16", "nvfp4"])
        few = fmt in ("e8m0_16", "nvfp4")  # formats for a few tokens
        K = _size(rng, 512, 12288, 256) if few else _size(rng, 512, 12288, 128) if fmt == "mxfp8" else \
            _size(rng, 512, 12288, 256, 256, 64)
        N = _size(rng, 256, 12288, 128, 8)
        M = min(_log_int(rng, 1, 128 if few else 8192), LARGEST_MNK // (N * K))
        return dict(kind=kind, fmt=fmt, M=M, N=N, K=K, r=0 if fmt in ("fp8", "mxfp8") else r,
                    y=rng.choice(["bf16", "bf16", "f32"]), reuse=reuse)
    if kind == "attn":
        K = _size(rng, 1024, 4096, 256)
        return dict(kind=kind, M=_log_int(rng, 1, 8192), K=K, Nq=_size(rng, 1024, 4096, 128), Nkv=_size(rng, 256, 1024, 128),
                    r=r, reuse=reuse)
    if kind == "ffn":
        return dict(kind=kind, M=_log_int(rng, 1, 4096), K=_size(rng, 1024, 4096, 256), inter=_size(rng, 2048, 12288, 128),
                    r=r, w2=rng.choice(["mxfp8", "fp8"]), reuse=reuse)
    if kind == "moe":
        return dict(kind=kind, T=_log_int(rng, 1, 4096), K=_size(rng, 1024, 2048, 256), inter=_size(rng, 512, 768, 128),
                    E=rng.choice([32, 64, 128]), top=rng.choice([2, 4, 8]), r=r, w2=rng.choice(["mxfp8", "fp8"]), reuse=reuse)
    if kind == "dynamic":
        return dict(kind=kind, M=_log_int(rng, 1, 2048), N=_size(rng, 512, 4096, 128, 8), K=_size(rng, 512, 4096, 256),
                    r=0, y="bf16", reuse=reuse)
    return dict(kind=kind, M=_log_int(rng, 256, 16384), K=_size(rng, 1024, 8192, 64), G=rng.choice([16, 32, 64]),
                R=rng.choice([1, 2]), reuse=reuse)


# ---- inputs -------------------------------------------------------------------------------------


def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(seed)


def _table(g, K, r, G=32):
    """r distinct local indices per group of G channels, ascending: int16 [K/G, max(r, 1)] on the host"""
    pick = torch.rand((K // G, G), generator=g, device=DEV).argsort(dim=1)[:, :max(r, 1)].sort(dim=1).values
    return (pick if r else torch.full_like(pick, -1)).to(torch.int16).cpu()


def _channels(g, K, r, G=32):
    """the protected channels of a random suppression table as the device list the entry points take"""
    if r == 0:
        return None
    return torch.from_numpy(osc.osc_table_to_index_g(_table(g, K, r, G).numpy(), G)).to(DEV)


def _activations(g, M, K, oidx):
    """N(0, 1) with token-persistent outlier channels, each with one factor between 20 and 100"""
    x = torch.randn((M, K), generator=g, device=DEV)
    if oidx is not None:
        f = torch.rand(oidx.numel(), generator=g, device=DEV) * math.log(5.0) + math.log(20.0)
        x[:, oidx.long()] *= f.exp()
    return x.to(torch.bfloat16)


def _diffuse(g, M, K):
    """N(0, 1) with scattered outliers (the inputs of the 8-bit fallback)"""
    x = torch.randn((M, K), generator=g, device=DEV)
    x *= 1.0 + 49.0 * (torch.rand((M, K), generator=g, device=DEV) < 0.005)
    return x.to(torch.bfloat16)


def _weight(g, N, K):
    return (torch.randn((N, K), generator=g, device=DEV) * 0.02).to(torch.bfloat16)


def _zeros(shape, dtype):
    return torch.zeros(shape, dtype=dtype, device=DEV)


def _up64(n):
    return (n + 63) // 64 * 64


def _quant_out(M, K, K_o):
    return (_zeros((M, K // 2), torch.uint8), _zeros(osc.osc_act_scale_bytes(M, K), torch.uint8),
            _zeros((M, _up64(K_o)), torch.uint16) if K_o else None)


def _w2_out(M, K, w2):
    return (_zeros((M, K), torch.uint8),
            _zeros(osc.osc_act_scale_bytes(M, K), torch.uint8) if w2 == "mxfp8" else _zeros(M, torch.float32))


def _experts(g, E, N, K, bytes_each, pack):
    """E packed weights at a uniform stride"""
    packs = torch.empty((E, bytes_each), dtype=torch.uint8, device=DEV)
    for e in range(E):
        pack(_weight(g, N, K), packs[e])
    return packs.view(-1)


def _routing(g, T, E, top):
    """top-k routing from random logits: first routed row of every expert, and the token of every routed row"""
    chosen = torch.randn((T, E), generator=g, device=DEV).topk(top, dim=1).indices.reshape(-1)
    order = chosen.argsort(stable=True)
    offsets = torch.zeros(E + 1, dtype=torch.int32, device=DEV)
    offsets[1:] = torch.bincount(chosen, minlength=E).cumsum(0)
    return offsets, (order // top).to(torch.int32)


def prepare(case, seed):
    g, kind, reuse = _gen(seed), case["kind"], case["reuse"]
    s = dict(case)
    if kind == "linear":
        M, N, K, fmt = case["M"], case["N"], case["K"], case["fmt"]
        G = 64 if fmt == "mxfp4_g64" else 32
        oidx = _channels(g, K, case["r"], G)
        K_o = 0 if oidx is None else oidx.numel()
        X = _diffuse(g, M, K) if fmt in ("fp8", "mxfp8") else _activations(g, M, K, oidx)
        W = _weight(g, N, K)
        s.update(X=X, oidx=oidx, K_o=K_o, ydt=BF16 if case["y"] == "bf16" else F32, q=None, Y=None, xts=1.0, wts=1.0)
        if fmt == "fp8":
            s["W"] = osc.osc_pack_weight_fp8(W)
            out = _w2_out(M, K, "fp8")
        elif fmt == "mxfp8":
            s["W"] = osc.osc_pack_weight_mxfp8(W)
            out = _w2_out(M, K, "mxfp8")
        elif fmt in ("e8m0_16", "nvfp4"):
            s["f16"] = osc.OSC_FMT16_NVFP4 if fmt == "nvfp4" else osc.OSC_FMT16_E8M0
            if fmt == "nvfp4":  # calibrated tensor scales: the largest magnitude maps to 6 * 448
                s["xts"], s["wts"] = 5.0 / (6 * 448), float(W.abs().max()) / (6 * 448)
            s["W"] = osc.osc_pack_weight_g16(W, oidx, s["f16"], s["wts"])
            out = (_zeros((M, K // 2), torch.uint8), _zeros((M, K // 16), torch.uint8),
                   _zeros((M, _up64(K_o)), torch.uint16) if K_o else None)
        else:
            s["W"] = osc.osc_pack_weight_g(W, oidx, G)
            out = _quant_out(M, K, K_o)
        if reuse:
            s["q"], s["Y"] = out, _zeros((M, N), torch.bfloat16 if case["y"] == "bf16" else torch.float32)
    elif kind == "attn":
        M, K, Nq, Nkv = case["M"], case["K"], case["Nq"], case["Nkv"]
        o1, o2 = _channels(g, K, case["r"]), _channels(g, Nq // 32 * 32, case["r"])
        s.update(o1=o1, o2=o2, X1=_activations(g, M, K, o1), X2=_activations(g, M, Nq, o2),
                 K1=0 if o1 is None else o1.numel(), K2=0 if o2 is None else o2.numel())
        s["Wqkv"] = [(n, osc.osc_pack_weight(_weight(g, n, K), o1)) for n in (Nq, Nkv, Nkv)]
        s["Wo"] = osc.osc_pack_weight(_weight(g, K, Nq), o2)
        s["q1"], s["q2"], s["Y"] = (_quant_out(M, K, s["K1"]), _quant_out(M, Nq, s["K2"]),
                                    [_zeros((M, n), torch.bfloat16) for n in (Nq, Nkv, Nkv, K)]) if reuse else (None, None, [None] * 4)
    elif kind == "ffn":
        M, K, F = case["M"], case["K"], case["inter"]
        oidx = _channels(g, K, case["r"])
        K_o = 0 if oidx is None else oidx.numel()
        s.update(oidx=oidx, K_o=K_o, X=_activations(g, M, K, oidx), q=None, q2=None, H=None, Y=None,
                 gamma=(1.0 + 0.1 * torch.randn(K, generator=g, device=DEV)).to(torch.bfloat16),
                 W13=osc.osc_pack_weight(_weight(g, 2 * F, K), oidx))
        pack2 = osc.osc_pack_weight_mxfp8 if case["w2"] == "mxfp8" else osc.osc_pack_weight_fp8
        s["W2"] = pack2(_weight(g, K, F))
        if reuse:
            s.update(q=_quant_out(M, K, K_o) + (None,), q2=_w2_out(M, F, case["w2"]) + (None,),
                     H=_zeros((M, 2 * F), torch.bfloat16), Y=_zeros((M, K), torch.bfloat16))
    elif kind == "moe":
        T, K, F, E = case["T"], case["K"], case["inter"], case["E"]
        oidx = _channels(g, K, case["r"])
        K_o = 0 if oidx is None else oidx.numel()
        off, rows = _routing(g, T, E, case["top"])
        s.update(oidx=oidx, K_o=K_o, off=off, rows=rows, n=T * case["top"], X=_activations(g, T, K, oidx), q=None, q2=None, H=None,
                 Y=None, W13=_experts(g, E, 2 * F, K, osc.osc_packed_weight_bytes(2 * F, K, K_o), lambda w, o: osc.osc_pack_weight(w, oidx, out=o)))
        if case["w2"] == "mxfp8":
            s["W2"] = _experts(g, E, K, F, osc.osc_packed_weight_mxfp8_bytes(K, F), osc.osc_pack_weight_mxfp8)
        else:
            s["W2"] = _experts(g, E, K, F, osc.osc_packed_weight_fp8_bytes(K, F), osc.osc_pack_weight_fp8)
        if reuse:
            s.update(q=_quant_out(T, K, K_o), q2=_w2_out(s["n"], F, case["w2"]) + (None,),
                     H=_zeros((s["n"], 2 * F), torch.bfloat16), Y=_zeros((s["n"], K), torch.bfloat16))
    elif kind == "dynamic":
        M, N, K = case["M"], case["N"], case["K"]
        oidx = _channels(g, K, 1)
        s.update(X=_activations(g, M, K, oidx), q=None, Y=None,
                 W=osc.osc_pack_weight(_weight(g, N, K), torch.arange(K, dtype=torch.int32, device=DEV)))
        if reuse:
            s.update(q=_quant_out(M, K, K) + (_zeros((M, K // 32), torch.uint8),), Y=_zeros((M, N), torch.bfloat16))
    else:
        M, K, G, R = case["M"], case["K"], case["G"], case["R"]
        s["X"] = _activations(g, M, K, _channels(g, K, R, G))
        kg = K // G
        s["work"], s["out"] = (_zeros(osc.osc_profile_workspace_bytes(K), torch.uint8),
                               (_zeros((kg, R), torch.int16), _zeros(kg, torch.int32), _zeros(kg, torch.int32),
                                _zeros(kg, torch.float32), _zeros(1, torch.float32), _zeros(1, torch.float32))) if reuse else (None, None)
    return s


# ---- one pass -----------------------------------------------------------------------------------


def _swiglu_down(s, H, n, expert_offsets):
    """SwiGLU + 8-bit quantiser on the gate|up results H [n, 2F], down projection"""
    F, K = s["inter"], s["K"]
    if s["w2"] == "mxfp8":
        x8, xs, _ = osc.osc_swiglu_quantize_act(H[:, :F], H[:, F:], out=s["q2"])
        return osc.osc_mxfp8_gemm(x8, xs, s["W2"], K, F, expert_offsets, BF16, out=s["Y"])
    x8, xs, _ = osc.osc_swiglu_quantize_act_fp8(H[:, :F], H[:, F:], out=s["q2"])
    return osc.osc_fp8_gemm(x8, xs, s["W2"], K, F, expert_offsets, BF16, out=s["Y"])


def run(s):
    kind = s["kind"]
    if kind == "linear":
        N, K, fmt = s["N"], s["K"], s["fmt"]
        if fmt == "fp8":
            q = osc.osc_quantize_act(s["X"], fmt=osc.OSC_FMT_FP8_E4M3_TOKEN, out=s["q"])
            return osc.osc_fp8_gemm(*q, s["W"], N, K, y_dtype=s["ydt"], out=s["Y"]), q[0]
        if fmt == "mxfp8":
            q = osc.osc_quantize_act(s["X"], fmt=osc.OSC_FMT_MXFP8, out=s["q"])
            return osc.osc_mxfp8_gemm(*q, s["W"], N, K, y_dtype=s["ydt"], out=s["Y"]), q[0]
        if fmt in ("e8m0_16", "nvfp4"):
            q = osc.osc_quantize_act_g16(s["X"], s["oidx"], s["f16"], s["xts"], out=s["q"])
            return osc.osc_dual_gemm_g16(*q, s["W"], N, K, s["K_o"], s["f16"], s["xts"], s["wts"], s["ydt"], out=s["Y"]), q[0], q[2]
        q = osc.osc_quantize_act(s["X"], s["oidx"], osc.OSC_FMT_MXFP4_OSC_G64 if fmt == "mxfp4_g64" else osc.OSC_FMT_MXFP4_OSC, out=s["q"])
        return osc.osc_dual_gemm(*q, s["W"], N, K, s["K_o"], s["ydt"], out=s["Y"]), q[0], q[2]
    if kind == "attn":
        q = osc.osc_quantize_act(s["X1"], s["o1"], out=s["q1"])
        ys = [osc.osc_dual_gemm(*q, w, n, s["K"], s["K1"], BF16, out=y) for (n, w), y in zip(s["Wqkv"], s["Y"])]
        q = osc.osc_quantize_act(s["X2"], s["o2"], out=s["q2"])
        return ys + [osc.osc_dual_gemm(*q, s["Wo"], s["K"], s["Nq"], s["K2"], BF16, out=s["Y"][3])]
    if kind == "ffn":
        xq, xs, b, _ = osc.osc_rmsnorm_quantize_act(s["X"], s["gamma"], 1e-6, s["oidx"], out=s["q"])
        H = osc.osc_dual_gemm(xq, xs, b, s["W13"], 2 * s["inter"], s["K"], s["K_o"], BF16, out=s["H"])
        return _swiglu_down(s, H, s["M"], None)
    if kind == "moe":
        q = osc.osc_quantize_act(s["X"], s["oidx"], out=s["q"])
        H = osc.osc_grouped_dual_gemm(*q, s["rows"], s["off"], s["n"], s["W13"], 2 * s["inter"], s["K"], s["K_o"], BF16, out=s["H"])
        return _swiglu_down(s, H, s["n"], s["off"])
    if kind == "dynamic":
        xq, xs, bd, idx = osc.osc_quantize_act_dynamic(s["X"], out=s["q"])
        return osc.osc_dual_gemm(xq, xs, bd, s["W"], s["N"], s["K"], s["K"], BF16, out=s["Y"]), xq, idx
    return osc.osc_profile_calibrate(s["X"], s["G"], 5.0, s["R"], s["work"], s["out"])


# ---- what a pass cannot do without --------------------------------------------------------------


def _channel_count(K, r, G=32):
    return K // G * r


def _w4(N, K, K_o):
    """bytes of a packed four-bit weight with its bf16 branch"""
    return N * (K / 2 + K / 32 + 2 * K_o)


def _dual(M, N, K, K_o):
    return 2.0 * M * N * (K + K_o)


def work(case):
    kind = case["kind"]
    if kind == "linear":
        M, N, K, fmt = case["M"], case["N"], case["K"], case["fmt"]
        K_o = _channel_count(K, case["r"], 64 if fmt == "mxfp4_g64" else 32)
        if fmt in ("fp8", "mxfp8"):
            w, codes = N * K * (1 if fmt == "fp8" else 1 + 1 / 32) + 4 * N, M * K
        else:
            w, codes = _w4(N, K, K_o) + (N * K / 32 if fmt in ("e8m0_16", "nvfp4") else 0), M * (K / 2 + 2 * _up64(K_o))
        return {"bytes": 2 * M * K + w + codes + M * N * (2 if case["y"] == "bf16" else 4), "flops": _dual(M, N, K, K_o)}
    if kind == "attn":
        M, K, Nq, Nkv = case["M"], case["K"], case["Nq"], case["Nkv"]
        k1, k2 = _channel_count(K, case["r"]), _channel_count(Nq, case["r"])
        return {"bytes": 2 * M * (K + Nq) + _w4(Nq + 2 * Nkv, K, k1) + _w4(K, Nq, k2) + 2 * M * (Nq + 2 * Nkv + K),
                "flops": _dual(M, Nq + 2 * Nkv, K, k1) + _dual(M, K, Nq, k2)}
    if kind in ("ffn", "moe"):
        K, F = case["K"], case["inter"]
        K_o = _channel_count(K, case["r"])
        if kind == "ffn":
            tokens = rows = case["M"]
            experts = 1
        else:
            tokens, rows = case["T"], case["T"] * case["top"]
            experts = case["E"] * (1 - (1 - case["top"] / case["E"]) ** tokens)  # expected number that any token reaches
        return {"bytes": 2 * tokens * K + experts * (_w4(2 * F, K, K_o) + K * F * (1 + 1 / 32 if case["w2"] == "mxfp8" else 1)) + 2 * rows * K,
                "flops": _dual(rows, 2 * F, K, K_o) + 2.0 * rows * K * F}
    if kind == "dynamic":
        M, N, K = case["M"], case["N"], case["K"]
        return {"bytes": 2 * M * K + _w4(N, K, K) + M * (K / 2 + K / 32) + 2 * M * N, "flops": _dual(M, N, K, K)}
    # the threshold needs every activation before the first comparison: two readings
    return {"bytes": 2 * 2 * case["M"] * case["K"], "flops": 4.0 * case["M"] * case["K"]}


def tolerance(case):
    """Measured against the same quantised operands multiplied in double precision, and against the other
    kernels' summation orders; stated at about four times what was seen.  Codes, gathered outliers,
    tables and counts are exact."""
    kind = case["kind"]
    if kind == "calibrate":  # doubles summed in any order, rounded to single precision once
        return {"rel": 1e-6}
    if kind == "linear" and case["y"] == "f32":  # 2.3e-7, largest 1.9e-6
        return {"rel": 1e-6, "max": 1e-5}
    if kind in ("ffn", "moe"):  # a bf16 result of the first GEMM on the other side of a tie moves an 8-bit code: 1.7e-3, largest 1.2e-2
        return {"rel": 7e-3, "max": 0.05}
    return {"rel": 7e-3, "max": 0.016}  # the bf16 result's own rounding: 1.7e-3, largest 4.3e-3
