"""GPU parity of the fused RMSNorm + OSC quantiser: the normalised row, the codes, the scales and
the gathered sub-tensor bit for bit against the oracle's RMSNorm followed by the oracle's quantiser."""
import numpy as np
import pytest
import torch

import oracle
import workloads as wl
from workloads import to_bf16_bits

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def osc():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2604_12782_amd as m
    m.lib()
    return m


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def check(osc, X, gamma, eps, oidx, ldb=None):
    M, K = X.shape
    K_o = len(oidx)
    if ldb is None:
        ldb = (K_o + 63) // 64 * 64
    Xq, Xs, B, Xn = osc.osc_rmsnorm_quantize_act(dev(X), dev(gamma), eps, dev(oidx.astype(np.int32)) if K_o else None,
                                                 ldb=ldb, want_norm=True)
    y = oracle.rmsnorm(X, gamma, eps)
    rq, rs, rb = oracle.quantize_mxfp4_osc(y, oidx, ldb=ldb)
    assert np.array_equal(Xn.cpu().numpy(), y), "normalised rows differ"
    assert np.array_equal(osc.osc_unpack_act_scales(Xs, M, K).cpu().numpy(), rs), "scales differ"
    assert np.array_equal(Xq.cpu().numpy(), rq), "codes differ"
    if ldb:
        assert np.array_equal(B.cpu().numpy(), rb), "gathered sub-tensor differs"
    # and the fused call equals the unfused GPU path on the normalised rows
    Uq, Us, Ub = osc.osc_quantize_act(Xn, dev(oidx.astype(np.int32)) if K_o else None, ldb=ldb)
    assert torch.equal(Uq, Xq) and (not ldb or torch.equal(Ub, B))
    assert torch.equal(osc.osc_unpack_act_scales(Us, M, K), osc.osc_unpack_act_scales(Xs, M, K))


@pytest.mark.parametrize("M,K,r", [(1, 32, 1), (5, 96, 0), (33, 1056, 2), (70, 4096, 2), (300, 2048, 1),
                                   (9, 8192, 1), (6, 12288, 2)])
def test_fused_matches_oracle(osc, M, K, r):
    gen = wl.rng(1100 + M)
    X, table = wl.activations_persistent(1100 + M, M, K, r, jitter=0.3)
    gamma = to_bf16_bits((1.0 + 0.3 * gen.standard_normal(K)).astype(np.float32))
    check(osc, X, gamma, 1e-6, oracle.table_to_index(table) if r else np.zeros(0, np.int32))


def test_fused_scales_and_edges(osc):
    gen = wl.rng(1201)
    K = 256
    gamma = to_bf16_bits((0.5 + gen.random(K)).astype(np.float32))
    oidx = np.array([3, 40, 41, 100, 255], np.int32)
    # rows of very different magnitude, a zero row, a row with one non-zero, wide range inside a row
    x = gen.standard_normal((8, K)).astype(np.float32)
    x[0] *= 1e-20
    x[1] *= 1e20
    x[2] = 0.0
    x[3] = 0.0
    x[3, 40] = -7.0
    x[4, 0], x[4, 1] = 2.0 ** 90, 2.0 ** -90
    x[5] = 3.0
    X = to_bf16_bits(x)
    X[6, ::3] = 0x8000
    for eps in (1e-6, 1e-12, 1.0):
        check(osc, X, gamma, eps, oidx)
        check(osc, X, gamma, eps, oidx, ldb=8)
    # eps = 0 on rows without an all-zero row
    check(osc, X[[0, 1, 3, 4, 5, 7]], gamma, 0.0, oidx)


# ---- SwiGLU + MXFP8 quantiser ---------------------------------------------------------------
def check_swiglu(osc, G, U, strided=False):
    M, K = G.shape
    if strided:  # the two halves of one fused gate||up buffer
        both = torch.from_numpy(np.concatenate([G, U], axis=1)).cuda()
        dG, dU = both[:, :K], both[:, K:]
    else:
        dG, dU = dev(G), dev(U)
    Xq, Xs, Yn = osc.osc_swiglu_quantize_act(dG, dU, want_y=True)
    y = oracle.swiglu(G, U)
    rq, rs = oracle.quantize_mxfp8(y)
    assert np.array_equal(Yn.cpu().numpy(), y), "activation values differ"
    assert np.array_equal(osc.osc_unpack_act_scales(Xs, M, K).cpu().numpy(), rs), "scales differ"
    assert np.array_equal(Xq.cpu().numpy(), rq), "codes differ"
    # and equal to the unfused GPU quantiser on the same values
    Uq, Us = osc.osc_quantize_act(Yn, None, osc.OSC_FMT_MXFP8)
    assert torch.equal(Uq, Xq)
    assert torch.equal(osc.osc_unpack_act_scales(Us, M, K), osc.osc_unpack_act_scales(Xs, M, K))


@pytest.mark.parametrize("M,K", [(1, 32), (7, 96), (40, 1056), (130, 4096), (9, 12288)])
def test_swiglu_fused_matches_oracle(osc, M, K):
    gen = wl.rng(1300 + M)
    G = to_bf16_bits((gen.standard_normal((M, K)) * 3).astype(np.float32))
    U = wl.activations_diffuse(1400 + M, M, K, p=0.01)
    check_swiglu(osc, G, U)
    check_swiglu(osc, G, U, strided=True)


def test_swiglu_every_gate_value(osc):
    """every bf16 bit pattern below 2^100 in magnitude as a gate (58 000 of them; above that the
    product with up leaves the bf16 range), against the oracle, bit for bit"""
    bits = np.arange(0x10000, dtype=np.uint32).astype(np.uint16)
    bits = bits[((bits >> 7) & 0xFF) < 227]
    K = 2048
    pad = (-len(bits)) % K
    G = np.concatenate([bits, np.zeros(pad, np.uint16)]).reshape(-1, K)
    gen = wl.rng(1501)
    U = to_bf16_bits((0.5 + gen.random(G.shape)).astype(np.float32))
    check_swiglu(osc, G, U)


# ---- SwiGLU + per-token FP8 quantiser -------------------------------------------------------
def check_swiglu_fp8(osc, G, U, strided=False):
    M, K = G.shape
    if strided:
        both = torch.from_numpy(np.concatenate([G, U], axis=1)).cuda()
        dG, dU = both[:, :K], both[:, K:]
    else:
        dG, dU = dev(G), dev(U)
    X8, xs, Yn = osc.osc_swiglu_quantize_act_fp8(dG, dU, want_y=True)
    y = oracle.swiglu(G, U)
    r8, rsc = oracle.quantize_fp8_rows(y)
    assert np.array_equal(Yn.cpu().numpy(), y), "activation values differ"
    assert np.array_equal(xs.cpu().numpy().view(np.uint32), rsc.view(np.uint32)), "scales differ"
    assert np.array_equal(X8.cpu().numpy(), r8), "codes differ"
    U8, us = osc.osc_quantize_act(Yn, None, osc.OSC_FMT_FP8_E4M3_TOKEN)
    assert torch.equal(U8, X8) and torch.equal(us, xs)
    X8b, xsb, none = osc.osc_swiglu_quantize_act_fp8(dG, dU)
    assert none is None and torch.equal(X8b, X8) and torch.equal(xsb, xs)


@pytest.mark.parametrize("M,K", [(122881, 1024), (122879, 1024), (245761, 512), (245759, 512)])
def test_swiglu_fp8_many_codes(osc, M, K):
    """Rows of one wavefront on both sides of the size from which on their codes are stored past the caches: many copies of a few rows
    give the rows' codes and scales everywhere."""
    gen = wl.rng(1601)
    G, U = to_bf16_bits((gen.standard_normal((97, K)) * 3).astype(np.float32)), wl.activations_diffuse(1602, 97, K, p=0.01)
    r8, rs = oracle.quantize_fp8_rows(oracle.swiglu(G, U))
    row = torch.arange(M, device="cuda") % 97
    big = lambda a: dev(a.view(np.int16))[row].view(torch.uint16)
    X8, xs, _ = osc.osc_swiglu_quantize_act_fp8(big(G), big(U))
    assert torch.equal(X8, dev(r8)[row])
    assert torch.equal(xs.view(torch.int32), dev(rs.view(np.int32))[row])


@pytest.mark.parametrize("M,K", [(1, 8), (7, 96), (40, 1056), (130, 4096), (9, 12288), (3, 16384), (5, 2056)])
def test_swiglu_fp8_fused_matches_oracle(osc, M, K):
    gen = wl.rng(1600 + M)
    G = to_bf16_bits((gen.standard_normal((M, K)) * 3).astype(np.float32))
    U = wl.activations_diffuse(1700 + M, M, K, p=0.01)
    if M > 4:
        G[2] = 0  # an all-zero row: scale 1, codes 0
        U[3] = to_bf16_bits(np.full(K, 1e-36, np.float32))  # a row below 2^-100: scale 1
    check_swiglu_fp8(osc, G, U)
    check_swiglu_fp8(osc, G, U, strided=True)


def test_swiglu_fp8_every_gate_value(osc):
    bits = np.arange(0x10000, dtype=np.uint32).astype(np.uint16)
    bits = bits[((bits >> 7) & 0xFF) < 227]
    K = 2048
    pad = (-len(bits)) % K
    G = np.concatenate([bits, np.zeros(pad, np.uint16)]).reshape(-1, K)
    U = to_bf16_bits((0.5 + wl.rng(1801).random(G.shape)).astype(np.float32))
    check_swiglu_fp8(osc, G, U)


# row lengths around every change of form: wavefront or workgroup per row (2048), chunks per thread
# (4096, 8192, 12288), and more short rows than the MXFP8 form's fixed grid holds at once
@pytest.mark.parametrize("M,K", [(5, 2048), (3, 4104), (2, 8200), (2, 12296), (1, 512), (6, 520)])
def test_swiglu_fp8_row_forms(osc, M, K):
    gen = wl.rng(1900 + K)
    check_swiglu_fp8(osc, to_bf16_bits((gen.standard_normal((M, K)) * 3).astype(np.float32)),
                     wl.activations_diffuse(1950 + K, M, K, p=0.01))


@pytest.mark.parametrize("M,K", [(16450, 32), (33, 992), (33, 1024)])
def test_swiglu_mxfp8_grid_forms(osc, M, K):
    gen = wl.rng(2000 + K)
    check_swiglu(osc, to_bf16_bits((gen.standard_normal((M, K)) * 3).astype(np.float32)),
                 wl.activations_diffuse(2050 + K, M, K, p=0.01))


@pytest.mark.parametrize("K", [64, 2048])
def test_swiglu_saturates_beyond_bf16(osc, K):
    """Finite gates and ups whose product leaves the bf16 range, infinite gates and ups, and NaN, beside finite values
    of the same block and of other blocks: the codes and scales are those of the quantiser on the values that the
    call returns (infinities saturate at +-448, no NaN code), in both 8-bit formats.  Exact."""
    gen = wl.rng(2100 + K)
    edge = np.array([0x7F7F, 0xFF7F, 0x7F80, 0xFF80, 0x7FC0, 0x7E96, 0xFE96, 0x3F80, 0xBF80, 0x0000], np.uint16)  # +-max, inf, nan, 1e38, 1, 0
    G = to_bf16_bits((gen.standard_normal((40, K)) * 3).astype(np.float32))
    U = to_bf16_bits((gen.standard_normal((40, K)) * 3).astype(np.float32))
    at = gen.random((40, K)) < np.repeat(gen.random((40, K // 32)) < 0.5, 32, axis=1) * 0.2  # in half of the blocks
    G[at], U[at] = gen.choice(edge, int(at.sum())), gen.choice(edge, int(at.sum()))
    G[0], U[0] = 0x7E96, to_bf16_bits(np.linspace(-4e38, 4e38, K).clip(-3e38, 3e38).astype(np.float32))  # finite only, overflowing
    Xq, Xs, Yn = osc.osc_swiglu_quantize_act(dev(G), dev(U), want_y=True)
    y = Yn.cpu().numpy()
    assert ((y[0] & 0x7FFF) == 0x7F80).any() and ((y & 0x7F80) != 0x7F80).any(), "the inputs miss what this test is about"
    Uq, Us = osc.osc_quantize_act(Yn, None, osc.OSC_FMT_MXFP8)
    assert torch.equal(osc.osc_unpack_act_scales(Us, 40, K), osc.osc_unpack_act_scales(Xs, 40, K))
    assert torch.equal(Uq, Xq), "codes differ from the quantiser's"
    codes = Xq.cpu().numpy()
    assert not ((codes & 0x7F) == 0x7F).any(), "NaN codes"
    inf = (y & 0x7FFF) == 0x7F80
    assert np.array_equal(codes[inf], np.where(y[inf] >> 15, 0xFE, 0x7E)), "infinities do not saturate"
    X8, xs, Y8 = osc.osc_swiglu_quantize_act_fp8(dev(G), dev(U), want_y=True)
    U8, us = osc.osc_quantize_act(Y8, None, osc.OSC_FMT_FP8_E4M3_TOKEN)
    assert torch.equal(Y8, Yn) and torch.equal(U8, X8) and torch.equal(us.view(torch.int32), xs.view(torch.int32))


@pytest.mark.parametrize("K,r", [(32, 1), (1056, 2), (2048, 32), (4096, 0), (4096, 2), (8192, 4), (12288, 1)])
def test_fused_row_forms(osc, K, r):
    """A workgroup per row (few rows) and a wavefront per row (many) give the same bits: one call on many rows against
    calls on pieces of them, rows of very different magnitude, more protected channels than a workgroup has threads."""
    gen = wl.rng(1300 + K + r)
    M = 1100
    x = gen.standard_normal((M, K)).astype(np.float32) * np.exp2(gen.integers(-40, 40, (M, 1))).astype(np.float32)
    x[7] = 0.0
    X, gamma = dev(to_bf16_bits(x)), dev(to_bf16_bits((1.0 + 0.3 * gen.standard_normal(K)).astype(np.float32)))
    oidx = None
    if r:
        table = np.stack([np.sort(gen.permutation(32)[:r]) for _ in range(K // 32)]).astype(np.int16)
        oidx = dev(osc.osc_table_to_index(table))
    Xq, Xs, B, Xn = osc.osc_rmsnorm_quantize_act(X, gamma, 1e-6, oidx, want_norm=True)
    Xs = osc.osc_unpack_act_scales(Xs, M, K)
    for a, b in ((0, 32), (32, 33), (64, 500), (512, 1012)):
        q, s, bb, xn = osc.osc_rmsnorm_quantize_act(X[a:b], gamma, 1e-6, oidx, want_norm=True)
        assert torch.equal(q, Xq[a:b]) and torch.equal(xn, Xn[a:b]) and torch.equal(osc.osc_unpack_act_scales(s, b - a, K), Xs[a:b])
        assert not r or torch.equal(bb, B[a:b])


@pytest.mark.parametrize("M,K", [(1, 512), (33, 640), (37, 768), (130, 1152), (65, 2304), (5, 3200), (1030, 768), (1999, 512), (2000, 512), (2001, 512), (2675, 640),
                                 (4001, 768), (1150, 1152), (1337, 2304), (1147, 3200)])
def test_swiglu_mxfp8_rows_in_one_line(osc, M, K):
    """Rows of whole 128-channel words that segments of 1024 would leave lanes idle on, few of them (in segments) and many (in one
    line, from 2000 rows of 512 channels on): wavefronts that cover one, two and three rows, a last one that ends
    past the last row, against the oracle's fixed sequence and quantiser, from the halves of one buffer."""
    gen = wl.rng(1400 + M + K)
    H = to_bf16_bits((gen.standard_normal((M, 2 * K)) * 2).astype(np.float32))
    d = dev(H).view(torch.bfloat16) if dev(H).dtype != torch.bfloat16 else dev(H)
    Xq, Xs, Yn = osc.osc_swiglu_quantize_act(d[:, :K], d[:, K:], want_y=True)
    y = oracle.swiglu(np.ascontiguousarray(H[:, :K]), np.ascontiguousarray(H[:, K:]))
    q, s = oracle.quantize_mxfp8(y)
    assert np.array_equal(Yn.view(torch.int16).cpu().numpy().view(np.uint16), y.view(np.uint16))
    assert np.array_equal(osc.osc_unpack_act_scales(Xs, M, K).cpu().numpy(), s)
    assert np.array_equal(Xq.cpu().numpy(), q)
