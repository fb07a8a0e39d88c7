"""GPU parity, MX family with a block-scaled FP branch, MXFP8e4 or MXFP6e2 (all-MX setting of the
mixed-precision tables, Section 4.3; element formats of App. A.3) against the CPU oracle.

Bar: every code and E8M0 byte computed from source data (X, P, L, R) bit-exact (+0 and -0 codes are
the same value); the intermediate T and the output pass through the matrix core's own accumulation
(block-scaled 8-bit products summed in an order and an internal width the instruction set does not
document; measured worst case 2^-14.9 of the sum of the magnitudes of the terms) and are bounded by
2^-13 of that sum; the re-quantised
intermediate must be a correct block quantisation of a value within that bound of the oracle's T.
"""
import dataclasses

import numpy as np
import pytest
import torch

from paper_2604_18117_amd import workloads as wl
from tests.gpu_util import bf16_to_bits, check_bf16_against_oracle, check_end_to_end, n, run_gpu

pytestmark = pytest.mark.gpu

E2M1 = np.array([0, .5, 1, 1.5, 2, 3, 4, 6, -0., -.5, -1, -1.5, -2, -3, -4, -6], np.float32)
# fp32 accumulation inside the 8-bit scaled matrix instruction against the oracle's fp64 sum: at most this fraction of the
# sum of |terms| (measured worst case over every committed and swept case: 2^-14.9; the bar leaves a factor 1.9)
ACC = 2.0 ** -14


def _compare(oracle, layer, X, W, L, R, rows=None, gamma=None):
    g = run_gpu(layer, X, W, L, R, debug=True, debug_acc=False, gamma=gamma)
    Xo = X if rows is None else X[rows]
    if gamma is not None:                       # fused smoothing: the oracle quantises the smoothed input
        Xo = oracle.smooth(Xo, gamma)
    sel = slice(None) if rows is None else rows
    r = layer.r
    elem = layer.br_w_bits                      # 8: E4M3 elements; 6: E2M3 elements
    pk = oracle.pack_mxb(W, L if r else None, R if r else None, elem=elem)
    act = oracle.quantize_act_mxb(Xo, pk)
    f8 = oracle.mxb_decode(np.arange(256, dtype=np.uint8), elem)   # E2M3 ignores the upper two bits
    top, min_exp = (448.0, -9) if elem == 8 else (7.5, -3)
    Mo = Xo.shape[0]
    # ---- offline packing: exact
    assert np.array_equal(E2M1[n(g.wv.pq).view(np.uint8)], E2M1[pk.pc]), "pq"
    assert np.array_equal(n(g.wv.pe), pk.pe), "pe"
    if r:
        assert np.array_equal(f8[n(g.wv.lq).view(np.uint8)], f8[pk.l8]), "l8"
        assert np.array_equal(n(g.wv.le), pk.le), "le"
        assert np.array_equal(f8[n(g.wv.rq).view(np.uint8)], f8[pk.r8]), "r8"
        assert np.array_equal(n(g.wv.re), pk.re), "re"
    # ---- activation step: codes and block scales from X exact
    assert np.array_equal(E2M1[n(g.av.xq).view(np.uint8)[sel]], E2M1[act.xc]), "xc"
    assert np.array_equal(n(g.av.xe)[sel], act.xe), "xe"
    tq_gpu = n(g.av.tq).view(np.uint8)[sel] if r else np.zeros((Mo, 0), np.uint8)
    te_gpu = n(g.av.te)[sel] if r else np.zeros((Mo, 0), np.uint8)
    if r:
        assert np.array_equal(f8[n(g.adbg.xb).view(np.uint8)[sel]], f8[act.xb8]), "xb8"
        assert np.array_equal(n(g.adbg.xbe)[sel], act.xbe), "xbe"
        T_gpu = n(g.adbg.T)[sel]
        xs = np.abs(f8[act.xb8].astype(np.float64).reshape(Mo, -1, 32)) * oracle.e8m0_decode(act.xbe)[:, :, None]
        rs = np.abs(f8[pk.r8].astype(np.float64).reshape(r, -1, 32)) * oracle.e8m0_decode(pk.re)[:, :, None]
        tb = ACC * (xs.reshape(Mo, -1) @ rs.reshape(r, -1).T) + 1e-300
        assert np.all(np.abs(T_gpu - act.T) <= tb), f"T max excess {np.max(np.abs(T_gpu - act.T) / tb)}"
        # block exponents: equal except where a block's amax sits within the bound of a power of two
        ediff = te_gpu != act.te
        assert np.all(np.abs(te_gpu.astype(int) - act.te.astype(int)) <= 1)
        # a block exponent may differ only where the block's largest |T| sits within the bound of a power of two
        if ediff.any():
            bm = np.abs(act.T.astype(np.float64)).reshape(Mo, -1, 32)
            amax, amax_b = bm.max(axis=2), np.take_along_axis(tb.reshape(Mo, -1, 32), bm.argmax(axis=2)[:, :, None], axis=2)[:, :, 0]
            p2 = np.exp2(np.round(np.log2(np.maximum(amax, 1e-300))))
            assert np.all(np.abs(amax - p2)[ediff] <= amax_b[ediff] * 1.0001), "block exponent differs away from a power of two"
            print(f"[parity mxb] block exponents that differ from the oracle's: {int(ediff.sum())} of {ediff.size}")
        # every GPU element is a correct saturating E4M3 rounding, under the GPU's block scale, of a
        # value within the accumulation bound of the oracle's T
        sc = np.repeat(oracle.e8m0_decode(te_gpu), 32, axis=1)
        u = np.abs(act.T.astype(np.float64)) / sc
        step = np.exp2(np.maximum(np.floor(np.log2(np.maximum(u, 2.0 ** (min_exp - 1)))) - 3, min_exp))
        half = np.where(u > top, u - top, 0.5 * step * (1 + 1e-6))
        deq = f8[tq_gpu].astype(np.float64) * sc
        assert np.all(np.abs(deq - act.T) <= sc * half + tb), "tq8 is not a block rounding of T"
        same = ~ediff.repeat(32, axis=1)
        diff = (f8[tq_gpu] != f8[act.tq8]) & same
        # under equal block scales a code may differ from the oracle's only where T sits within the accumulation bound
        # of a rounding boundary (the check above bounds every element; the end-to-end comparison below bounds the
        # distance of the two dequantised intermediates).  The count is reported.
        if diff.any():
            print(f"[parity mxb] re-quantised codes that differ from the oracle's: {int(diff.sum())} of {diff.size}")
    # ---- forward: the oracle is fed the GPU's re-quantised intermediate
    act_g = dataclasses.replace(act, tq8=np.ascontiguousarray(tq_gpu), te=np.ascontiguousarray(te_gpu))
    out = oracle.fwd_mxb(pk, act_g)
    y_gpu = n(g.fdbg.y32)[sel]
    Xd = np.abs(E2M1[act.xc].astype(np.float64).reshape(Mo, -1, 32)) * oracle.e8m0_decode(act.xe)[:, :, None]
    Wd = np.abs(E2M1[pk.pc].astype(np.float64).reshape(layer.N, -1, 32)) * oracle.e8m0_decode(pk.pe)[:, :, None]
    A = Xd.reshape(Mo, -1) @ Wd.reshape(layer.N, -1).T
    if r:
        Td = np.abs(f8[tq_gpu].astype(np.float64).reshape(Mo, -1, 32)) * oracle.e8m0_decode(te_gpu)[:, :, None]
        Ld = np.abs(f8[pk.l8].astype(np.float64).reshape(layer.N, -1, 32)) * oracle.e8m0_decode(pk.le)[:, :, None]
        A = A + Td.reshape(Mo, -1) @ Ld.reshape(layer.N, -1).T
    bound = ACC * A + 1e-300
    assert np.all(np.abs(y_gpu - out.y32) <= bound), f"y32 max excess {np.max(np.abs(y_gpu - out.y32) / bound)}"
    Yb = bf16_to_bits(g.Y)[sel]
    check_bf16_against_oracle(oracle, Yb, y_gpu, out, bound, " mxb")
    # ---- end to end: the oracle alone (its own T, block exponents and codes)
    if r:
        out_alone = oracle.fwd_mxb(pk, act)
        sc_o = np.repeat(oracle.e8m0_decode(act.te), 32, axis=1)
        deq_o = f8[act.tq8].astype(np.float64) * sc_o
        D = np.abs(deq - deq_o)
        uo = np.abs(act.T.astype(np.float64)) / sc_o
        step_o = np.exp2(np.maximum(np.floor(np.log2(np.maximum(uo, 2.0 ** (min_exp - 1)))) - 3, min_exp))
        half_o = np.where(uo > top, uo - top, 0.5 * step_o * (1 + 1e-6))
        assert np.all(D <= sc * half + sc_o * half_o + tb), "intermediates further apart than two half steps"
        Labs = (np.abs(f8[pk.l8].astype(np.float64).reshape(layer.N, -1, 32)) * oracle.e8m0_decode(pk.le)[:, :, None]).reshape(layer.N, -1)
        To = (np.abs(deq_o).reshape(Mo, -1)) @ Labs.T
        Am = Xd.reshape(Mo, -1) @ Wd.reshape(layer.N, -1).T
        check_end_to_end(oracle, Yb, y_gpu, out_alone, ACC * (Am + To) + 1e-300, D, Labs, " mxb")
    g2 = run_gpu(layer, X, W, L, R, debug=False, gamma=gamma)
    assert torch.equal(g2.Y, g.Y)
    return g


SMALL = [
    # M (ragged), K (multiple of 128), N (partial 256-wide tile), r (multiple of 32), x_dtype
    (300, 256, 320, 32, "bf16"),
    (77, 384, 64, 32, "f32"),
    (130, 1152, 192, 64, "bf16"),
    (100, 2240, 128, 64, "bf16"),     # 35 chunks of 64: the 2240-wide transformer; one padding chunk in the layouts
    (70, 192, 64, 32, "f32"),
    (64, 128, 64, 0, "bf16"),
    (33, 640, 128, 128, "bf16"),
    (1, 128, 64, 32, "f32"),
    (50, 256, 64, 96, "bf16"),     # a 6-bit budget of 512 bits per channel gives rank 85: padded to three blocks of 32
    (31, 64, 768, 96, "bf16"),     # rank > K: the factor views are larger than N x K
    (255, 192, 256, 0, "f32"),     # rank 0: no branch section of either blob is read (they may hold anything)
    (128, 384, 1344, 0, "f32"),
]


@pytest.mark.parametrize("elem", [8, 6])
@pytest.mark.parametrize("M,K,N,r,xd", SMALL)
def test_small_shapes(oracle, M, K, N, r, xd, elem):
    layer = wl.Layer("t", M, K, N, r, "mxb", 32, elem, elem, xd, seed=M + K)
    X, W, L, R = wl.make_inputs(layer)
    _compare(oracle, layer, X, W, L, R)


@pytest.mark.parametrize("elem", [8, 6])
def test_large_k_and_rank(oracle, elem):
    """K beyond the register-resident row of the fp32-scaled MX activation kernel, rank 128, fp32 input."""
    layer = wl.Layer("t", 40, 5120, 64, 128, "mxb", 32, elem, elem, "f32", seed=9)
    X, W, L, R = wl.make_inputs(layer)
    _compare(oracle, layer, X, W, L, R)


@pytest.mark.parametrize("elem", [8, 6])
def test_degenerate_inputs(oracle, elem):
    layer = wl.Layer("t", 70, 256, 64, 32, "mxb", 32, elem, elem, "bf16", seed=3)
    X, W, L, R = wl.make_inputs(layer)
    X[3] = 0.0
    X[5, :] = 0.0
    X[5, 7] = -2.0
    X[9, 32:64] = 0.0
    W[2] = 0.0
    W[4, 64:96] = 0.0
    L[4] = 0.0
    R[1] = 0.0
    _compare(oracle, layer, X, W, L, R)
    _compare(oracle, layer, np.zeros_like(X), W, L, R)


@pytest.mark.parametrize("elem", [8, 6])
def test_wide_dynamic_range_blocks(oracle, elem):
    layer = wl.Layer("t", 64, 256, 64, 32, "mxb", 32, elem, elem, "bf16", seed=5)
    X, W, L, R = wl.make_inputs(layer)
    rng = np.random.default_rng(7)
    X *= wl.round_to_bf16(np.exp2(rng.integers(-20, 20, size=(64, 8)).repeat(32, axis=1)).astype(np.float32))
    W *= np.exp2(rng.integers(-10, 10, size=(64, 8)).repeat(32, axis=1)).astype(np.float32)
    R *= np.exp2(rng.integers(-6, 6, size=(32, 8)).repeat(32, axis=1)).astype(np.float32)
    _compare(oracle, layer, wl.round_to_bf16(X), W, L, R)


@pytest.mark.parametrize("elem", [8, 6])
@pytest.mark.parametrize("r,first", [(32, 0), (32, 1), (64, 0), (96, 2), (128, 0)])
def test_packed_codes_over_the_whole_range_of_factor_scales(oracle, r, first, elem):
    """Blocks of R with the largest scale bytes against blocks of L with the smallest (0: 2^-127), the other way round, and between;
    K with a padding chunk."""
    from paper_2604_18117_amd import binding as lq
    N, K = 128, 320
    rng = np.random.default_rng(r + first)
    W, L, R = (rng.standard_normal(s).astype(np.float32) for s in ((N, K), (N, r), (r, K)))
    for b in range(r // 32):
        eR, eL = [(125, -131), (-131, 125), (60, -66), (0, -6)][(first + b) % 4]
        R[32 * b:32 * b + 32] *= np.float32(2.0 ** eR)
        L[:, 32 * b:32 * b + 32] *= np.float32(2.0 ** eL)
    cfg = lq.make_config(N, K, r, "mxb", 32, elem, elem)
    got = lq.lq_unpack_weights(cfg, lq.lq_pack_weights(cfg, *(torch.from_numpy(a).cuda() for a in (W, L, R))))
    pk = oracle.pack_mxb(W, L, R, elem=elem)
    assert pk.re.max() > 230 or pk.le.max() > 230
    f8 = oracle.mxb_decode(np.arange(256, dtype=np.uint8), elem)
    for name, want in (("le", pk.le), ("re", pk.re), ("pe", pk.pe)):
        assert np.array_equal(n(getattr(got, name)), want), name
    for name, want, val in (("lq", pk.l8, f8), ("rq", pk.r8, f8), ("pq", pk.pc, E2M1)):
        assert np.array_equal(val[n(getattr(got, name)).view(np.uint8)], val[want]), name


# Blocks of X at both ends of the scale bytes, in each form of the activation step's kernel.  Low: byte 0 (a subnormal 2^-127 as the converters' operand), with subnormal values, largest
# magnitudes on both sides of where each format leaves byte 0, saturating values, and blocks of the smallest numbers; high: up to byte 246 (254 less the 8 of E4M3's
# largest exponent; 252 with E2M3 and for the main codes).  The factors are scaled the other way so that T and Y are normal numbers.
@pytest.mark.parametrize("elem", [8, 6])
@pytest.mark.parametrize("end", ["low", "high"])
@pytest.mark.parametrize("M,K,r,xd,smooth", [(40, 1152, 32, "bf16", False), (70, 1088, 128, "bf16", False), (4100, 192, 32, "bf16", False), (40, 1152, 64, "f32", False),
                                             (40, 1152, 64, "bf16", True)])
def test_codes_of_x_at_the_ends_of_its_range(oracle, M, K, r, xd, smooth, end, elem):
    layer = wl.Layer("t", M, K, 64, r, "mxb", 32, elem, elem, xd, seed=M + K)
    X, W, L, R = wl.make_inputs(layer)
    rng = np.random.default_rng(elem + K)
    blocks = X.reshape(M, K // 32, 32)
    blocks /= np.abs(blocks).max(axis=2, keepdims=True)                  # largest magnitude 1
    low = [-133, -130, -127, -126, -125, -124, -123, -121, -120, -119, -118, -117]
    e = rng.choice(low if end == "low" else [127, 126, 125, 120, 119], size=(M, K // 32, 1))
    top = rng.choice([1.0, 1.5, 1.75, 1.9375, 1.9921875], size=e.shape)  # (the last two saturate in both formats)
    blocks[:] = (blocks * top * np.exp2(e.astype(np.float64))).astype(np.float32)
    if xd == "bf16":
        X = wl.round_to_bf16(X)
    f = np.float32(2.0 ** (100 if end == "low" else -110))
    gamma = np.exp2(rng.integers(0, 4, K) * (-1 if end == "low" else 1)).astype(np.float32) if smooth else None
    rows = None if M < 100 else np.unique(np.concatenate([np.arange(40), np.arange(M - 20, M)]))
    _compare(oracle, layer, X, W * f, L, R * f, rows=rows, gamma=gamma)


@pytest.mark.parametrize("name", ["c5b_qkv", "c5b_fc2", "c5b6_qkv", "c5b6_fc2", "c4m_qkv"])
def test_full_size_sampled_rows(oracle, name):
    layer = wl.LAYERS[name]
    X, W, L, R = wl.make_inputs(layer)
    rng = np.random.default_rng(1)
    rows = np.sort(np.concatenate([[0, layer.M - 1], rng.choice(layer.M, 14, replace=False)]))
    _compare(oracle, layer, X, W, L, R, rows=rows)


# Every form of the activation step (4 or 8 wavefronts, one workgroup per 32 columns of the rank) and every length of a wavefront's run of
# 128-chunks around its unrolled pairs: 3 chunks (a padding one among them) to 41, rows that end inside a group of 16, smoothed or not.
@pytest.mark.parametrize("elem", [8, 6])
@pytest.mark.parametrize("K,r,xd,smooth", [(320, 64, "bf16", False), (704, 128, "bf16", False), (1088, 32, "bf16", False), (2112, 96, "bf16", False), (3200, 64, "bf16", False),
                                           (5184, 32, "bf16", False), (1600, 128, "f32", False), (640, 32, "f32", False), (384, 0, "bf16", False),
                                           (1088, 32, "bf16", True), (2112, 96, "bf16", True), (1600, 128, "bf16", True), (3200, 64, "f32", True), (576, 0, "bf16", True)])
def test_forms_of_the_activation_step(oracle, K, r, xd, smooth, elem):
    from paper_2604_18117_amd import binding as lq
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    layer = wl.Layer("t", 37, K, 64, r, "mxb", 32, elem, elem, xd, seed=K + r)
    X, W, L, R = wl.make_inputs(layer)
    X[2, :] = -0.0                # blocks of zeros have codes 0, also where the zeros are negative
    X[3, 32:64] = -0.0
    X[3, 70] = -0.0               # (in other blocks a zero keeps its sign)
    gamma = np.exp2(np.random.default_rng(K).integers(-3, 4, K)).astype(np.float32) if smooth else None
    _compare(oracle, layer, X, W, L, R, gamma=gamma)
    cfg = lq.config_for_layer(layer, smooth=smooth)
    packed = lq.lq_pack_weights(cfg, *(torch.from_numpy(a).cuda() if r or a is W else None for a in (W, L, R)))
    if smooth:
        lq.lq_set_smoothing(cfg, packed, torch.from_numpy(gamma).cuda())

    def blob(x, debug):
        act = torch.full((lq.lq_act_sizes(cfg, x.shape[0]),), 0xFF, dtype=torch.uint8, device="cuda")
        return lq.lq_quantize_act(cfg, packed, x, act=act, debug=debug)[0] if debug else lq.lq_quantize_act(cfg, packed, x, act=act)

    def views(x, act):
        v = lq.lq_unpack_act(cfg, act, x.shape[0])
        return (v.xq, v.xe, v.tq, v.te) if r else (v.xq, v.xe)
    Xd = wl.to_dev_x(X, xd)
    want = blob(Xd, False)
    assert torch.equal(want, blob(Xd, True))                           # with and without the parity taps
    assert not bool(views(Xd, want)[0][2].any()) and not bool(views(Xd, want)[0][3, 32:64].any())
    wide = torch.full((37, K + 64), float("nan"), dtype=Xd.dtype, device="cuda")
    wide[:, :K] = Xd
    assert torch.equal(blob(wide[:, :K], False), want)                 # rows further apart than K
    for groups in (cus // 4 + 1, cus // 2 + 1, cus, cus + 1):
        M = 16 * groups - 3
        big = Xd.repeat((M + 36) // 37, 1)[:M].contiguous()
        for a, b in zip(views(big, blob(big, False)), views(Xd, want)):   # every row
            assert torch.equal(a, b.repeat((M + 36) // 37, 1)[:M]), M


# Rows of few 128-chunks have kernels of their own: lengths on both sides of their lines (7 chunks with four wavefronts, 8 with eight), one chunk to a
# workgroup, an odd number of 64-chunks.  The kernels with parity taps, which the tests above check against the oracle, are the looped ones at every length: same bytes.
@pytest.mark.parametrize("elem", [8, 6])
@pytest.mark.parametrize("r,xd,smooth", [(0, "bf16", False), (32, "f32", True), (64, "bf16", False), (96, "f32", False), (128, "bf16", True)])
def test_short_rows(r, xd, smooth, elem):
    from paper_2604_18117_amd import binding as lq
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    for K in (64, 128, 192, 512, 640, 832, 896, 960, 1024, 1088):
        layer = wl.Layer("t", 37, K, 64, r, "mxb", 32, elem, elem, xd, seed=K + r)
        X, W, L, R = wl.make_inputs(layer)
        X[2, :] = -0.0
        cfg = lq.config_for_layer(layer, smooth=smooth)
        packed = lq.lq_pack_weights(cfg, *(torch.from_numpy(a).cuda() if r or a is W else None for a in (W, L, R)))
        if smooth:
            lq.lq_set_smoothing(cfg, packed, torch.from_numpy(np.random.default_rng(K).uniform(0.5, 2, K).astype(np.float32)).cuda())
        Xd = wl.to_dev_x(X, xd)
        for M in (37, 16 * (cus // 2) + 5, 16 * cus + 5):                 # eight wavefronts, a workgroup per 32 columns of the rank, four
            big = Xd.repeat((M + 36) // 37, 1)[:M].contiguous()
            act, tap = [torch.full((lq.lq_act_sizes(cfg, M),), 0xFF, dtype=torch.uint8, device="cuda") for _ in range(2)]
            lq.lq_quantize_act(cfg, packed, big, act=act)
            lq.lq_quantize_act(cfg, packed, big, act=tap, debug=True)
            assert torch.equal(act, tap), (K, M)
