"""GPU parity, MXI family (MXINT4 main on the 6-bit scaled MFMA, MXINT8 / MXINT4 branch on the bf16
MFMA; integer MX formats of App. A.3, integer rows of the tables of Section 4.3) against the CPU oracle.

Bar: every code and E8M0 byte computed from source data (X, P, L, R) bit-exact; products are exact on
both sides, so the only difference is the matrix core's fp32 accumulation across blocks against the
oracle's fp64: the intermediate T and the output are bounded by 2^-13 of the sum of the magnitudes of
their terms (the same bound as for the other block-scaled family), and are bit-exact where every
partial sum is exactly representable (uniform block scales); the re-quantised intermediate must be a
correct block quantisation of a value within that bound of the oracle's T.
"""
import dataclasses

import numpy as np
import pytest
import torch

from paper_2604_18117_amd import workloads as wl
from tests.gpu_util import bf16_to_bits, check_bf16_against_oracle, check_end_to_end, n, run_gpu

pytestmark = pytest.mark.gpu

# fp32 accumulation inside the scaled / bf16 matrix instructions against the oracle's fp64 sum: at most this fraction of the
# sum of |terms| (measured worst case over every committed and swept case: 2^-14.9; the bar leaves a factor 1.9)
ACC = 2.0 ** -14


def _vals(oracle, codes, ebytes, bits):
    """|value| of MXINT elements: rows x (blocks x 32)."""
    rows = codes.shape[0]
    return (np.abs(codes.astype(np.float64)).reshape(rows, -1, 32) * oracle.mxint_scale(ebytes, bits)[:, :, None]).reshape(rows, -1)


def _compare(oracle, layer, X, W, L, R, rows=None, exact=False, gamma=None):
    g = run_gpu(layer, X, W, L, R, debug=True, debug_acc=False, gamma=gamma)
    Xo = X if rows is None else X[rows]
    if gamma is not None:                       # fused smoothing: the oracle quantises the smoothed input
        Xo = oracle.smooth(Xo, gamma)
    sel = slice(None) if rows is None else rows
    r, bw = layer.r, layer.br_w_bits
    pk = oracle.pack_mxi(W, L if r else None, R if r else None, bw)
    act = oracle.quantize_act_mxi(Xo, pk)
    Mo = Xo.shape[0]
    # ---- offline packing: exact
    assert np.array_equal(n(g.wv.pq), pk.pq), "pq"
    assert np.array_equal(n(g.wv.pe), pk.pe), "pe"
    if r:
        assert np.array_equal(n(g.wv.lq), pk.lq), "lq"
        assert np.array_equal(n(g.wv.le), pk.le), "le"
        assert np.array_equal(n(g.wv.rq), pk.rq), "rq"
        assert np.array_equal(n(g.wv.re), pk.re), "re"
    # ---- activation step: codes and block scales from X exact
    assert np.array_equal(n(g.av.xq)[sel], act.xq), "xq"
    assert np.array_equal(n(g.av.xe)[sel], act.xe), "xe"
    tq_gpu = n(g.av.tq)[sel] if r else np.zeros((Mo, 0), np.int8)
    te_gpu = n(g.av.te)[sel] if r else np.zeros((Mo, 0), np.uint8)
    if r:
        assert np.array_equal(n(g.adbg.xb)[sel], act.xb), "xb"
        assert np.array_equal(n(g.adbg.xbe)[sel], act.xbe), "xbe"
        T_gpu = n(g.adbg.T)[sel]
        tb = ACC * (_vals(oracle, act.xb, act.xbe, 8) @ _vals(oracle, pk.rq, pk.re, bw).T) + 1e-300
        assert np.all(np.abs(T_gpu - act.T) <= tb), f"T max excess {np.max(np.abs(T_gpu - act.T) / tb)}"
        ediff = te_gpu != act.te
        assert np.all(np.abs(te_gpu.astype(int) - act.te.astype(int)) <= 1)
        # a block exponent may differ only where the block's largest |T| sits within the bound of a power of two
        if ediff.any():
            bm = np.abs(act.T.astype(np.float64)).reshape(Mo, -1, 32)
            amax, amax_b = bm.max(axis=2), np.take_along_axis(tb.reshape(Mo, -1, 32), bm.argmax(axis=2)[:, :, None], axis=2)[:, :, 0]
            p2 = np.exp2(np.round(np.log2(np.maximum(amax, 1e-300))))
            assert np.all(np.abs(amax - p2)[ediff] <= amax_b[ediff] * 1.0001), "block exponent differs away from a power of two"
            print(f"[parity mxi] block exponents that differ from the oracle's: {int(ediff.sum())} of {ediff.size}")
        # every GPU element is a correct saturating rounding, on the GPU's block grid, of a value within
        # the accumulation bound of the oracle's T
        step = np.repeat(oracle.mxint_scale(te_gpu, 8), 32, axis=1)
        u = np.abs(act.T.astype(np.float64)) / step
        half = np.where(u > 127.0, u - 127.0, 0.5 * (1 + 1e-9))
        deq = tq_gpu.astype(np.float64) * step
        assert np.abs(tq_gpu.astype(int)).max() <= 127
        assert np.all(np.abs(deq - act.T) <= step * half + tb), "tq is not a block rounding of T"
        same = ~ediff.repeat(32, axis=1)
        diff = (tq_gpu != act.tq) & same
        # under equal block scales a code may differ from the oracle's only where T sits within the accumulation bound
        # of a rounding boundary (the check above bounds every element; the end-to-end comparison below bounds the
        # distance of the two dequantised intermediates).  The count is reported.
        if diff.any():
            print(f"[parity mxi] re-quantised codes that differ from the oracle's: {int(diff.sum())} of {diff.size}")
        if exact:
            assert np.array_equal(T_gpu, act.T) and np.array_equal(tq_gpu, act.tq) and np.array_equal(te_gpu, act.te)
    # ---- forward: the oracle is fed the GPU's re-quantised intermediate
    act_g = dataclasses.replace(act, tq=np.ascontiguousarray(tq_gpu), te=np.ascontiguousarray(te_gpu))
    out = oracle.fwd_mxi(pk, act_g)
    y_gpu = n(g.fdbg.y32)[sel]
    A = _vals(oracle, act.xq, act.xe, 4) @ _vals(oracle, pk.pq, pk.pe, 4).T
    if r:
        A = A + _vals(oracle, tq_gpu, te_gpu, 8) @ _vals(oracle, pk.lq, pk.le, bw).T
    bound = ACC * A + 1e-300
    assert np.all(np.abs(y_gpu - out.y32) <= bound), f"y32 max excess {np.max(np.abs(y_gpu - out.y32) / bound)}"
    if exact:
        assert np.array_equal(y_gpu, out.y32), "y32 (exactly representable partial sums)"
    Yb = bf16_to_bits(g.Y)[sel]
    check_bf16_against_oracle(oracle, Yb, y_gpu, out, bound, " mxi")
    # ---- end to end: the oracle alone (its own T, block exponents and codes)
    if r:
        out_alone = oracle.fwd_mxi(pk, act)
        step_o = np.repeat(oracle.mxint_scale(act.te, 8), 32, axis=1)
        deq_o = act.tq.astype(np.float64) * step_o
        D = np.abs(deq - deq_o)
        uo = np.abs(act.T.astype(np.float64)) / step_o
        half_o = np.where(uo > 127.0, uo - 127.0, 0.5 * (1 + 1e-9))
        assert np.all(D <= step * half + step_o * half_o + tb), "intermediates further apart than two half steps"
        Labs = _vals(oracle, pk.lq, pk.le, bw)
        Am = _vals(oracle, act.xq, act.xe, 4) @ _vals(oracle, pk.pq, pk.pe, 4).T
        check_end_to_end(oracle, Yb, y_gpu, out_alone, ACC * (Am + np.abs(deq_o) @ Labs.T) + 1e-300, D, Labs, " mxi")
    g2 = run_gpu(layer, X, W, L, R, debug=False, gamma=gamma)
    assert torch.equal(g2.Y, g.Y)
    return g


SMALL = [
    # M (ragged), K (multiple of 64), N (partial 256-wide tile), r (multiple of 32), branch weight bits, x_dtype
    (300, 256, 320, 32, 8, "bf16"),
    (77, 320, 64, 32, 4, "f32"),
    (130, 1152, 192, 64, 8, "bf16"),
    (64, 64, 64, 0, 8, "bf16"),
    (33, 704, 128, 128, 4, "bf16"),
    (1, 128, 64, 32, 8, "f32"),
    (257, 576, 512, 64, 8, "bf16"),
    (40, 5120, 64, 32, 8, "bf16"),      # K beyond what the row-resident activation kernels of the other families take
    (18, 2368, 64, 64, 4, "f32"),
    (50, 256, 64, 96, 8, "bf16"),
    (97, 64, 384, 128, 8, "bf16"),      # rank > K: the factor views are larger than N x K
    (15, 64, 320, 96, 4, "f32"),
    (255, 192, 256, 0, 8, "f32"),       # rank 0: no branch section of either blob is read
]


@pytest.mark.parametrize("M,K,N,r,bw,xd", SMALL)
def test_small_shapes(oracle, M, K, N, r, bw, xd):
    layer = wl.Layer("t", M, K, N, r, "mxi", 32, bw, 8, xd, seed=M + K)
    X, W, L, R = wl.make_inputs(layer)
    _compare(oracle, layer, X, W, L, R)


def test_uniform_scales_are_bit_exact(oracle):
    """All blocks share one scale per operand and every partial sum stays below 2^24 code units:
    the fp32 accumulators hold the integer contractions exactly, so nothing may differ."""
    M, K, N, r = 96, 384, 128, 32
    layer = wl.Layer("t", M, K, N, r, "mxi", 32, 8, 8, "bf16", seed=11)
    rng = np.random.default_rng(11)
    X = (rng.integers(-7, 8, size=(M, K)) / 4.0).astype(np.float32); X[:, 0::32] = 1.75
    W = (rng.integers(-7, 8, size=(N, K)) / 64.0).astype(np.float32); W[:, 1::32] = 7 / 64.0
    R = (rng.integers(-3, 4, size=(r, K)) / 256.0).astype(np.float32); R[:, 2::32] = 1 / 64.0
    L = np.zeros((N, r), np.float32); L[:, 0] = rng.integers(-5, 6, size=N) / 16.0; L[:, 5] = 1.0
    _compare(oracle, layer, X, W, L, R, exact=True)


def test_degenerate_inputs(oracle):
    layer = wl.Layer("t", 70, 256, 64, 32, "mxi", 32, 8, 8, "bf16", seed=3)
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


def test_wide_dynamic_range_blocks(oracle):
    layer = wl.Layer("t", 64, 256, 64, 32, "mxi", 32, 8, 8, "bf16", seed=5)
    X, W, L, R = wl.make_inputs(layer)
    rng = np.random.default_rng(7)
    X *= wl.round_to_bf16(np.exp2(rng.integers(-20, 20, size=(64, 8)).repeat(32, axis=1)).astype(np.float32))
    W *= np.exp2(rng.integers(-10, 10, size=(64, 8)).repeat(32, axis=1)).astype(np.float32)
    R *= np.exp2(rng.integers(-6, 6, size=(32, 8)).repeat(32, axis=1)).astype(np.float32)
    _compare(oracle, layer, wl.round_to_bf16(X), W, L, R)


@pytest.mark.parametrize("name", ["c5i_qkv", "c5i_fc2", "c5i4_attn_out"])
def test_full_size_sampled_rows(oracle, name):
    layer = wl.LAYERS[name]
    X, W, L, R = wl.make_inputs(layer)
    rng = np.random.default_rng(1)
    rows = np.sort(np.concatenate([[0, layer.M - 1], rng.choice(layer.M, 14, replace=False)]))
    _compare(oracle, layer, X, W, L, R, rows=rows)


# rows per workgroup of the activation step: 16, and where there is R enough (rank times K) 32 and 64 in batches that fill most of the device;
# last workgroup partly or wholly past M
@pytest.mark.parametrize("M,K,r,bw,xd", [(6143, 320, 64, 8, "bf16"), (6113, 320, 64, 8, "bf16"), (12281, 448, 128, 4, "bf16"), (12289, 64, 96, 8, "f32"),
                                         (12287, 576, 32, 8, "bf16"), (6150, 1152, 96, 8, "f32"),
                                         (13281, 1152, 128, 8, "bf16"), (13345, 1600, 96, 4, "f32"), (5130, 2304, 128, 8, "bf16"),
                                         (5101, 2240, 96, 4, "f32"), (14337, 2304, 64, 8, "bf16"), (14001, 4608, 32, 8, "bf16")])
def test_activation_row_forms(oracle, M, K, r, bw, xd):
    layer = wl.Layer("t", M, K, 64, r, "mxi", 32, bw, 8, xd, seed=M + r)
    X, W, L, R = wl.make_inputs(layer)
    rows = np.unique(np.concatenate([np.arange(M - 70, M), np.arange(40), np.arange(0, M, 997)]))
    _compare(oracle, layer, X, W, L, R, rows=rows)


# Forms of the forward by the number of 32 x 32 tiles: 1 x 1 to 1400, 2 x 1 to 3600, 2 x 2 to a line between 4000 and 8000 that depends on the
# rows' length, the hand-off and the number of large tiles, 128 x 256 tiles above; ragged M, an odd
# number of row blocks, fewer and more quads of chunks than are kept in flight, last quads of one to four chunks.
@pytest.mark.parametrize("M,K,N,r,bw", [(790, 1152, 1664, 32, 8), (397, 704, 4032, 64, 4), (1130, 320, 2176, 128, 8), (1700, 448, 2176, 96, 4),
                                        (2300, 64, 2112, 64, 8), (3300, 576, 2176, 32, 8), (401, 2240, 4032, 0, 8)])
def test_forward_forms(oracle, M, K, N, r, bw):
    layer = wl.Layer("t", M, K, N, r, "mxi", 32, bw, 8, "bf16", seed=M + N)
    X, W, L, R = wl.make_inputs(layer)
    rows = np.unique(np.concatenate([np.arange(M - 40, M), np.arange(0, M, 61)]))
    _compare(oracle, layer, X, W, L, R, rows=rows)


@pytest.mark.parametrize("M,K,N,r,bw", [(3845, 128, 1856, 32, 8), (3901, 192, 1920, 64, 4), (3840, 320, 1984, 96, 8), (3930, 832, 1728, 128, 8),
                                        (3969, 832, 1728, 128, 8)])
def test_last_column_of_large_layers(oracle, M, K, N, r, bw):
    """More tiles than the small form takes, a last column of 64, 128 or 192 channels (the first two as 2 x 2 wavefronts) and a last row of
    tiles of one to four row blocks."""
    layer = wl.Layer("t", M, K, N, r, "mxi", 32, bw, 8, "bf16", seed=M)
    _compare(oracle, layer, *wl.make_inputs(layer))


# The large tiles' loop takes its chunks in groups of eight and every shorter tail by calls of its own: 4, 6 and 7 chunks and 8 + 4, 8 + 6, 8 + 7
# (the others are in the cases above); rank 0, and layers of which the last column is all there is.
@pytest.mark.parametrize("M,K,N,r,bw", [(3845, 256, 1856, 0, 8), (3901, 384, 1920, 128, 4), (3841, 448, 1984, 96, 8), (3841, 768, 1984, 32, 8),
                                        (6989, 896, 960, 0, 8), (6989, 960, 960, 64, 4), (56001, 448, 128, 32, 8), (128100, 64, 64, 128, 4),
                                        (128100, 256, 64, 0, 8)])
def test_large_tiles_tails_and_ranks(oracle, M, K, N, r, bw):
    layer = wl.Layer("t", M, K, N, r, "mxi", 32, bw, 8, "bf16", seed=M + K)
    rows = np.unique(np.concatenate([np.arange(M - 140, M), np.arange(130), np.arange(0, M, 61)]))
    _compare(oracle, layer, *wl.make_inputs(layer), rows=rows)


def test_rows_as_long_as_the_contract_allows():
    """K = 2^24 at rank 128: the dequantised R is 4 GB.  Everything but the last chunk of X and R is zero, so the intermediate
    is that of the last chunk alone: the codes of a layer with K = 64."""
    from paper_2604_18117_amd import binding as lq
    M, K, N, r = 3, 1 << 24, 64, 128
    g = torch.Generator(device="cuda")
    g.manual_seed(7)
    x = torch.randn((M, 64), generator=g, device="cuda").to(torch.bfloat16)
    Rs = torch.randn((r, 64), generator=g, device="cuda")
    L = torch.randn((N, r), generator=g, device="cuda")

    def layer(k):
        cfg = lq.make_config(N, k, r, "mxi", 32, 8, 8)
        X, R, W = (torch.zeros(s, dtype=t, device="cuda") for s, t in (((M, k), torch.bfloat16), ((r, k), torch.float32), ((N, k), torch.float32)))
        X[:, -64:], R[:, -64:] = x, Rs
        packed = lq.lq_pack_weights(cfg, W, L, R)
        del R, W
        act = lq.lq_quantize_act(cfg, packed, X)
        # the step from codes, on the codes the activation step rounds X to
        codes = torch.zeros(lq.lq_handoff_sizes(cfg, M), dtype=torch.uint8, device="cuda")
        blocks = X.float().view(M, k // 32, 32)
        e = torch.frexp(blocks.abs().amax(2))[1].to(torch.int32) - 1
        q = torch.round(torch.ldexp(blocks, 6 - e[..., None])).clamp(-127, 127).to(torch.int8)
        q[blocks.abs().amax(2) == 0] = 0
        codes[:M * k] = q.view(torch.uint8).reshape(-1)
        scales = codes[codes.numel() - (32 * (k // 32) + 255) // 256 * 256:]
        scales[:M * (k // 32)] = torch.where(blocks.abs().amax(2) == 0, 0, e + 127).to(torch.uint8).reshape(-1)
        from_codes = lq.lq_branch_from_codes(cfg, packed, codes, M, torch.full_like(act, 0xFF))
        views = [lq.lq_unpack_act(cfg, a, M) for a in (act, from_codes)]
        torch.cuda.synchronize()
        return [(v.tq.cpu(), v.te.cpu()) for v in views]

    want = layer(64)[0]
    assert want[0].any()
    for got in layer(K):
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])


@pytest.mark.parametrize("fam,g,bw,ag,r", [("mxi", 32, 8, 32, 128), ("mxi", 32, 4, 32, 64), ("mxi", 32, 8, 32, 32), ("mx", 32, 8, 32, 64),
                                           ("mxb", 32, 8, 32, 128), ("mxb", 32, 6, 32, 64), ("int", 64, 8, 0, 64), ("int", 64, 6, 64, 32)])
def test_a_token_does_not_depend_on_its_batch(fam, g, bw, ag, r):
    """A token's codes and outputs are the same bits in every batch, whatever form of the kernels the batch size takes.  Block scales spread
    over 2^+-10, so that the fp32 sums of the intermediate round."""
    from paper_2604_18117_amd import binding as lq
    M, K, N = 14300, 2304, 576  # (past the small forms in every family)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(r + bw)

    def spread(rows, cols):
        e = torch.randint(-10, 11, (rows, cols // 32, 1), generator=gen, device="cuda")
        return torch.ldexp(torch.randn((rows, cols // 32, 32), generator=gen, device="cuda"), e).reshape(rows, cols)
    cfg = lq.make_config(N, K, r, fam, g, bw, bw if fam == "mxb" else 8, a_group=ag)
    packed = lq.lq_pack_weights(cfg, spread(N, K) * 0.02, torch.randn((N, r), generator=gen, device="cuda"), spread(r, K))
    X = spread(M, K).to(torch.bfloat16)

    def run(m):
        act = lq.lq_quantize_act(cfg, packed, X[:m])
        v = lq.lq_unpack_act(cfg, act, m)
        Y = lq.lq_linear_lowrank_fwd(cfg, packed, act, m)
        parts = [v.tq, v.st, v.te, Y.view(torch.int16)]
        if fam == "mxi":  # the step from codes too: those that a producer with this output would leave
            blocks = X[:m].float().view(m, K // 32, 32)
            e = torch.frexp(blocks.abs().amax(2))[1].to(torch.int32) - 1
            codes = torch.zeros(lq.lq_handoff_sizes(cfg, m), dtype=torch.uint8, device="cuda")
            codes[:m * K] = torch.round(torch.ldexp(blocks, 6 - e[..., None])).clamp(-127, 127).to(torch.int8).view(torch.uint8).reshape(-1)
            mp = (m + 31) // 32 * 32
            codes[(mp * K + 255) // 256 * 256:][:m * (K // 32)] = (e + 127).to(torch.uint8).reshape(-1)
            vc = lq.lq_unpack_act(cfg, lq.lq_branch_from_codes(cfg, packed, codes, m, torch.zeros_like(act)), m)
            assert torch.equal(vc.tq, v.tq) and torch.equal(vc.te, v.te)
        return parts
    whole = run(M)
    for m in (5, 300, 2000, 6200, 8300):
        for name, a, b in zip(("tq", "st", "te", "Y"), run(m), whole):
            assert torch.equal(a, b[:m]), (m, name)


# Layers narrow and wide, long and short: each order of the small forms' tiles, and the large tiles beside them (by the number of tiles, at
# three and four chunks, above 80 MB of X codes, more large tiles than compute units)
@pytest.mark.parametrize("fam,g,bw,ag,K,N,ms", [("mx", 32, 8, 32, 4608, 64, (33, 700, 20011, 36001)), ("mxb", 32, 6, 32, 576, 192, (40, 9001, 19000)),
                                                ("mxi", 32, 8, 32, 1152, 192, (65, 5000, 37333, 42600, 42700)), ("mxi", 32, 8, 32, 896, 320, (40, 16600, 22401, 25600, 25700)),
                                                ("mxi", 32, 4, 32, 896, 1152, (33, 5700, 5762)), ("mxi", 32, 8, 32, 2240, 128, (65, 39000, 46400, 46500)),
                                                ("mxi", 32, 8, 32, 64, 64, (33, 112100, 128000, 128100)), ("int", 128, 4, 0, 256, 1152, (70, 900, 2939, 4000, 4700)),
                                                ("int", 64, 8, 0, 512, 128, (97, 6500, 40000, 41000)), ("int", 64, 6, 64, 192, 4480, (33, 420, 1601, 1700))])
def test_outputs_do_not_depend_on_the_tiles(fam, g, bw, ag, K, N, ms):
    from paper_2604_18117_amd import binding as lq
    r = 64
    gen = torch.Generator(device="cuda")
    gen.manual_seed(K + N)
    cfg = lq.make_config(N, K, r, fam, g, bw, bw if fam == "mxb" else 8, a_group=ag)
    W, L, R = (torch.randn(s, generator=gen, device="cuda") * f for s, f in (((N, K), 0.02), ((N, r), 0.1), ((r, K), 0.1)))
    packed = lq.lq_pack_weights(cfg, W, L, R)
    X = (torch.randn((ms[-1], K), generator=gen, device="cuda") * torch.exp2(torch.randint(-8, 9, (1, K), generator=gen, device="cuda"))).to(torch.bfloat16)
    Y = [lq.lq_linear_lowrank_fwd(cfg, packed, lq.lq_quantize_act(cfg, packed, X[:m]), m).view(torch.int16) for m in ms]
    for m, y in zip(ms, Y):
        assert torch.equal(y, Y[-1][:m]), m


# Small batches deal a group of 16 rows to a workgroup per 32 columns of the rank: the codes are those of one workgroup per group, from X and from
# codes, on both sides of the line.
@pytest.mark.parametrize("r,K,xd,smooth", [(64, 1152, "bf16", False), (96, 320, "f32", False), (128, 64, "bf16", False), (128, 1600, "bf16", True), (96, 4608, "bf16", False)])
def test_workgroups_per_block_of_the_rank(r, K, xd, smooth):
    from paper_2604_18117_amd import binding as lq
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    gen = torch.Generator(device="cuda")
    gen.manual_seed(r + K)
    W, L, R = (torch.randn(s, generator=gen, device="cuda") * f for s, f in (((64, K), 0.02), ((64, r), 0.1), ((r, K), 0.1)))
    cfg = lq.make_config(64, K, r, "mxi", 32, 8, x_dtype=xd, smooth=smooth)
    packed = lq.lq_pack_weights(cfg, W, L, R)
    if smooth:
        lq.lq_set_smoothing(cfg, packed, torch.rand(K, generator=gen, device="cuda") + 0.5)
    groups = cus // (r // 32)                               # the last number of groups that are dealt so
    X = torch.randn((16 * groups + 16, K), generator=gen, device="cuda")
    X = X if xd == "f32" else X.bfloat16()
    views = []
    for m in (16 * groups + 16, 16 * groups - 3, 5, 167, 330):   # (the last two: a number of groups that is not a multiple of 8)
        act = lq.lq_quantize_act(cfg, packed, X[:m], act=torch.full((lq.lq_act_sizes(cfg, m),), 0xFF, dtype=torch.uint8, device="cuda"))
        dbg = lq.lq_quantize_act(cfg, packed, X[:m], act=torch.full_like(act, 0xFF), debug=True)[0]
        assert torch.equal(act, dbg), m
        v = lq.lq_unpack_act(cfg, act, m)
        views.append((v.xq, v.xe, v.tq, v.te))
        if not smooth:
            codes = torch.randint(0, 256, (lq.lq_handoff_sizes(cfg, m),), generator=torch.Generator(device="cuda").manual_seed(1), dtype=torch.uint8, device="cuda")
            codes[(((m + 31) // 32 * 32) * K + 255) // 256 * 256:] = 120   # scale bytes
            if m == 16 * groups + 16:
                all_codes = codes
            else:                                           # the same rows
                codes[:m * K] = all_codes[:m * K]
            vc = lq.lq_unpack_act(cfg, lq.lq_branch_from_codes(cfg, packed, codes, m, act.clone()), m)
            views[-1] += (vc.tq, vc.te)
        for a, b in zip(views[-1], views[0]):
            assert torch.equal(a, b[:m]), m
