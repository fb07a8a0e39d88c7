"""Quantized hand-off between two MXINT linears (Section 4.5) on the GPU, through the C-ABI.

Bar: the consumer's activation blob built by the producer's epilogue plus lq_branch_from_codes holds the same codes and
scales, bit for bit, as lq_quantize_act applied to the producer's stored bf16 output (the reading: codes come from the
bf16 value), so the consumer's output is bit-equal too; and the codes equal the CPU oracle's activation step run on that
bf16 output (main codes, branch codes, every block scale: integer decisions on identical inputs, compared exactly)."""
import numpy as np
import pytest
import torch

from paper_2604_18117_amd import workloads as wl
from tests.gpu_util import bf16_to_bits, n

pytestmark = pytest.mark.gpu


def _layer(name, M, K, N, r, bw, seed):
    return wl.Layer(name, M, K, N, r, "mxi", 32, bw, 8, "bf16", seed=seed)


def _pack(lq, layer, W, L, R):
    cfg = lq.config_for_layer(layer)
    d = lambda a: torch.from_numpy(a).cuda()
    return cfg, lq.lq_pack_weights(cfg, d(W), d(L) if layer.r else None, d(R) if layer.r else None)


def _run(oracle, M, K1, N1, N2, r1, r2, bw, seed, with_y):
    from paper_2604_18117_amd import binding as lq
    l1, l2 = _layer("p", M, K1, N1, r1, bw, seed), _layer("c", M, N1, N2, r2, bw, seed + 1)
    X, W1, L1, R1 = wl.make_inputs(l1)
    _, W2, L2, R2 = wl.make_inputs(l2)
    cfg1, pk1 = _pack(lq, l1, W1, L1, R1)
    cfg2, pk2 = _pack(lq, l2, W2, L2, R2)
    act1 = lq.lq_quantize_act(cfg1, pk1, wl.to_dev_x(X, "bf16"))
    # two-call path: bf16 output stored, read back by the consumer's activation step
    Y1 = lq.lq_linear_lowrank_fwd(cfg1, pk1, act1, M)
    act2_ref = lq.lq_quantize_act(cfg2, pk2, Y1)
    Y2_ref = lq.lq_linear_lowrank_fwd(cfg2, pk2, act2_ref, M)
    # hand-off path (blobs start as 0xFF bytes: a section nobody wrote would show)
    act2 = torch.full((lq.lq_act_sizes(cfg2, M),), 0xFF, dtype=torch.uint8, device="cuda")
    codes = torch.full((lq.lq_handoff_sizes(cfg2, M),), 0xFF, dtype=torch.uint8, device="cuda")
    Yh = torch.full((M, N1), -1, dtype=torch.int16, device="cuda").view(torch.bfloat16) if with_y else None
    lq.lq_linear_lowrank_fwd_handoff(cfg1, pk1, act1, M, cfg2, act2, codes, Y=Yh)
    lq.lq_branch_from_codes(cfg2, pk2, codes, M, act2)
    Y2 = lq.lq_linear_lowrank_fwd(cfg2, pk2, act2, M)
    torch.cuda.synchronize()
    if with_y:
        assert torch.equal(Yh, Y1), "the bf16 output written beside the hand-off"
    va, vr = lq.lq_unpack_act(cfg2, act2, M), lq.lq_unpack_act(cfg2, act2_ref, M)
    for f in ("xq", "xe") + (("tq", "te") if r2 else ()):
        assert torch.equal(getattr(va, f), getattr(vr, f)), f"{f}: hand-off differs from lq_quantize_act on the stored output"
    assert torch.equal(Y2, Y2_ref), "the consumer's output"
    # against the oracle's activation step on the same bf16 values
    pk2o = oracle.pack_mxi(W2, L2 if r2 else None, R2 if r2 else None, bw)
    ho = oracle.handoff_mxi(bf16_to_bits(Y1), pk2o)
    assert np.array_equal(n(va.xq), ho.xq) and np.array_equal(n(va.xe), ho.xe), "main codes / scales vs oracle"
    Mp = (M + 31) // 32 * 32
    cb = n(codes[:Mp * N1]).view(np.int8).reshape(Mp, N1)[:M]
    off = (Mp * N1 + 255) // 256 * 256
    cbe = n(codes[off:off + Mp * (N1 // 32)]).reshape(Mp, N1 // 32)[:M]
    if r2:
        assert np.array_equal(cb, ho.xb) and np.array_equal(cbe, ho.xbe), "branch codes / scales vs oracle"
    else:   # (a consumer without a branch: the codes are still those of its activation format)
        ho8 = oracle.handoff_mxi(bf16_to_bits(Y1), oracle.pack_mxi(W2, np.zeros((N2, 32), np.float32), np.zeros((32, N1), np.float32), bw))
        assert np.array_equal(cb, ho8.xb) and np.array_equal(cbe, ho8.xbe)


@pytest.mark.parametrize("M,K1,N1,N2,r1,r2,bw,with_y", [
    (300, 256, 320, 192, 32, 32, 8, False),    # ragged M; N1 = 5 chunks: padding chunks in the consumer's scale layout
    (77, 192, 64, 64, 32, 64, 4, True),
    (130, 576, 512, 128, 64, 32, 8, True),
    (33, 128, 704, 64, 128, 128, 4, False),
    (64, 64, 128, 64, 0, 0, 8, False),          # no branch on either side
    (200, 320, 192, 320, 32, 0, 8, False),
    (1, 128, 64, 64, 32, 32, 8, True),
    (397, 192, 4032, 64, 32, 32, 8, True),      # the producer's 64 x 32 tiles, an odd number of row blocks
    (1700, 320, 2240, 64, 32, 64, 4, True),     # ... and its 64 x 64 tiles
    (6145, 64, 320, 64, 32, 64, 8, False),      # the step from codes on 32-row workgroups
    (12290, 64, 576, 64, 32, 128, 4, False),    # ... and on 64-row workgroups, the last one partly past M
    (16630, 1280, 320, 64, 32, 32, 4, True),    # small tiles where the large ones number more than the compute units: long rows,
    (33850, 64, 192, 64, 32, 32, 8, False),     # ... a last column with one wavefront idle,
    (73590, 768, 64, 64, 32, 32, 8, False),     # ... and two of four
])
def test_handoff_equals_the_two_call_path(oracle, M, K1, N1, N2, r1, r2, bw, with_y):
    _run(oracle, M, K1, N1, N2, r1, r2, bw, 40 + M, with_y)


@pytest.mark.parametrize("M,K1,N1,with_y", [(2085, 128, 2112, False), (1999, 192, 2176, True), (2021, 64, 2240, True)])
def test_handoff_of_large_layers(oracle, M, K1, N1, with_y):
    """Layers past the small form: codes formed in registers, the last column of 64 and 128 channels as 2 x 2 wavefronts."""
    _run(oracle, M, K1, N1, 64, 32, 32, 8, M, with_y)


@pytest.mark.parametrize("M,K1,N1,r1,bw,with_y", [(1210, 576, 3456, 128, 4, False), (1243, 704, 3392, 128, 4, True), (1281, 448, 3264, 96, 8, True),
                                                  (1999, 256, 2176, 0, 8, False), (2021, 384, 2112, 0, 4, True), (32900, 64, 128, 64, 8, True)])
def test_handoff_of_large_layers_by_rank(oracle, M, K1, N1, r1, bw, with_y):
    """... at every depth of the branch's operands in flight, without a branch, with one tile column only."""
    _run(oracle, M, K1, N1, 64, r1, 32, bw, M, with_y)


def test_handoff_degenerate_blocks(oracle):
    """All-zero tokens (scale byte 0, codes 0) and a producer with an all-zero channel block."""
    from paper_2604_18117_amd import binding as lq
    M, K1, N1, N2, r = 70, 128, 128, 64, 32
    l1, l2 = _layer("p", M, K1, N1, r, 8, 5), _layer("c", M, N1, N2, r, 8, 6)
    X, W1, L1, R1 = wl.make_inputs(l1)
    _, W2, L2, R2 = wl.make_inputs(l2)
    X[3] = 0.0
    W1[32:64] = 0.0
    L1[32:64] = 0.0           # outputs 32..63 are exactly zero for every token: an all-zero block of the consumer
    cfg1, pk1 = _pack(lq, l1, W1, L1, R1)
    cfg2, pk2 = _pack(lq, l2, W2, L2, R2)
    act1 = lq.lq_quantize_act(cfg1, pk1, wl.to_dev_x(X, "bf16"))
    Y1 = lq.lq_linear_lowrank_fwd(cfg1, pk1, act1, M)
    act2_ref = lq.lq_quantize_act(cfg2, pk2, Y1)
    act2, codes = lq.lq_linear_lowrank_fwd_handoff(cfg1, pk1, act1, M, cfg2)
    lq.lq_branch_from_codes(cfg2, pk2, codes, M, act2)
    va, vr = lq.lq_unpack_act(cfg2, act2, M), lq.lq_unpack_act(cfg2, act2_ref, M)
    for f in ("xq", "xe", "tq", "te"):
        assert torch.equal(getattr(va, f), getattr(vr, f)), f
    assert not n(va.xq)[:, 32:64].any() and not n(va.xq)[3].any()
    assert torch.equal(lq.lq_linear_lowrank_fwd(cfg2, pk2, act2, M), lq.lq_linear_lowrank_fwd(cfg2, pk2, act2_ref, M))


@pytest.mark.parametrize("M,N1,with_y", [(70, 128, True), (2085, 2112, False), (2085, 2112, True)])
def test_handoff_degenerate_blocks_of_both_forms(oracle, M, N1, with_y):
    """All-zero tokens (scale byte 0, codes 0), tokens near both ends of the range, and a producer with an all-zero channel block; in
    the small form and in the large tiles."""
    from paper_2604_18117_amd import binding as lq
    K1, N2, r = 128, 64, 32
    l1, l2 = _layer("p", M, K1, N1, r, 8, 5), _layer("c", M, N1, N2, r, 8, 6)
    X, W1, L1, R1 = wl.make_inputs(l1)
    _, W2, L2, R2 = wl.make_inputs(l2)
    X[3] = 0.0
    X[5:15] *= np.float32(2.0 ** -88)     # both ends of the range that block maxima may take
    X[15:25] *= np.float32(2.0 ** 110)
    X[30, 1:] = 0.0           # (a token whose outputs are one column of W)
    X = wl.round_to_bf16(X)
    W1[32:64] = 0.0
    L1[32:64] = 0.0           # outputs 32..63 are exactly zero for every token: an all-zero block of the consumer
    cfg1, pk1 = _pack(lq, l1, W1, L1, R1)
    cfg2, pk2 = _pack(lq, l2, W2, L2, R2)
    act1 = lq.lq_quantize_act(cfg1, pk1, wl.to_dev_x(X, "bf16"))
    Y1 = lq.lq_linear_lowrank_fwd(cfg1, pk1, act1, M)
    act2_ref = lq.lq_quantize_act(cfg2, pk2, Y1)
    Yh = torch.full((M, N1), -1, dtype=torch.int16, device="cuda").view(torch.bfloat16) if with_y else None
    act2, codes = lq.lq_linear_lowrank_fwd_handoff(cfg1, pk1, act1, M, cfg2, Y=Yh)
    lq.lq_branch_from_codes(cfg2, pk2, codes, M, act2)
    if with_y:
        assert torch.equal(Yh, Y1)
    va, vr = lq.lq_unpack_act(cfg2, act2, M), lq.lq_unpack_act(cfg2, act2_ref, M)
    for f in ("xq", "xe", "tq", "te"):
        assert torch.equal(getattr(va, f), getattr(vr, f)), f
    assert not n(va.xq)[:, 32:64].any() and not n(va.xq)[3].any()
    ho = oracle.handoff_mxi(bf16_to_bits(Y1), oracle.pack_mxi(W2, L2, R2, 8))
    assert np.array_equal(n(va.xq), ho.xq) and np.array_equal(n(va.xe), ho.xe)
    Mp = (M + 31) // 32 * 32
    cb, off = n(codes[:Mp * N1]).view(np.int8).reshape(Mp, N1)[:M], (Mp * N1 + 255) // 256 * 256
    cbe = n(codes[off:off + Mp * (N1 // 32)]).reshape(Mp, N1 // 32)[:M]
    assert np.array_equal(cb, ho.xb) and np.array_equal(cbe, ho.xbe)
    assert torch.equal(lq.lq_linear_lowrank_fwd(cfg2, pk2, act2, M), lq.lq_linear_lowrank_fwd(cfg2, pk2, act2_ref, M))


def test_handoff_full_size_block_pair(oracle):
    """The QKV-sized projection feeding an attention-output-sized one, at the benchmark's token count."""
    _run(oracle, 16384, 1152, 3456, 1152, 64, 64, 8, 9, False)
