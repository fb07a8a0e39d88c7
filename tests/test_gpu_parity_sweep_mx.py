"""Seeded sweeps over small shapes around the tile edges for the block-scaled families (MX, MXB, MXI), each compared by
its family's own parity routine (codes and scale bytes bit-exact, floating-point results to the family's bound)."""
import numpy as np
import pytest

from paper_2604_18117_amd import workloads as wl
from tests.smoothing import smoothing_vector
from tests import test_gpu_parity_mx as t_mx
from tests import test_gpu_parity_mxb as t_mxb
from tests import test_gpu_parity_mxi as t_mxi

pytestmark = pytest.mark.gpu

EDGE_M = [1, 31, 32, 33, 63, 64, 65, 127, 128, 129, 255, 257]


@pytest.mark.parametrize("family", ["mx", "mxb8", "mxb6", "mxi8", "mxi4"])
def test_seeded_shape_sweep(oracle, family):
    rng = np.random.default_rng(sum(map(ord, family)))
    for it in range(20):
        M = int(rng.choice(EDGE_M))
        K = 64 * int(rng.integers(1, 12))        # odd multiples of 64 included (padded to whole 128-stages inside the blobs)
        N = 64 * int(rng.integers(1, 10)) if it % 8 else 64 * int(rng.integers(10, 40))
        xd = "bf16" if rng.integers(0, 2) else "f32"
        if family == "mx":
            r = int(rng.choice([0, 16, 32, 64, 128]))
            layer, cmp = wl.Layer("t", M, K, N, r, "mx", 32, 8, 8, xd, seed=200 + it), t_mx._compare
        elif family.startswith("mxb"):
            r, e = int(rng.choice([0, 32, 64, 96, 128])), int(family[-1])
            layer, cmp = wl.Layer("t", M, K, N, r, "mxb", 32, e, e, xd, seed=200 + it), t_mxb._compare
        else:
            r, bw = int(rng.choice([0, 32, 64, 96, 128])), int(family[-1])
            layer, cmp = wl.Layer("t", M, K, N, r, "mxi", 32, bw, 8, xd, seed=200 + it), t_mxi._compare
        X, W, L, R = wl.make_inputs(layer)
        try:
            cmp(oracle, layer, X, W, L, R)
        except AssertionError as e:
            raise AssertionError(f"{family}: M={M} K={K} N={N} r={r} {xd}: {e}") from e


@pytest.mark.parametrize("family", ["mx", "mxb8", "mxb6", "mxi8", "mxi4"])
@pytest.mark.parametrize("M,K,N,r,xd", [(200, 1152, 320, 32, "bf16"), (77, 2304, 64, 64, "f32"), (33, 256, 64, 0, "bf16")])
def test_fused_smoothing(oracle, family, M, K, N, r, xd):
    """Activation smoothing (Section 3.4; App. A.1) fused into the MX families' activation kernels: the GPU gets the raw X
    and the smoothing vector, the oracle quantises the smoothed input; same bars as without smoothing."""
    base = wl.shrink(wl.LAYERS["c2_qkv"], M=M, K=K, N=N, r=r)           # outlier channels for the vector to tame
    kw = dict(base.__dict__, x_dtype=xd, seed=M + K, g=32)
    if family == "mx":
        layer, cmp = wl.Layer(**dict(kw, family="mx", br_w_bits=8, br_a_bits=8)), t_mx._compare
    elif family.startswith("mxb"):
        e = int(family[-1])
        layer, cmp = wl.Layer(**dict(kw, family="mxb", br_w_bits=e, br_a_bits=e)), t_mxb._compare
    else:
        layer, cmp = wl.Layer(**dict(kw, family="mxi", br_w_bits=int(family[-1]), br_a_bits=8)), t_mxi._compare
    X, W, L, R = wl.make_inputs(layer)
    gamma = smoothing_vector(X, W)
    Ws = (W.astype(np.float64) * gamma).astype(np.float32)            # the caller folds gamma into W before packing
    cmp(oracle, layer, X, Ws, L, R, gamma=gamma)
    # the vector did change the codes: the unsmoothed run differs
    from tests.gpu_util import n, run_gpu
    a = run_gpu(layer, X, Ws, L, R, debug=True, debug_acc=False)
    b = run_gpu(layer, X, Ws, L, R, debug=True, debug_acc=False, gamma=gamma)
    assert not np.array_equal(n(a.av.xq), n(b.av.xq))


@pytest.mark.parametrize("family,g,bw,ag", [("int", 64, 8, 0), ("int", 128, 4, 0), ("int", 64, 6, 64), ("mx", 32, 8, 32), ("mxb", 32, 8, 32),
                                            ("mxb", 32, 6, 32), ("mxi", 32, 8, 32)])
@pytest.mark.parametrize("r", [32, 96, 128])
def test_packing_runs_of_groups_and_unaligned_sources(oracle, family, g, bw, ag, r):
    """Workgroups that pack several scale groups of their rows (runs of two and three), and W, L, R that are aligned to
    their elements only: codes and scales against the oracle, and the same blob from both."""
    import torch
    from paper_2604_18117_amd import binding as lq
    from tests.gpu_util import n
    if family == "mx" and r == 96:
        pytest.skip("rank 96 is not a rank of the fp32-scaled FP8 branch")
    N, K = 4096, 4736
    layer = wl.Layer("t", 1, K, N, r, family, g, bw, 8 if family != "mxb" else bw, "bf16", seed=N + r, a_group=ag)
    _, W, L, R = wl.make_inputs(layer)
    cfg = lq.config_for_layer(layer)

    def shifted(a):
        t = torch.empty(a.size + 1, dtype=torch.float32, device="cuda")[1:].view(a.shape)
        return t.copy_(torch.from_numpy(a))
    blobs = [lq.lq_pack_weights(cfg, *s, packed=torch.zeros(lq.lq_packed_sizes(cfg), dtype=torch.uint8, device="cuda"))
             for s in ([torch.from_numpy(a).cuda() for a in (W, L, R)], [shifted(a) for a in (W, L, R)])]
    assert torch.equal(blobs[0], blobs[1])
    wv = lq.lq_unpack_weights(cfg, blobs[0])
    rows = np.arange(0, N, 129)  # (a row's codes depend on its own values and on R alone)
    if family == "int":
        pk = oracle.pack_int(W[rows], L[rows], R, g, bw, sint4_blocks=ag == 64)
        assert np.array_equal(n(wv.sw)[rows], pk.sw)
    elif family == "mx":
        pk = oracle.pack_mx(W[rows], L[rows], R)
    elif family == "mxb":
        pk = oracle.pack_mxb(W[rows], L[rows], R, elem=bw)
    else:
        pk = oracle.pack_mxi(W[rows], L[rows], R, bw)
    if family in ("mx", "mxb"):
        assert np.array_equal(t_mxb.E2M1[n(wv.pq).view(np.uint8)[rows]], t_mxb.E2M1[pk.pc])
    else:
        assert np.array_equal(n(wv.pq)[rows], pk.pq)
    if family != "int":
        assert np.array_equal(n(wv.pe)[rows], pk.pe)


@pytest.mark.parametrize("family,g,bw,ag", [("int", 64, 8, 0), ("int", 128, 4, 0), ("int", 64, 6, 64), ("mx", 32, 8, 32), ("mxb", 32, 8, 32),
                                            ("mxb", 32, 6, 32), ("mxi", 32, 8, 32), ("mxi", 32, 4, 32)])
@pytest.mark.parametrize("r", [0, 16, 32, 64, 96, 128])
@pytest.mark.parametrize("from_q", [True, False])
def test_packing_residual_of_quantised_and_given_factors(oracle, family, g, bw, ag, r, from_q):
    """Runs of one scale group and of several, whose last chunk requests nothing up to rank 32; an odd number of chunks, which MX layouts pad
    with one that is the last of its run or a run of its own."""
    import torch
    from paper_2604_18117_amd import binding as lq
    from tests.gpu_util import n
    if (family == "mx" and r == 96) or (family in ("mxb", "mxi") and r == 16):
        pytest.skip("not a rank of this branch")
    for N, K in ((64, 64), (192, 320), (4096, 4672)):
        K = (K + g - 1) // g * g
        rng = np.random.default_rng(N + r)
        W, L, R = ((rng.standard_normal(s) * f).astype(np.float32) for s, f in (((N, K), 0.02), ((N, r), 0.03), ((r, K), 0.03)))
        cfg = lq.make_config(N, K, r, family, g, bw, bw if family == "mxb" else 8, residual_from_quantized=from_q, a_group=ag)
        dW, dL, dR = (torch.from_numpy(a).cuda() if a.size else None for a in (W, L, R))
        wv = lq.lq_unpack_weights(cfg, lq.lq_pack_weights(cfg, dW, dL, dR))
        rows = np.arange(0, N, 1 if N < 200 else 129)
        args = (W[rows], L[rows] if r else None, R if r else None)
        if family == "int":
            pk = oracle.pack_int(*args, g, bw, residual_from_quantized=from_q, sint4_blocks=ag == 64)
            assert np.array_equal(n(wv.sw)[rows], pk.sw) and np.array_equal(n(wv.pq)[rows], pk.pq), (N, K)
            continue
        pk = oracle.pack_mxi(*args, bw, residual_from_quantized=from_q) if family == "mxi" else \
            oracle.pack_mx(*args, residual_from_quantized=from_q) if family == "mx" else oracle.pack_mxb(*args, residual_from_quantized=from_q, elem=bw)
        assert np.array_equal(n(wv.pe)[rows], pk.pe), (N, K)
        if family == "mxi":
            assert np.array_equal(n(wv.pq)[rows], pk.pq), (N, K)
        else:
            assert np.array_equal(t_mxb.E2M1[n(wv.pq).view(np.uint8)[rows]], t_mxb.E2M1[pk.pc]), (N, K)
