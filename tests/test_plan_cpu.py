"""Host-only checks of the workspace layout: over a grid of shapes, no launch of any entry point's sequence
plans more partial-sum bytes than the layout reserves for them.  (The calls refuse such a launch at run
time; this shows on the CPU that the refusal never triggers for a workspace of fhpc_workspace_bytes.)"""
import itertools

import pytest

import paper_2402_13533_amd as fhpc

Ms = [1, 16, 33, 64, 65, 130, 256, 300, 515, 1024, 1100, 1152, 2048, 4000, 4096, 16384]
KNs = [64, 136, 256, 264, 520, 1024, 1216, 2048, 4096, 5120, 11008, 13824]
RANKS = [1, 5, 8, 16, 24, 32, 40, 64, 128, 512, 1024]


def _assert_fits(call, tag, **kw):
    rc, planned, reserved = fhpc.plan_slab_bytes(call, **kw)
    assert rc == 0, (tag, kw, rc)
    assert planned <= reserved, (tag, kw, planned, reserved)
    return planned


def test_factorised_layer_slabs_fit():
    n = 0
    for M, K, N, r in itertools.product(Ms, KNs, KNs, RANKS):
        if (M + K + N + r) % 3:            # a third of the grid, spread evenly
            continue
        for outputs in (7, 1, 6, 15, 2 | 8, 4):
            _assert_fits(fhpc.FHPC_OP_LOWRANK_BWD, "lowrank_bwd", M=M, K=K, r=r, N=N, outputs=outputs)
        for outputs in (0, 1):
            _assert_fits(fhpc.FHPC_OP_LOWRANK_FWD, "lowrank_fwd", M=M, K=K, r=r, N=N, outputs=outputs)
        n += 1
    assert n > 3000


def test_shared_x_slabs_fit():
    """Includes g = 1 with r > 32 and N > K, where dH = dY B^T of the single (dense) block may take the split
    route: the shape class a fixed workspace bug lived in."""
    worst = 0
    for M, K, N, r, g in itertools.product(Ms, KNs, KNs, [8, 16, 32, 40, 64, 128, 512, 1024], [1, 2, 3, 8]):
        if (M + K + N + r + g) % 3:
            continue
        for outputs in (7, 1, 6, 15, 2 | 8, 4):
            worst = max(worst, _assert_fits(fhpc.FHPC_PLAN_SHARED_BWD, "shared_bwd", M=M, K=K, r=r, N=N, g=g, outputs=outputs))
        for outputs in (0, 1):
            _assert_fits(fhpc.FHPC_PLAN_SHARED_FWD, "shared_fwd", M=M, K=K, r=r, N=N, g=g, outputs=outputs)
    assert worst > 0
    # the two shapes the finding was reported on
    for M, K, r, N in ((64, 1024, 64, 4096), (33, 64, 40, 256)):
        rc, planned, reserved = fhpc.plan_slab_bytes(fhpc.FHPC_PLAN_SHARED_BWD, M, K, r, N, g=1)
        assert rc == 0 and 0 < planned <= reserved, (M, K, r, N, planned, reserved)


def test_shared_x_slabs_fit_when_some_dB_are_left_out():
    """The weight gradients that are wanted then go out one by one, each cut deeper than in the launch that carries all g."""
    _assert_fits(fhpc.FHPC_PLAN_SHARED_BWD, "shared_bwd", M=1861, K=5816, r=296, N=5104, g=4, outputs=7 | 16)
    for M, K, N, r, g in itertools.product(Ms, KNs, KNs, [8, 16, 32, 40, 64, 128, 296, 512, 1024], [1, 2, 3, 4, 8]):
        if (M + K + N + r + g) % 3 == 0:
            for outputs in (7 | 16, 4 | 8 | 16):
                _assert_fits(fhpc.FHPC_PLAN_SHARED_BWD, "shared_bwd", M=M, K=K, r=r, N=N, g=g, outputs=outputs)


@pytest.mark.parametrize("M,K,r,N,g", [(15060, 464, 168, 368, 1), (9531, 664, 48, 576, 1), (5315, 1192, 200, 912, 1), (9339, 608, 96, 568, 4)])
def test_input_gradient_does_not_displace_the_slices_of_the_weight_gradients(M, K, r, N, g):
    """Many tokens on a small layer: the tiles of dX would leave one workgroup per tile of dA and dB to walk all tokens
    (155 microseconds against 56 on the first of these)."""
    call = fhpc.FHPC_OP_LOWRANK_BWD if g == 1 else fhpc.FHPC_PLAN_SHARED_BWD
    slabs = _assert_fits(call, "dB", M=M, K=K, r=r, N=N, g=g, outputs=4 | 8)          # (the slabs of dA and dB, nothing else)
    assert slabs >= 4 * 4 * g * r * (K + N)


@pytest.mark.parametrize("M,K,r,N,sliced", [(936, 416, 40, 264, True), (386, 504, 112, 688, True), (153, 448, 168, 264, True), (1430, 464, 45, 704, True),
                                            (600, 264, 256, 2048, False), (590, 264, 264, 712, False), (1431, 360, 160, 264, False)])
def test_short_reductions_in_slices(M, K, r, N, sliced):
    """H = X A of few ranks goes out in slices of a reduction down to 256, larger outputs whole (what either takes stands at the rule)."""
    assert (_assert_fits(fhpc.FHPC_OP_LOWRANK_FWD, "forward", M=M, K=K, r=r, N=N, outputs=1) > 0) == sliced


def test_ffn_gate_calls_slabs_fit():
    """lowrank_ffn_gate_up_fwd and lowrank_ffn_down_bwd: the gate in the epilogue of the large tiles, the streaming
    gate kernel elsewhere, the same workspace layouts as the calls they stand for."""
    n = 0
    for M, K, N, r in itertools.product(Ms, KNs, KNs, [8, 16, 32, 40, 64, 128, 512, 1024]):
        if (M + K + N + r) % 3:
            continue
        for outputs in (0, 1):
            _assert_fits(fhpc.FHPC_PLAN_FFN_GATE_UP, "ffn_gate_up", M=M, K=K, r=r, N=N, outputs=outputs)
        for outputs in (6, 6 | 8, 2, 4 | 8, 0):
            _assert_fits(fhpc.FHPC_PLAN_FFN_DOWN_BWD, "ffn_down_bwd", M=M, K=K, r=r, N=N, outputs=outputs)
        n += 1
    assert n > 2000


@pytest.mark.parametrize("qscheme", [fhpc.FHPC_Q_INT4_BLOCK, fhpc.FHPC_Q_INT8_PER_CHANNEL, fhpc.FHPC_W_BF16, fhpc.FHPC_W_MERGED])
def test_quantised_layer_slabs_fit(qscheme):
    for M, K, N, r in itertools.product(Ms, [64, 256, 1024, 4096, 5120, 13824], [64, 264, 1024, 4096, 5120, 13824],
                                        [1, 8, 16, 24, 40, 64, 128]):
        for base_scale in (1.0, 0.0, 0.25):
            if qscheme == fhpc.FHPC_W_MERGED and base_scale != 1.0:
                continue
            for outputs in (7, 1, 6, 15, 2 | 8, 4):
                _assert_fits(fhpc.FHPC_OP_QLINEAR_BWD, "qlinear_bwd", M=M, K=K, r=r, N=N, qscheme=qscheme,
                             outputs=outputs, base_scale=base_scale)
            for outputs in (0, 1):
                _assert_fits(fhpc.FHPC_OP_QLINEAR_FWD, "qlinear_fwd", M=M, K=K, r=r, N=N, qscheme=qscheme,
                             outputs=outputs, base_scale=base_scale)


def test_decompose_slabs_fit():
    """r close to K with N a little larger: the Gram product over K needs more slices than the one over N."""
    dims = [64, 256, 512, 1024, 1088, 1216, 2048, 4096, 4160, 8192]
    seen = 0
    for K, N in itertools.product(dims, dims):
        for r in (8, 64, 256, 512, 1024, 2048):
            if r > min(K, N):
                continue
            seen = max(seen, _assert_fits(fhpc.FHPC_OP_DECOMPOSE, "decompose", M=1, K=K, r=r, N=N))
    assert seen > 0
    rc, planned, reserved = fhpc.plan_slab_bytes(fhpc.FHPC_OP_DECOMPOSE, 1, 1024, 1024, 1216)
    assert rc == 0 and 0 < planned <= reserved


@pytest.mark.parametrize("M,K,N,slices", [
    (300, 4096, 4096, 3), (150, 2816, 5120, 4), (100, 4096, 2048, 8),      # 64-row tiles
    (13, 1728, 12096, 3),                                                  # one block of rows
    (83, 4864, 4224, 9), (75, 3264, 4736, 6), (205, 3840, 5120, 6),        # 128-row tiles, which read the weight half as often
    (213, 3520, 2560, 6),                                                  # (64 rows: a few workgroups more than units)
])
def test_rows_of_dequantising_tiles(M, K, N, slices):
    """The slices of the dequantising product tell its tile (what either takes stands at the rule)."""
    for scheme in (fhpc.FHPC_W_BF16,) if M <= 64 else (fhpc.FHPC_Q_INT8_PER_CHANNEL, fhpc.FHPC_W_BF16):
        assert _assert_fits(fhpc.FHPC_OP_QLINEAR_FWD, "qlinear_fwd", M=M, K=K, r=16, N=N, qscheme=scheme) == slices * M * N * 4


@pytest.mark.parametrize("M,K,r,sliced", [(3500, 6144, 512, True), (3500, 5120, 384, True), (2000, 6144, 512, True), (1645, 4040, 648, True),
                                          (2600, 3584, 384, False), (2000, 4096, 512, False), (1000, 4096, 1000, False)])
def test_slices_of_long_reductions(M, K, r, sliced):
    """H = X A where 64 x 64 tiles fill the chip by themselves: whole on those, or on large tiles in slices (what either takes stands at the rule)."""
    assert (_assert_fits(fhpc.FHPC_OP_LOWRANK_FWD, "forward", M=M, K=K, r=r, N=1600, outputs=1) > 0) == sliced


@pytest.mark.parametrize("M,K,r,N,scheme", [(2895, 1280, 64, 4808, 4), (1241, 20544, 128, 88, 8), (2751, 44544, 40, 8, 8), (1577, 21504, 128, 64, 8), (1770, 50560, 64, 8, 4), (1028, 45312, 64, 16, 4)])
def test_slabs_of_the_rank_product_fit_the_fixed_scratch(M, K, r, N, scheme):
    """Sizes whose other regions leave a part of the no-allocation entry point's array: the slabs of X A stay within it."""
    assert fhpc.workspace_bytes(fhpc.FHPC_OP_QLINEAR_FWD, M, K, r, N, fhpc.FHPC_BF16, scheme) <= fhpc.FHPC_NOALLOC_SCRATCH_BYTES
    for outputs in (0, 1):
        _assert_fits(fhpc.FHPC_OP_QLINEAR_FWD, "qlinear_fwd", M=M, K=K, r=r, N=N, qscheme=scheme, outputs=outputs)


def test_middle_fp32_layers_are_planned_as_quickly_as_small_ones():
    """504 tokens are below the size from which three-part operands are priced at all, 520 above it, with the same plans: 1.0 times as long a
    call, and 1.3 when every slice count of those tiles is priced first."""
    import time
    need = fhpc.load_library().fhpc_workspace_bytes
    best = {504: 1.0, 520: 1.0}
    for _ in range(30):
        for M in best:
            start = time.perf_counter()
            for _ in range(1000):
                need(fhpc.FHPC_OP_LOWRANK_BWD, M, 1024, 64, 1024, fhpc.FHPC_F32, 0)
            best[M] = min(best[M], time.perf_counter() - start)
    assert best[520] <= 1.15 * best[504], best
