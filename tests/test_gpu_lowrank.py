"""GPU parity of lowrank_linear_fwd / lowrank_linear_bwd against the CPU oracle on the
same seeded inputs (element by element, relative Frobenius error per output tensor)."""
import numpy as np
import pytest

import oracle
from harness import Guarded, TOL_BF16, TOL_F32, Bf16, from_device, lowrank_inputs, sample_rows, parity_err

pytestmark = pytest.mark.gpu


def _fhpc():
    import paper_2402_13533_amd as fhpc
    return fhpc


def _check_all(tag, got, ref, tol):
    for name, g, r in zip(("Y", "dX", "dA", "dB"), got, ref):
        if g is None:
            continue
        err = parity_err(from_device(g), r, tol, "%s %s" % (tag, name))
        print("%s %s rel_fro=%.3e" % (tag, name, err), flush=True)
        assert err <= tol, (tag, name, err)


def test_config1_fp32():
    """Config 1: fp32, X 256x768, r = 32; tolerance 1e-5."""
    import torch
    fhpc = _fhpc()
    M, K, r, N = 256, 768, 32, 768
    X, A, B, dY = lowrank_inputs(1, M, K, r, N, bf16=False)
    Yr, Hr = oracle.lowrank_fwd(X, A, B)
    ref = (Yr,) + oracle.lowrank_bwd(X, A, B, dY)
    d = lambda a: torch.from_numpy(a).cuda()
    Xd, Ad, Bd, dYd = d(X), d(A), d(B), d(dY)
    Y, H = fhpc.lowrank_linear_fwd(Xd, Ad, Bd, save_H=True)
    assert parity_err(from_device(H), Hr) <= TOL_F32
    dX, dA, dB = fhpc.lowrank_linear_bwd(Xd, Ad, Bd, dYd, H_saved=H)
    _check_all("c1 saved-H", (Y, dX, dA, dB), ref, TOL_F32)
    dX, dA, dB = fhpc.lowrank_linear_bwd(Xd, Ad, Bd, dYd)             # recompute H
    _check_all("c1 recompute", (None, dX, dA, dB), ref, TOL_F32)


@pytest.mark.parametrize("M,K,r,N", [
    (16, 48, 16, 64),        # chain: whole 16-row, 16-rank and 64-column blocks
    (17, 1032, 17, 72),      # chain: one row, one rank and eight columns beyond; a reduction that ends half-way through a step
    (257, 512, 48, 520),     # chain: more rows than 256 at the largest product of reduction and rank taken there
    (257, 520, 48, 512),     # ... one beyond it: products of their own in one direction, a chain in the other
    (65, 3080, 66, 264),     # products: rank not a multiple of four (single-word loads), the reduction in slices
    (1030, 264, 129, 776),   # products: odd rank, ragged tiles of 64 and 32
    (4100, 136, 24, 4104),   # products: a rank the chain would hold, too many rows; gradients in many slices
    (2049, 72, 192, 200),    # products: reductions that end inside a 32-deep step
])
def test_fp32_products_and_chain(M, K, r, N):
    """The fp32 matrix-core products (two tile sizes, whole and sliced reductions, 16-byte and single-word loads) and the
    chained pair at the edges of the rule between them, against the oracle; H saved and recomputed have the same bits."""
    import torch
    fhpc = _fhpc()
    X, A, B, dY = lowrank_inputs(3, M, K, r, N, bf16=False)
    Yr, Hr = oracle.lowrank_fwd(X, A, B)
    ref = (Yr,) + oracle.lowrank_bwd(X, A, B, dY)
    Xd, Ad, Bd, dYd = (torch.from_numpy(a).cuda() for a in (X, A, B, dY))
    guard = Guarded()
    g = [guard.alloc(s, torch.float32) for s in ((M, N), (M, r), (M, K), (K, r), (r, N))]
    Y, H = fhpc.lowrank_linear_fwd(Xd, Ad, Bd, Y=g[0], H_out=g[1])
    assert parity_err(from_device(H), Hr, TOL_F32, "H") <= TOL_F32
    out = fhpc.lowrank_linear_bwd(Xd, Ad, Bd, dYd, H_saved=H, dX=g[2], dA=g[3], dB=g[4])
    _check_all("f32 %s" % ((M, K, r, N),), (Y,) + out, ref, TOL_F32)
    guard.check("f32 %s" % ((M, K, r, N),))
    again = fhpc.lowrank_linear_bwd(Xd, Ad, Bd, dYd)                  # H recomputed
    assert all(torch.equal(a, b) for a, b in zip(out, again))


@pytest.mark.parametrize("M,K,r,N", [(20, 72, 5, 40), (300, 1032, 70, 40)])      # the chain; products of their own
def test_fp32_infinities_stay_in_their_row(M, K, r, N):
    """An infinite input makes its own token's outputs infinite or NaN exactly where IEEE arithmetic says, and nothing
    else: what pads ranks, rows and reductions to the blocks of the matrix instructions must not meet it."""
    import torch
    fhpc = _fhpc()
    X, A, B, _ = lowrank_inputs(3, M, K, r, N, bf16=False)
    A, B = np.abs(A) + 0.1, np.abs(B) + 0.1
    X[3, 7] = np.inf
    Y, H = fhpc.lowrank_linear_fwd(*(torch.from_numpy(a).cuda() for a in (X, A, B)), save_H=True)
    for got, cols in ((H, r), (Y, N)):
        got = got.cpu().numpy()
        assert np.all(got[3] == np.inf) and got.shape[1] == cols
        assert np.all(np.isfinite(np.delete(got, 3, 0)))


@pytest.mark.parametrize("M,K,r,N", [
    (50, 136, 5, 72),        # ragged token count and rank (K and N are multiples of 8 by contract); one launch per chain: H and dH stay in LDS
    (33, 64, 64, 264),       # the largest rank that fits, a ragged row block, more columns than threads
    (17, 200, 65, 96),       # one rank beyond: two launches per chain
    (1, 8, 1, 8),
])
def test_fp32_shapes(M, K, r, N):
    """fp32 storage and arithmetic on shapes other than config 1's (tolerance 1e-5), with H saved, recomputed, and
    with outputs left out."""
    import torch
    fhpc = _fhpc()
    X, A, B, dY = lowrank_inputs(2, M, K, r, N, bf16=False)
    Yr, Hr = oracle.lowrank_fwd(X, A, B)
    ref = (Yr,) + oracle.lowrank_bwd(X, A, B, dY)
    d = lambda a: torch.from_numpy(a).cuda()
    Xd, Ad, Bd, dYd = d(X), d(A), d(B), d(dY)
    Y, H = fhpc.lowrank_linear_fwd(Xd, Ad, Bd, save_H=True)
    assert parity_err(from_device(H), Hr, TOL_F32, "H") <= TOL_F32
    Y2 = fhpc.lowrank_linear_fwd(Xd, Ad, Bd)                          # H not asked for
    assert torch.equal(Y, Y2)
    dX, dA, dB = fhpc.lowrank_linear_bwd(Xd, Ad, Bd, dYd, H_saved=H)
    _check_all("f32 saved-H %s" % ((M, K, r, N),), (Y, dX, dA, dB), ref, TOL_F32)
    dX, dA, dB = fhpc.lowrank_linear_bwd(Xd, Ad, Bd, dYd)
    _check_all("f32 recompute %s" % ((M, K, r, N),), (None, dX, dA, dB), ref, TOL_F32)
    dX3, dA3, dB3 = fhpc.lowrank_linear_bwd(Xd, Ad, Bd, dYd, H_saved=H, need_dA=False)
    assert dA3 is None and torch.equal(dX3, dX) and torch.equal(dB3, dB)


@pytest.mark.parametrize("M,K,r,N", [
    (300, 320, 64, 264),     # ragged in every dimension, several tiles
    (1, 64, 8, 72),          # a single token
    (257, 136, 5, 200),      # rank not a multiple of 8 (padded internally)
    (515, 1024, 16, 520),    # LoRA-sized rank: split reductions for H and dH
    (640, 512, 96, 1032),    # rank between tile sizes
    (1100, 768, 512, 776),   # pretraining-sized rank
    (48, 520, 40, 264),      # few tokens, small rank: dA and dB as token-deep sums in one launch
    (64, 1032, 512, 776),    # few tokens, large rank: dA and dB as tiles of outer-product sums
    (33, 328, 77, 264),      # the same with a rank that is padded (dA rows not 16-byte aligned)
    (1, 264, 130, 520),
    (4000, 2048, 512, 2056), # X A and dY B^T: 64 tiles of 256 x 128 (ragged last row), reductions cut into 4 slices on the large tiles
    (1300, 8192, 520, 264),  # X A: 6 x 3 tiles of 256 x 256 in 16 slices of 512
])
def test_bf16_shapes(M, K, r, N):
    fhpc = _fhpc()
    X, A, B, dY = lowrank_inputs(9, M, K, r, N, tensor_base=10)
    Yr, Hr = oracle.lowrank_fwd(X.f64, A.f64, B.f64)
    ref = (Yr,) + oracle.lowrank_bwd(X.f64, A.f64, B.f64, dY.f64)
    import torch
    Xd, Ad, Bd, dYd = X.cuda(), A.cuda(), B.cuda(), dY.cuda()
    # every output sits between guard regions: nothing may be written outside it
    g = Guarded()
    bf = torch.bfloat16
    Y, H = fhpc.lowrank_linear_fwd(Xd, Ad, Bd, Y=g.alloc((M, N), bf), H_out=g.alloc((M, r), bf))
    assert parity_err(from_device(H), Hr) <= TOL_BF16
    dX, dA, dB = fhpc.lowrank_linear_bwd(Xd, Ad, Bd, dYd, H_saved=H, dX=g.alloc((M, K), bf),
                                         dA=g.alloc((K, r), torch.float32), dB=g.alloc((r, N), torch.float32))
    g.check("bf16 %s" % ((M, K, r, N),))
    _check_all("bf16 %s saved-H" % ((M, K, r, N),), (Y, dX, dA, dB), ref, TOL_BF16)
    Y2 = fhpc.lowrank_linear_fwd(Xd, Ad, Bd)                          # no H_out
    # (against the oracle, not bit for bit against Y: with H not asked for the products may take another route)
    assert parity_err(from_device(Y2), Yr) <= TOL_BF16
    dX2, dA2, dB2 = fhpc.lowrank_linear_bwd(Xd, Ad, Bd, dYd)          # recompute H
    _check_all("bf16 %s recompute" % ((M, K, r, N),), (None, dX2, dA2, dB2), ref, TOL_BF16)


@pytest.mark.parametrize("M,K,r,N", [
    (1, 4096, 512, 4096),    # one token at the pretraining configuration's layer
    (16, 1024, 128, 776),
    (32, 520, 5, 264),       # odd rank, ragged reduction
    (7, 768, 24, 72),
])
def test_bf16_few_tokens_forward(M, K, r, N):
    """At most 32 tokens: both products of the forward run as split reductions on a 32-row tile."""
    fhpc = _fhpc()
    X, A, B, _ = lowrank_inputs(9, M, K, r, N, tensor_base=30)
    Yr, Hr = oracle.lowrank_fwd(X.f64, A.f64, B.f64)
    Y, H = fhpc.lowrank_linear_fwd(X.cuda(), A.cuda(), B.cuda(), save_H=True)
    eY, eH = parity_err(from_device(Y), Yr), parity_err(from_device(H), Hr)
    print("few tokens %s: Y %.3e H %.3e" % ((M, K, r, N), eY, eH), flush=True)
    assert eY <= TOL_BF16 and eH <= TOL_BF16
    Y2 = fhpc.lowrank_linear_fwd(X.cuda(), A.cuda(), B.cuda())
    assert np.array_equal(from_device(Y2), from_device(Y))


def test_bf16_optional_outputs_and_canaries():
    """NULL outputs are skipped; nothing is written outside the output tensors."""
    import torch
    fhpc = _fhpc()
    M, K, r, N = 130, 72, 24, 88
    X, A, B, dY = lowrank_inputs(9, M, K, r, N, tensor_base=20)
    ref = oracle.lowrank_bwd(X.f64, A.f64, B.f64, dY.f64)
    Xd, Ad, Bd, dYd = X.cuda(), A.cuda(), B.cuda(), dY.cuda()
    pad = 1024
    big = torch.full((M * K + 2 * pad,), 7.0, dtype=torch.bfloat16, device="cuda")
    dX = big[pad:pad + M * K].view(M, K)
    out = fhpc.lowrank_linear_bwd(Xd, Ad, Bd, dYd, need_dA=False, need_dB=False, dX=dX)
    assert out[1] is None and out[2] is None
    assert parity_err(from_device(dX), ref[0]) <= TOL_BF16
    assert bool((big[:pad] == 7.0).all()) and bool((big[pad + M * K:] == 7.0).all())
    _, dA, dB = fhpc.lowrank_linear_bwd(Xd, Ad, Bd, dYd, need_dX=False)
    assert parity_err(from_device(dA), ref[1]) <= TOL_BF16
    assert parity_err(from_device(dB), ref[2]) <= TOL_BF16


def test_config2_full_size_sampled():
    """Config 2 at full size (16384 tokens, d = 4096, r = 512), the launch configuration the
    benchmark times.  Y and dX are checked on sampled rows (rows are independent), dA on
    sampled columns and dB on sampled rows (column j of dA / row j of dB depends only on
    column j of A / row j of B through the rank index, so the oracle evaluates the layer
    restricted to those rank indices)."""
    fhpc = _fhpc()
    M, K, r, N = 16384, 4096, 512, 4096
    for proj in range(4):                     # q, k, v, o: four independent calls
        X, A, B, dY = lowrank_inputs(2, M, K, r, N, tensor_base=10 * proj)
        Xd, Ad, Bd, dYd = X.cuda(), A.cuda(), B.cuda(), dY.cuda()
        Y, H = fhpc.lowrank_linear_fwd(Xd, Ad, Bd, save_H=True)
        dX, dA, dB = fhpc.lowrank_linear_bwd(Xd, Ad, Bd, dYd, H_saved=H)
        rows = sample_rows(M, 100 + proj)
        Yr, _ = oracle.lowrank_fwd(X.rows(rows).f64, A.f64, B.f64)
        dXr, _, _ = oracle.lowrank_bwd(X.rows(rows).f64, A.f64, B.f64, dY.rows(rows).f64)
        J = np.unique(np.random.default_rng(200 + proj).integers(0, r, size=8))
        Af, Bf = A.f64, B.f64
        _, dAr, dBr = oracle.lowrank_bwd(X.f64, Af[:, J], Bf[J, :], dY.f64)
        errs = {
            "Y": parity_err(from_device(Y)[rows], Yr),
            "dX": parity_err(from_device(dX)[rows], dXr),
            "dA": parity_err(from_device(dA)[:, J], dAr),
            "dB": parity_err(from_device(dB)[J, :], dBr),
        }
        print("c2 proj %d: %s" % (proj, {k: "%.3e" % v for k, v in errs.items()}), flush=True)
        for k, v in errs.items():
            assert v <= TOL_BF16, (proj, k, v)


def test_config2_shared_x_full_size_sampled():
    """Config 2 at full size through the calls the benchmark times: q, k and v (g = 3) read one X through
    lowrank_linear_fwd/bwd_shared_x, whose wide products (X A_all 1536 wide, the input gradient over a reduction
    of 1536, dA_all 4096 x 1536) choose their own tiles and splits.  Y_i and the summed dX on sampled token rows,
    dA_all on sampled columns of every layer's block, dB_i on the same rank rows; the o projection goes through
    the single-layer calls (test_config2_full_size_sampled)."""
    fhpc = _fhpc()
    M, K, r, N, g = 16384, 4096, 512, 4096, 3
    X, As, Bs, dYs = None, [], [], []
    for i in range(g):
        Xi, A, B, dY = lowrank_inputs(2, M, K, r, N, tensor_base=40 + 10 * i)
        X = Xi if X is None else X
        As.append(A); Bs.append(B); dYs.append(dY)
    A_all = Bf16(np.concatenate([A.bits for A in As], axis=1)).cuda()
    Xd, Bd, dYd = X.cuda(), [B.cuda() for B in Bs], [dY.cuda() for dY in dYs]
    Ys, H = fhpc.lowrank_linear_fwd_shared_x(Xd, A_all, Bd, save_H=True)
    dX, dA, dBs = fhpc.lowrank_linear_bwd_shared_x(Xd, A_all, Bd, dYd, H_all_saved=H)
    rows = sample_rows(M, 300)
    Xr, Xf = X.rows(rows).f64, X.f64
    dXr = np.zeros((rows.size, K))
    H_got, dA_got = from_device(H), from_device(dA)
    for i in range(g):
        Af, Bf = As[i].f64, Bs[i].f64
        Yr, Hr = oracle.lowrank_fwd(Xr, Af, Bf)
        dx, _, _ = oracle.lowrank_bwd(Xr, Af, Bf, dYs[i].rows(rows).f64)
        dXr += dx
        J = np.unique(np.random.default_rng(310 + i).integers(0, r, size=8))
        _, dAr, dBr = oracle.lowrank_bwd(Xf, Af[:, J], Bf[J, :], dYs[i].f64)
        errs = {
            "Y%d" % i: parity_err(from_device(Ys[i])[rows], Yr, what="Y%d" % i),
            "H%d" % i: parity_err(H_got[rows][:, i * r:(i + 1) * r], Hr, what="H%d" % i),
            "dA%d" % i: parity_err(dA_got[:, i * r + J], dAr, what="dA%d" % i),
            "dB%d" % i: parity_err(from_device(dBs[i])[J, :], dBr, what="dB%d" % i),
        }
        print("c2 shared-x layer %d: %s" % (i, {k: "%.3e" % v for k, v in errs.items()}), flush=True)
        for k, v in errs.items():
            assert v <= TOL_BF16, (k, v)
    e = parity_err(from_device(dX)[rows], dXr, what="dX")
    print("c2 shared-x dX (sum of the three input gradients) %.3e" % e, flush=True)
    assert e <= TOL_BF16


@pytest.mark.parametrize("M", [1, 40, 300])
def test_bf16_rank_one_and_three(M):
    """Degenerate ranks: the pair is a single outer product (r = 1), and r = 3."""
    fhpc = _fhpc()
    for r in (1, 3):
        K, N = 264, 136
        X, A, B, dY = lowrank_inputs(9, M, K, r, N, tensor_base=50 + r)
        Yr, Hr = oracle.lowrank_fwd(X.f64, A.f64, B.f64)
        ref = (Yr,) + oracle.lowrank_bwd(X.f64, A.f64, B.f64, dY.f64)
        Xd, Ad, Bd, dYd = X.cuda(), A.cuda(), B.cuda(), dY.cuda()
        Y, H = fhpc.lowrank_linear_fwd(Xd, Ad, Bd, save_H=True)
        assert tuple(H.shape) == (M, r) and parity_err(from_device(H), Hr) <= TOL_BF16
        dX, dA, dB = fhpc.lowrank_linear_bwd(Xd, Ad, Bd, dYd, H_saved=H)
        _check_all("rank %d M=%d" % (r, M), (Y, dX, dA, dB), ref, TOL_BF16)


def test_results_are_bit_reproducible_from_run_to_run():
    """The header promises it: reductions over tokens go to slabs that are added in a fixed order (no
    atomics), so two runs of the same call give the same bits, whatever ran in between."""
    import torch
    fhpc = _fhpc()
    M, K, r, N = 2100, 520, 24, 392
    X, A, B, dY = lowrank_inputs(9, M, K, r, N, tensor_base=70)
    Xd, Ad, Bd, dYd = X.cuda(), A.cuda(), B.cuda(), dY.cuda()

    def run():
        Y, H = fhpc.lowrank_linear_fwd(Xd, Ad, Bd, save_H=True)
        dX, dA, dB = fhpc.lowrank_linear_bwd(Xd, Ad, Bd, dYd, H_saved=H)
        torch.cuda.synchronize()
        return [t.clone() for t in (Y, H, dX, dA, dB)]

    first = run()
    fhpc.lowrank_linear_fwd(Xd[:77], Ad, Bd)                     # other work on the same workspace
    filler = torch.randn(1 << 22, device="cuda").sum().item()     # and on the device
    for _ in range(3):
        for a, b in zip(first, run()):
            assert torch.equal(a, b)
    assert np.isfinite(filler)


def _shared_inputs(M, K, r, N, g, base):
    """g factor pairs on one X: (X, [A_i], [B_i], [dY_i]) with the usual distributions."""
    X = None
    As, Bs, dYs = [], [], []
    for i in range(g):
        Xi, A, B, dY = lowrank_inputs(9, M, K, r, N, tensor_base=base + 4 * i)
        X = Xi if X is None else X
        As.append(A); Bs.append(B); dYs.append(dY)
    return X, As, Bs, dYs


@pytest.mark.parametrize("M,K,r,N,g", [
    (300, 320, 64, 264, 3),      # q/k/v, rank above the split threshold, ragged everywhere
    (515, 1024, 16, 520, 2),     # gate/up at a LoRA-sized rank: every narrow product splits its reduction
    (257, 136, 8, 200, 3),       # g r = 24
    (640, 512, 24, 1032, 3),     # r <= 32 < g r: dH_i split, X A_all whole
    (1100, 768, 128, 776, 2),
    (1, 64, 8, 72, 2),           # a single token
    (130, 264, 40, 136, 1),      # g = 1 is the plain layer
    (64, 264, 64, 1032, 1),      # g = 1, r > 32, N > K: dH = dY B^T of the one (dense) block splits its reduction
    (96, 128, 8, 64, 8),         # the most layers one call takes
])
def test_shared_x_factorised_layers(M, K, r, N, g):
    """lowrank_linear_fwd/bwd_shared_x against g runs of the oracle: dX is the sum of the layers' input
    gradients, dA_all and H_all hold the layers' blocks side by side."""
    import torch
    fhpc = _fhpc()
    X, As, Bs, dYs = _shared_inputs(M, K, r, N, g, base=60)
    Yr, Hr, dXr, dAr, dBr = [], [], np.zeros((M, K)), [], []
    for A, B, dY in zip(As, Bs, dYs):
        y, h = oracle.lowrank_fwd(X.f64, A.f64, B.f64)
        dx, da, db = oracle.lowrank_bwd(X.f64, A.f64, B.f64, dY.f64)
        Yr.append(y); Hr.append(h); dXr += dx; dAr.append(da); dBr.append(db)
    Hr, dAr = np.concatenate(Hr, axis=1), np.concatenate(dAr, axis=1)
    A_all = Bf16(np.concatenate([A.bits for A in As], axis=1)).cuda()
    Xd, Bd, dYd = X.cuda(), [B.cuda() for B in Bs], [dY.cuda() for dY in dYs]
    tag = "shared-x %s" % ((M, K, r, N, g),)

    def check(name, got, ref):
        err = parity_err(from_device(got), ref)
        print("%s %s rel_fro=%.3e" % (tag, name, err), flush=True)
        assert err <= TOL_BF16, (tag, name, err)

    Ys, H = fhpc.lowrank_linear_fwd_shared_x(Xd, A_all, Bd, save_H=True)
    check("H_all", H, Hr)
    for i in range(g):
        check("Y%d" % i, Ys[i], Yr[i])
    Ys2 = fhpc.lowrank_linear_fwd_shared_x(Xd, A_all, Bd)                 # H kept in the workspace
    for i in range(g):
        check("Y%d (no H_out)" % i, Ys2[i], Yr[i])
    dX, dA, dBs = fhpc.lowrank_linear_bwd_shared_x(Xd, A_all, Bd, dYd, H_all_saved=H)
    check("dX", dX, dXr); check("dA_all", dA, dAr)
    for i in range(g):
        check("dB%d" % i, dBs[i], dBr[i])
    # recomputed H; one dB left out; then weight gradients only, then the input gradient only
    flags = [i != 0 for i in range(g)]
    dX2, dA2, dBs2 = fhpc.lowrank_linear_bwd_shared_x(Xd, A_all, Bd, dYd, need_dB=flags)
    check("dX (recompute)", dX2, dXr); check("dA_all (recompute)", dA2, dAr)
    assert dBs2[0] is None
    for i in range(1, g):
        check("dB%d (recompute)" % i, dBs2[i], dBr[i])
    dX3, dA3, dBs3 = fhpc.lowrank_linear_bwd_shared_x(Xd, A_all, Bd, dYd, H_all_saved=H, need_dX=False)
    assert dX3 is None
    check("dA_all (no dX)", dA3, dAr)
    dX4, dA4, dBs4 = fhpc.lowrank_linear_bwd_shared_x(Xd, A_all, Bd, dYd, need_dA=False, need_dB=False)
    assert dA4 is None and all(b is None for b in dBs4)
    check("dX (alone)", dX4, dXr)
    torch.cuda.synchronize()


def test_shared_x_matches_the_single_layer_calls():
    """The layers' outputs and weight gradients of the shared call against those of the single-layer entry
    point on the same operands, GPU against GPU.  The wide products of the shared call may run on another
    tile shape or another split of the reduction than the narrow ones, which sums in another order, so a
    few per cent of the bf16 values differ by one ulp: the bound is a fraction of the bf16 tolerance."""
    import torch
    fhpc = _fhpc()
    M, K, r, N, g = 520, 512, 64, 264, 3
    X, As, Bs, dYs = _shared_inputs(M, K, r, N, g, base=90)
    A_all = Bf16(np.concatenate([A.bits for A in As], axis=1)).cuda()
    Xd, Bd, dYd = X.cuda(), [B.cuda() for B in Bs], [dY.cuda() for dY in dYs]
    Ys, H = fhpc.lowrank_linear_fwd_shared_x(Xd, A_all, Bd, save_H=True)
    dX, dA, dBs = fhpc.lowrank_linear_bwd_shared_x(Xd, A_all, Bd, dYd, H_all_saved=H)
    dX_sum = np.zeros((M, K))
    for i in range(g):
        Ad = As[i].cuda()
        Y1, H1 = fhpc.lowrank_linear_fwd(Xd, Ad, Bd[i], save_H=True)
        dX1, dA1, dB1 = fhpc.lowrank_linear_bwd(Xd, Ad, Bd[i], dYd[i], H_saved=H1)
        assert oracle.rel_fro(from_device(H[:, i * r:(i + 1) * r].contiguous()), from_device(H1)) <= 2e-3
        assert oracle.rel_fro(from_device(Ys[i]), from_device(Y1)) <= 2e-3
        assert oracle.rel_fro(from_device(dBs[i]), from_device(dB1)) <= 2e-3
        assert oracle.rel_fro(from_device(dA[:, i * r:(i + 1) * r].contiguous()), from_device(dA1)) <= 2e-3
        dX_sum += from_device(dX1)
    assert parity_err(from_device(dX), dX_sum) <= TOL_BF16
    torch.cuda.synchronize()


@pytest.mark.parametrize("M,K,r,N", [
    (65, 264, 40, 520),          # one token more than the vector-ALU gradients take at this rank; tiles mostly outside
    (130, 1032, 100, 264),       # a padded rank
    (1100, 264, 264, 776),       # ragged tiles of all three products; the reductions in slices
    (300, 4096, 1024, 4104),     # two rounds of workgroups
    (4097, 136, 64, 264),        # one token beyond two rounds
])
def test_backward_products_in_one_launch(M, K, r, N):
    """dX, dA and dB of one layer from a single launch, against the oracle, between guard regions; each output has the same
    bits when others are left out and when H is recomputed."""
    import torch
    fhpc = _fhpc()
    X, A, B, dY = lowrank_inputs(12, M, K, r, N)
    ref = oracle.lowrank_bwd(X.f64, A.f64, B.f64, dY.f64)
    Xd, Ad, Bd, dYd = X.cuda(), A.cuda(), B.cuda(), dY.cuda()
    _, H = fhpc.lowrank_linear_fwd(Xd, Ad, Bd, save_H=True)
    guard = Guarded()
    g = [guard.alloc((M, K), torch.bfloat16), guard.alloc((K, r), torch.float32), guard.alloc((r, N), torch.float32)]
    out = fhpc.lowrank_linear_bwd(Xd, Ad, Bd, dYd, H_saved=H, dX=g[0], dA=g[1], dB=g[2])
    guard.check("one launch %s" % ((M, K, r, N),))
    _check_all("one launch %s" % ((M, K, r, N),), (None,) + out, (None,) + ref, TOL_BF16)
    for want in ((True, True, False), (True, False, True), (False, True, True), (False, True, False), (True, False, False)):
        some = fhpc.lowrank_linear_bwd(Xd, Ad, Bd, dYd, need_dX=want[0], need_dA=want[1], need_dB=want[2])
        assert all(s is None if not w else torch.equal(s, o) for s, o, w in zip(some, out, want)), want


@pytest.mark.parametrize("M,K,r,N,g", [
    (65, 264, 40, 520, 1),       # dX in the launch of the weight gradients
    (300, 4096, 1024, 4104, 1),
    (1100, 2056, 264, 776, 2),
    (33, 264, 40, 1032, 2),
    (40, 264, 40, 520, 1),       # few tokens: gradients on the vector ALU, dX by itself
    (4200, 2056, 40, 520, 1),    # dX by itself, beside a launch of the weight gradients
    (4200, 2056, 40, 520, 2),
])
def test_input_gradient_alone_has_the_bits_of_the_full_call(M, K, r, N, g):
    """dX of a frozen pair (no weight gradients wanted), of one layer and of g on one X."""
    import torch
    fhpc = _fhpc()
    X, A = Bf16.normal(1, (M, K)).cuda(), Bf16.normal(2, (K, g * r), K ** -0.5).cuda()
    Bs = [Bf16.normal(3 + i, (r, N), r ** -0.5).cuda() for i in range(g)]
    dYs = [Bf16.normal(20 + i, (M, N)).cuda() for i in range(g)]
    if g == 1:
        full = fhpc.lowrank_linear_bwd(X, A, Bs[0], dYs[0])
        alone = fhpc.lowrank_linear_bwd(X, A, Bs[0], dYs[0], need_dA=False, need_dB=False)
        assert alone[1] is None and alone[2] is None and bool((alone[0] == full[0]).all())
    full = fhpc.lowrank_linear_bwd_shared_x(X, A, Bs, dYs)
    alone = fhpc.lowrank_linear_bwd_shared_x(X, A, Bs, dYs, need_dA=False, need_dB=False)
    assert alone[1] is None and bool((alone[0] == full[0]).all())


@pytest.mark.parametrize("M,K,r,N,g", [
    (33, 264, 40, 1032, 2),      # few tokens; dH in slices into column blocks of 40
    (200, 520, 136, 1032, 3),    # all of it in one launch, dH in slices
    (1000, 264, 64, 2056, 8),    # the most layers on one X
])
def test_shared_x_backward_in_few_launches(M, K, r, N, g):
    """dH of all layers in slices of one launch and the products that follow it in another, against the oracle's single
    layers; each dB has the same bits when others are left out."""
    import torch
    fhpc = _fhpc()
    X, A = Bf16.normal(1, (M, K)), Bf16.normal(2, (K, g * r), K ** -0.5)
    Bs = [Bf16.normal(3 + i, (r, N), r ** -0.5) for i in range(g)]
    dYs = [Bf16.normal(20 + i, (M, N)) for i in range(g)]
    Xd, Ad, Bd, dYd = X.cuda(), A.cuda(), [b.cuda() for b in Bs], [d.cuda() for d in dYs]
    guard = Guarded()
    o = [guard.alloc((M, K), torch.bfloat16), guard.alloc((K, g * r), torch.float32), [guard.alloc((r, N), torch.float32) for _ in range(g)]]
    dX, dA, dBs = fhpc.lowrank_linear_bwd_shared_x(Xd, Ad, Bd, dYd, dX=o[0], dA_all=o[1], dBs=o[2])
    guard.check("shared one launch")
    rX = 0.0
    for i in range(g):
        a = A.f64[:, i * r:(i + 1) * r]
        x, da, db = oracle.lowrank_bwd(X.f64, np.ascontiguousarray(a), Bs[i].f64, dYs[i].f64)
        rX = rX + x
        assert parity_err(from_device(dA)[:, i * r:(i + 1) * r], da) <= TOL_BF16
        assert parity_err(from_device(dBs[i]), db) <= TOL_BF16
    assert parity_err(from_device(dX), rX) <= TOL_BF16
    _, dA2, dB2 = fhpc.lowrank_linear_bwd_shared_x(Xd, Ad, Bd, dYd, need_dX=False, need_dB=[i % 2 == 1 for i in range(g)])
    assert torch.equal(dA2, dA) and all(torch.equal(dB2[i], dBs[i]) for i in range(1, g, 2))


@pytest.mark.parametrize("M,K,r,N,g", [(40, 264, 16, 136, 3), (300, 1024, 64, 2048, 2), (2500, 520, 128, 512, 3)])
def test_shared_x_calls_write_their_scratch_before_they_read_it(M, K, r, N, g):
    """The binding hands the shared-X calls a workspace it has not cleared: with one full of NaN bit patterns they give
    the bits they give with a cleared one."""
    import torch
    fhpc = _fhpc()
    X, A = Bf16.normal(1, (M, K)).cuda(), Bf16.normal(2, (K, g * r), K ** -0.5).cuda()
    Bs = [Bf16.normal(3 + i, (r, N), r ** -0.5).cuda() for i in range(g)]
    dYs = [Bf16.normal(20 + i, (M, N)).cuda() for i in range(g)]
    got = []
    for fill in (0, 255):
        need = fhpc.load_library().fhpc_workspace_bytes_lowrank_shared_x(1, M, K, r, N, g)
        ws = torch.full((need,), fill, dtype=torch.uint8, device="cuda")
        Ys, H = fhpc.lowrank_linear_fwd_shared_x(X, A, Bs, save_H=True, workspace=ws)
        ws.fill_(fill)
        dX, dA, dBs = fhpc.lowrank_linear_bwd_shared_x(X, A, Bs, dYs, workspace=ws)
        ws.fill_(fill)
        gate_up = fhpc.lowrank_ffn_gate_up_fwd(X, A[:, :2 * r].contiguous(), Bs[0], Bs[1], save_H=True, workspace=ws)
        got.append([*Ys, H, dX, dA, *dBs, *gate_up])
    assert all(torch.equal(a, b) for a, b in zip(*got))


@pytest.mark.parametrize("M,K,r,N", [
    (1, 8, 8, 8),            # the smallest: one step of the reduction, most of it outside
    (16, 1536, 40, 1544),    # whole 16-row block; a reduction at the limit of the uncut ones, and one beyond it
    (17, 2056, 96, 520),     # one row beyond; slices that end inside a step
    (33, 1032, 1024, 264),   # the largest rank of these launches; more rows than one block
    (64, 4104, 72, 8456),    # all 64 tokens; wide outputs in 64-column tiles
])
def test_few_token_launches(M, K, r, N):
    """At most 64 tokens: rank products whole and in slices, outputs on both column tiles and the weight gradients beside
    them, against the oracle; each output has the same bits whatever else is asked for, and the header is left zero."""
    import torch
    fhpc = _fhpc()
    X = Bf16.normal(31, (M, K)); A = Bf16.normal(32, (K, r), K ** -0.5)
    B = Bf16.normal(33, (r, N), r ** -0.5); dY = Bf16.normal(34, (M, N))
    Yr, Hr = oracle.lowrank_fwd(X.f64, A.f64, B.f64)
    ref = (Yr,) + oracle.lowrank_bwd(X.f64, A.f64, B.f64, dY.f64)
    Xd, Ad, Bd, dYd = X.cuda(), A.cuda(), B.cuda(), dY.cuda()
    ws = torch.full((fhpc.workspace_bytes(fhpc.FHPC_OP_LOWRANK_BWD, M, K, r, N) + 4096,), 0xFF, dtype=torch.uint8, device="cuda")
    ws[:16384] = 0                                                   # (the header; everything behind it is written before it is read)
    guard = Guarded()
    g = [guard.alloc(s, t) for s, t in (((M, N), torch.bfloat16), ((M, r), torch.bfloat16), ((M, K), torch.bfloat16),
                                        ((K, r), torch.float32), ((r, N), torch.float32))]
    Y, H = fhpc.lowrank_linear_fwd(Xd, Ad, Bd, Y=g[0], H_out=g[1], workspace=ws)
    assert parity_err(from_device(H), Hr, TOL_BF16, "H") <= TOL_BF16
    out = fhpc.lowrank_linear_bwd(Xd, Ad, Bd, dYd, H_saved=H, dX=g[2], dA=g[3], dB=g[4], workspace=ws)
    _check_all("few %s" % ((M, K, r, N),), (Y,) + out, ref, TOL_BF16)
    guard.check("few %s" % ((M, K, r, N),))
    assert torch.equal(fhpc.lowrank_linear_fwd(Xd, Ad, Bd, workspace=ws), Y)
    assert all(torch.equal(a, b) for a, b in zip(fhpc.lowrank_linear_bwd(Xd, Ad, Bd, dYd, workspace=ws), out))     # H recomputed
    for i in range(3):
        only = fhpc.lowrank_linear_bwd(Xd, Ad, Bd, dYd, H_saved=H, need_dX=i == 0, need_dA=i == 1, need_dB=i == 2, workspace=ws)
        assert torch.equal(only[i], out[i])
    assert int(ws[:16384].sum()) == 0


def test_few_token_launches_replayed_from_a_graph():
    import torch
    fhpc = _fhpc()
    M, K, r, N = 5, 4096, 64, 2048
    A = Bf16.normal(41, (K, r), K ** -0.5).cuda(); B = Bf16.normal(42, (r, N), r ** -0.5).cuda()
    X = [Bf16.normal(43 + i, (M, K)).cuda() for i in range(4)]
    dY = [Bf16.normal(53 + i, (M, N)).cuda() for i in range(4)]
    def step(x, dy):
        Y, H = fhpc.lowrank_linear_fwd(x, A, B, save_H=True)
        return (Y, *fhpc.lowrank_linear_bwd(x, A, B, dy, H_saved=H))
    eager = [step(x, dy) for x, dy in zip(X, dY)]
    xs, dys = X[0].clone(), dY[0].clone()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        step(xs, dys)
    torch.cuda.current_stream().wait_stream(side)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        out = step(xs, dys)
    for i in range(4):
        xs.copy_(X[i]); dys.copy_(dY[i])
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(out, eager[i])), i
        step(X[3], dY[3])                                            # other work on the eager workspace between the replays


@pytest.mark.parametrize("M,K,r,N", [
    (100, 2000, 100, 2008),  # 32 x 32 tiles in 16 slices: as many slabs as the four waves take at a time
    (20, 4096, 130, 4104),   # in 32 slices, twice as many
    (1100, 4040, 170, 1928), # 64 x 64 tiles in four slices, the last step of the reduction outside; rank not a multiple of four
    (595, 2688, 101, 608),   # in 12, three times what a wave takes at a time
    (1098, 512, 119, 608),   # both weight gradients in seven, operands by 16 and by 4 bytes
    (5, 8, 129, 40),         # a reduction shorter than a step
])
def test_fp32_slices_on_uncleared_scratch(M, K, r, N):
    """The last slice to arrive at a tile adds the slabs: scratch full of NaN bit patterns gives the oracle's results, twice
    the same, and the header is left zero."""
    import torch
    fhpc = _fhpc()
    X, A, B, dY = lowrank_inputs(5, M, K, r, N, bf16=False)
    Yr, Hr = oracle.lowrank_fwd(X, A, B)
    ref = (Yr,) + oracle.lowrank_bwd(X, A, B, dY)
    Xd, Ad, Bd, dYd = (torch.from_numpy(a).cuda() for a in (X, A, B, dY))
    need = max(fhpc.workspace_bytes(op, M, K, r, N, fhpc.FHPC_F32) for op in (fhpc.FHPC_OP_LOWRANK_FWD, fhpc.FHPC_OP_LOWRANK_BWD))
    first = None
    for _ in range(2):
        ws = torch.full((need,), 0xFF, dtype=torch.uint8, device="cuda")
        ws[:16384] = 0                                               # (the header)
        Y, H = fhpc.lowrank_linear_fwd(Xd, Ad, Bd, save_H=True, workspace=ws)
        out = (Y,) + fhpc.lowrank_linear_bwd(Xd, Ad, Bd, dYd, H_saved=H, workspace=ws)
        assert int(ws[:16384].sum()) == 0
        if first is None:
            first = out
            _check_all("f32 slices %s" % ((M, K, r, N),), out, ref, TOL_F32)
        assert all(torch.equal(a, b) for a, b in zip(out, first))


@pytest.mark.parametrize("M,K,r,N", [
    (65, 264, 40, 72),        # one row and a part of a tile beyond 64; everything whole
    (127, 776, 64, 712),      # slices of a few steps, a rank of one tile exactly
    (128, 4104, 72, 568),     # many slices, the last one short; eight of 64 columns of the second tile
    (300, 2056, 16, 520),     # at most 32 wide: most of the tile outside
    (1000, 1600, 376, 1544),  # outputs of two workgroups per compute unit
    (2100, 1032, 264, 264),   # large and small tiles beside each other, a ragged last tile in both directions
    (8200, 520, 64, 1288),    # whole over many tokens
])
def test_small_tile_products(M, K, r, N):
    """Outputs with few large tiles run on 64 x 64 ones, whole or in slices: against the oracle, inside their buffers, from scratch
    that nobody cleared, and with the same bits whether H is saved or formed again."""
    import torch
    fhpc = _fhpc()
    X = Bf16.normal(61, (M, K)); A = Bf16.normal(62, (K, r), K ** -0.5)
    B = Bf16.normal(63, (r, N), r ** -0.5); dY = Bf16.normal(64, (M, N))
    Yr, Hr = oracle.lowrank_fwd(X.f64, A.f64, B.f64)
    ref = (Yr,) + oracle.lowrank_bwd(X.f64, A.f64, B.f64, dY.f64)
    Xd, Ad, Bd, dYd = X.cuda(), A.cuda(), B.cuda(), dY.cuda()
    ws = torch.full((fhpc.workspace_bytes(fhpc.FHPC_OP_LOWRANK_BWD, M, K, r, N) + 4096,), 0xFF, dtype=torch.uint8, device="cuda")
    ws[:16384] = 0
    guard = Guarded()
    g = [guard.alloc(s, t) for s, t in (((M, N), torch.bfloat16), ((M, r), torch.bfloat16), ((M, K), torch.bfloat16),
                                        ((K, r), torch.float32), ((r, N), torch.float32))]
    Y, H = fhpc.lowrank_linear_fwd(Xd, Ad, Bd, Y=g[0], H_out=g[1])
    assert parity_err(from_device(H), Hr, TOL_BF16, "H") <= TOL_BF16
    out = fhpc.lowrank_linear_bwd(Xd, Ad, Bd, dYd, H_saved=H, dX=g[2], dA=g[3], dB=g[4], workspace=ws)
    _check_all("small tiles %s" % ((M, K, r, N),), (Y,) + out, ref, TOL_BF16)
    guard.check("small tiles %s" % ((M, K, r, N),))
    assert all(torch.equal(a, b) for a, b in zip(fhpc.lowrank_linear_bwd(Xd, Ad, Bd, dYd, workspace=ws), out))


def test_graphs_in_one_pool_replayed_in_any_order():
    """Calls without a workspace, captured: each graph clears the arrival counters it uses, so that neither the order of the replays
    nor what another graph of the pool left in the memory changes a result."""
    import torch
    fhpc = _fhpc()
    def layer(i, M, K, r, N, t):
        X, A, B, dY = (torch.from_numpy(a).to(t).cuda() for a in lowrank_inputs(i, M, K, r, N, bf16=False))
        def step():
            Y, H = fhpc.lowrank_linear_fwd(X, A, B, save_H=True)
            return (Y, *fhpc.lowrank_linear_bwd(X, A, B, dY, H_saved=H))
        return step
    steps = [layer(1, 5, 4096, 64, 2048, torch.bfloat16), layer(2, 300, 2048, 64, 520, torch.float32), layer(3, 40, 2056, 96, 4104, torch.bfloat16)]
    eager = [[t.clone() for t in s()] for s in steps]
    torch.cuda.synchronize()
    fill = torch.cuda.CUDAGraph()
    with torch.cuda.graph(fill):
        for n in (1 << 14, 1 << 19, 1 << 21, 1 << 25):
            torch.empty(n, dtype=torch.uint8, device="cuda").fill_(0xFF)        # freed: the other graphs' memory
    graphs, outs = [], []
    for s in steps:
        graphs.append(torch.cuda.CUDAGraph())
        with torch.cuda.graph(graphs[-1], pool=fill.pool()):
            outs.append(s())
    assert all(type(t) is torch.Tensor for t in fhpc._workspaces.values()) and len(fhpc._capture_workspaces) <= 1
    for i in (2, 1, 0, 1, 2, 0):
        fill.replay()
        graphs[i].replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(outs[i], eager[i])), i
        assert all(torch.equal(a, b) for a, b in zip(steps[0](), eager[0])), i      # eager work between the replays
    assert not fhpc._capture_workspaces


@pytest.mark.parametrize("M,K,r,N", [
    (4100, 1032, 195, 776),   # both weight gradients on 64 x 64 tiles; the last step of the reduction over the rank holds three
    (70, 264, 45, 136),       # 32 x 32 tiles, everything whole
    (1000, 1600, 66, 2056),   # rows of the rank 8-byte aligned; 32 x 32 tiles in slices
])
def test_fp32_ranks_that_are_not_a_multiple_of_four(M, K, r, N):
    """X, dY and B by 16 bytes beside A, H and dH by four, in every product alone and in the launch that carries both weight gradients."""
    import torch
    fhpc = _fhpc()
    X, A, B, dY = lowrank_inputs(6, M, K, r, N, bf16=False)
    Yr, Hr = oracle.lowrank_fwd(X, A, B)
    Xd, Ad, Bd, dYd = (torch.from_numpy(a).cuda() for a in (X, A, B, dY))
    guard = Guarded()
    g = [guard.alloc(s, torch.float32) for s in ((M, N), (M, r), (M, K), (K, r), (r, N))]
    Y, H = fhpc.lowrank_linear_fwd(Xd, Ad, Bd, Y=g[0], H_out=g[1])
    out = fhpc.lowrank_linear_bwd(Xd, Ad, Bd, dYd, H_saved=H, dX=g[2], dA=g[3], dB=g[4])
    _check_all("f32 rank %s" % ((M, K, r, N),), (Y,) + out, (Yr,) + oracle.lowrank_bwd(X, A, B, dY), TOL_F32)
    assert parity_err(from_device(H), Hr, TOL_F32, "H") <= TOL_F32
    guard.check("f32 rank %s" % ((M, K, r, N),))
    for i in range(3):
        only = fhpc.lowrank_linear_bwd(Xd, Ad, Bd, dYd, H_saved=H, need_dX=i == 0, need_dA=i == 1, need_dB=i == 2)
        assert torch.equal(only[i], out[i])


@pytest.mark.parametrize("M,r", [(1, 8), (13, 64), (32, 40), (33, 64)])
def test_shared_x_outputs_of_few_tokens_share_a_launch(M, r):
    import torch
    fhpc = _fhpc()
    K, N, g = 520, 776, 3
    X = Bf16.normal(71, (M, K)); A = [Bf16.normal(72 + i, (K, r), K ** -0.5) for i in range(g)]; B = [Bf16.normal(82 + i, (r, N), r ** -0.5) for i in range(g)]
    args = (X.cuda(), torch.cat([a.cuda() for a in A], 1).contiguous(), [b.cuda() for b in B])
    fhpc.profile_start(64)
    Ys = fhpc.lowrank_linear_fwd_shared_x(*args)
    assert sum(name.startswith("gemm") for name, *_ in fhpc.profile_stop()) == 2          # X A_all, and the outputs
    for Y, a, b in zip(Ys, A, B):
        assert parity_err(from_device(Y), oracle.lowrank_fwd(X.f64, a.f64, b.f64)[0], TOL_BF16, "Y") <= TOL_BF16


def _fp32_launches(fhpc, call):
    """What `call` returns, and the names of the fp32 products it launched."""
    fhpc.profile_start(64)
    try:
        out = call()
    finally:
        names = [name for name, *_ in fhpc.profile_stop()]
    return out, [n for n in names if n.startswith("gemm_f32")]


def _fp32_tiles(names):
    """Of each launch: "-" on the fp32 instructions; on three-part operands the tile's edge, "s" if in slices, and after a "/" the operands loaded
    by 16 bytes (bits 0 and 1 a and b of the first product, 2 and 3 of the second) where not all are."""
    import re
    out = []
    for n in names:
        kind, tile, vec, s0, s1 = re.match(r"gemm_f32(x3)?<(\d+),a\d,b\d,v(\d+),s(\d+)\+(\d+)>", n).groups()
        out.append(tile + "s" * (max(int(s0), int(s1)) > 1) + ("" if vec == "15" else "/" + vec) if kind else "-")
    return out


@pytest.mark.parametrize("M,K,r,N,tiles", [       # tiles of H, Y, dH, dX and both weight gradients
    (2050, 1032, 132, 4104, ["-", "64", "64s", "-", "64s"]),             # two rows and eight columns beyond the tiles; four ranks beyond
    (4100, 2008, 256, 1000, ["128s", "64", "128s", "128", "128s"]),      # everything on three-part operands; reductions that end inside a trip of 64
    (8185, 776, 191, 3080, ["-", "128/10", "-", "-", "-"]),              # odd rank and token count
    (520, 4096, 250, 4104, ["-", "-", "-", "-", "-"]),                   # few rows: all on the fp32 instructions
    (4406, 1488, 40, 1664, ["64s", "128", "64s", "64", "64s"]),          # fewer ranks than a tile
    (2689, 2808, 103, 264, ["128s/5", "-", "-", "128/0", "128s/9"]),     # words of the rank by four bytes: one operand, both, one of each product
    (6366, 256, 228, 312, ["64", "64", "64", "64", "128s"]),             # short reductions, whole
    (165, 4088, 232, 2760, ["-", "-", "-", "-", "64"]),                  # weight gradients over few tokens, whole
    (5185, 256, 33, 2224, ["-", "128/10", "-", "-", "-"]),               # a reduction of 33
])
def test_fp32_products_in_three_parts(M, K, r, N, tiles):
    """Large fp32 products multiply bf16 parts: as close to the oracle as fp32 sums are.  1e-6: a chain of 4104 fp32 additions of terms
    without order is off by sqrt(4104 / 3) 2^-24 = 2.2e-6 at most where every partial sum is as large as the last; sums of 64 apart,
    that is 4.6e-7 and three times that in the parts' roundings and the second product."""
    import torch
    fhpc = _fhpc()
    X, A, B, dY = lowrank_inputs(9, M, K, r, N, bf16=False)
    Yr, Hr = oracle.lowrank_fwd(X, A, B)
    ref = (Yr,) + oracle.lowrank_bwd(X, A, B, dY)
    Xd, Ad, Bd, dYd = (torch.from_numpy(a).cuda() for a in (X, A, B, dY))
    guard = Guarded()
    g = [guard.alloc(s, torch.float32) for s in ((M, N), (M, r), (M, K), (K, r), (r, N))]
    ws = torch.full((max(fhpc.workspace_bytes(op, M, K, r, N, fhpc.FHPC_F32) for op in (fhpc.FHPC_OP_LOWRANK_FWD, fhpc.FHPC_OP_LOWRANK_BWD)),),
                    0xFF, dtype=torch.uint8, device="cuda")
    ws[:16384] = 0
    (Y, H), fwd = _fp32_launches(fhpc, lambda: fhpc.lowrank_linear_fwd(Xd, Ad, Bd, Y=g[0], H_out=g[1], workspace=ws))
    assert parity_err(from_device(H), Hr, 1e-6, "H") <= 1e-6
    out, bwd = _fp32_launches(fhpc, lambda: fhpc.lowrank_linear_bwd(Xd, Ad, Bd, dYd, H_saved=H, dX=g[2], dA=g[3], dB=g[4], workspace=ws))
    assert _fp32_tiles(fwd + bwd) == tiles
    _check_all("f32 parts %s" % ((M, K, r, N),), (Y,) + out, ref, 1e-6)
    guard.check("f32 parts %s" % ((M, K, r, N),))
    again = fhpc.lowrank_linear_bwd(Xd, Ad, Bd, dYd)                  # H recomputed
    assert all(torch.equal(a, b) for a, b in zip(out, again))
    for i in range(3):
        only = fhpc.lowrank_linear_bwd(Xd, Ad, Bd, dYd, H_saved=H, need_dX=i == 0, need_dA=i == 1, need_dB=i == 2)
        assert torch.equal(only[i], out[i])


@pytest.mark.parametrize("where", ["X", "A", "B", "dY"])
def test_fp32_subnormal_words_in_three_parts(where):
    """Subnormal words beside words of about 1e30, every product on three-part operands: the results are ordinary numbers and made of
    those words alone, in an input gradient, a forward output or H.  The words are exact in three parts, so each result has the accuracy of
    a single product carried through two sums: 1e-6."""
    import torch
    fhpc = _fhpc()
    M, K, r, N = 4100, 2008, 256, 1000
    X, A, B, dY = lowrank_inputs(12, M, K, r, N, bf16=False)
    # (multiples of 2^-149 = 1.4e-45; those of the first tile of rows below 2^-134, which bf16 rounds to zero)
    sub = np.float32([1e-41, -3e-42, 2.2e-44, 4.5e-41, 1e-44, 9e-39, -4.6e-41, 1e-38])
    rows = np.r_[300:305, 1000:1003]
    if where == "X":                                                  # H = X A
        X[:, 7], X[rows] = 0, 0
        X[rows, 7] = sub
        A[7] *= np.float32(1e30)
    elif where == "dY":                                               # dH = dY B^T
        dY[:, 5], dY[rows] = 0, 0
        dY[rows, 5] = sub
        B[:, 5] *= np.float32(1e30)
    elif where == "A":
        A[9], A[:, 3] = 0, 0
        A[9, 3] = sub[0]
        X[:, 9] *= np.float32(1e30)
    else:                                                             # Y = H B
        A[:, 3] *= np.float32(1e30)
        B[3], B[:, 11] = 0, 0
        B[3, 11] = sub[0]
    d = [torch.from_numpy(t).cuda() for t in (X, A, B, dY)]
    (Y, H), fwd = _fp32_launches(fhpc, lambda: fhpc.lowrank_linear_fwd(*d[:3], save_H=True))
    (dX, dA, dB), bwd = _fp32_launches(fhpc, lambda: fhpc.lowrank_linear_bwd(*d, H_saved=H))
    assert len(fwd) == 2 and len(bwd) == 3 and all(n.startswith("gemm_f32x3<") for n in fwd + bwd), (fwd, bwd)
    X, A, B, dY = (t.astype(np.float64) for t in (X, A, B, dY))
    if where == "X":
        pairs = [(H[rows], X[rows] @ A), (Y[rows], X[rows] @ A @ B)]
    elif where == "dY":
        pairs = [(dX[rows], dY[rows] @ B.T @ A.T)]
    elif where == "A":
        pairs = [(H[:, 3:4], X @ A[:, 3:4])]
    else:
        pairs = [(Y[:, 11:12], X @ A @ B[:, 11:12])]
    for got, ref in pairs:
        got = from_device(got)
        for g, f in zip(got, ref) if where in ("X", "dY") else [(got, ref)]:
            assert np.linalg.norm(f) > 0 and np.linalg.norm(g - f) <= 1e-6 * np.linalg.norm(f), where


def _elementwise(got, ref, size, what):
    """Non-finite where `ref` is, and each element within 4e-6 of `size`, the product of the operands' magnitudes: the sums of a launch round
    some 60 times (24 in a trip, as many trips and slabs), 60 x 2^-24 = 3.6e-6; what falls below the normal numbers besides."""
    got = from_device(got)
    ok = np.isfinite(ref)
    assert np.array_equal(got[~ok], ref[~ok], equal_nan=True), what
    assert np.all(np.abs(got[ok] - ref[ok]) <= 4e-6 * size[ok] + 1e-40), what


@pytest.mark.parametrize("M,K,r,N,tiles", [
    (4100, 2008, 256, 1000, ["128s", "64", "128s", "128", "128s"]),       # H, Y, dH, dX, both weight gradients; s: in slices
    (8192, 768, 192, 3072, ["64s", "128", "128s", "64", "128s"]),
    (4406, 1488, 40, 1664, ["64s", "128", "64s", "64", "64s"]),
    (2689, 2808, 103, 264, ["128s/5", "-", "-", "128/0", "128s/9"]),
])
@pytest.mark.parametrize("where", ["X", "A", "B", "dY", "X inf", "dY nan"])
def test_fp32_tiles_formed_again(M, K, r, N, tiles, where):
    """One word that does not come in three parts, 3.4e38 beside small ones so that results are finite, an infinity or a NaN: its tiles are formed
    again on the fp32 instructions, whole, in slices beside other slabs, and in every layout; all elements of all outputs."""
    import torch
    fhpc = _fhpc()
    X, A, B, dY = lowrank_inputs(13, M, K, r, N, bf16=False)
    top, f = np.float32(3.4e38), np.float32
    if where == "X":
        A[5] *= f(1e-20); dY[700] *= f(1e-20); X[700, 5] = top
    elif where == "A":
        X[:, 5] *= f(1e-30); B[3] *= f(1e-8); A[5, 3] = top
    elif where == "B":
        A[:, 3] *= f(1e-30); dY[:, 5] *= f(1e-30); B[3, 5] = top
    elif where == "dY":
        B[:, 5] *= f(1e-20); X[700] *= f(1e-18); dY[700, 5] = top
    elif where == "X inf":
        X[700, 5] = np.inf
    else:
        dY[700, 5] = np.nan
    d = [torch.from_numpy(t).cuda() for t in (X, A, B, dY)]
    (Y, H), fwd = _fp32_launches(fhpc, lambda: fhpc.lowrank_linear_fwd(*d[:3], save_H=True))
    (dX, dA, dB), bwd = _fp32_launches(fhpc, lambda: fhpc.lowrank_linear_bwd(*d, H_saved=H))
    assert _fp32_tiles(fwd + bwd) == tiles
    X, A, B, dY = (t.astype(np.float64) for t in (X, A, B, dY))
    Hd = from_device(H)
    with np.errstate(invalid="ignore"):
        m = [np.abs(t) for t in (X, A, B, dY, Hd)]
        dH, mH = dY @ B.T, m[3] @ m[2].T
        _elementwise(H, X @ A, m[0] @ m[1], "H")
        _elementwise(Y, Hd @ B, m[4] @ m[2], "Y")
        _elementwise(dX, dH @ A.T, 2 * (mH @ m[1].T), "dX")
        _elementwise(dA, X.T @ dH, 2 * (m[0].T @ mH), "dA")
        _elementwise(dB, Hd.T @ dY, m[4].T @ m[3], "dB")


def test_fp32_three_parts_are_as_exact_as_the_fp32_instructions():
    """Relative errors no larger than those of the fp32 instructions' tiles for the same operands, 1.92 1.21 2.29 2.46 2.12e-7.  H, two slices of
    six trips of 64 k: roundings of the variance of 4.5 (in trips) + 3.3 (trips) + 1 (slabs) final ones, .42 x 2^-24 each: 7.4e-8."""
    import torch
    fhpc = _fhpc()
    d = [torch.from_numpy(t).cuda() for t in lowrank_inputs(15, 8192, 768, 192, 3072, bf16=False)]
    (Y, H), fwd = _fp32_launches(fhpc, lambda: fhpc.lowrank_linear_fwd(*d[:3], save_H=True))
    (dX, dA, dB), bwd = _fp32_launches(fhpc, lambda: fhpc.lowrank_linear_bwd(*d, H_saved=H))
    assert all(n.startswith("gemm_f32x3<") for n in fwd + bwd), (fwd, bwd)
    X, A, B, dY = (t.double() for t in d)
    Hr, dHr = X @ A, dY @ B.T.contiguous()
    for name, got, ref, most in (("Y", Y, Hr @ B, 1.92e-7), ("H", H, Hr, 1.0e-7), ("dX", dX, dHr @ A.T.contiguous(), 2.29e-7),
                                 ("dA", dA, X.T.contiguous() @ dHr, 2.46e-7), ("dB", dB, Hr.T.contiguous() @ dY, 2.12e-7)):
        err = float((got.double() - ref).norm() / ref.norm())
        print(name, "rel %.3e" % err, flush=True)
        assert err <= most, (name, err)


def test_fp32_tiles_formed_again_take_their_time():
    """Every tile formed twice, on both kinds of instruction, takes 2.3 times as long as once; word by word from memory it took 7.7 times as long."""
    import torch
    fhpc = _fhpc()
    X, A, B, dY = (torch.from_numpy(t).cuda() for t in lowrank_inputs(14, 8192, 768, 192, 3072, bf16=False))

    def shortest():
        times = []
        for _ in range(6):
            e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            e[0].record()
            Y, H = fhpc.lowrank_linear_fwd(X, A, B, save_H=True)
            fhpc.lowrank_linear_bwd(X, A, B, dY, H_saved=H)
            e[1].record()
            e[1].synchronize()
            times.append(e[0].elapsed_time(e[1]))
        return min(times)

    plain = shortest()
    X.view(-1)[::997] = float("nan")
    dY.view(-1)[::997] = float("nan")
    assert shortest() <= 4 * plain


def test_fp32_words_that_do_not_come_in_parts():
    """Tokens of about 1e-36, of infinities, of the largest finite words and of zeros beside ordinary ones in one tile of a layer whose Y runs on
    three-part operands: every token has the accuracy of its own magnitude and nothing else meets the infinities."""
    import torch
    fhpc = _fhpc()
    M, K, r, N = 2048, 1024, 128, 4096
    X, A, B, _ = lowrank_inputs(10, M, K, r, N, bf16=False)
    tiny, inf, zero, top = slice(300, 310), 700, slice(1000, 1200), 1300
    X[tiny] *= np.float32(1e-36)
    X[zero] = 0
    X[inf, 5] = np.inf
    X[top] = 0
    X[top, 9] = np.float32(3.4e38)                                    # rounds to an infinity in bf16
    A[5], A[9] = np.abs(A[5]) + 0.1, np.clip(A[9], -0.5, 0.5)
    Y, H = (from_device(t) for t in fhpc.lowrank_linear_fwd(*(torch.from_numpy(a).cuda() for a in (X, A, B)), save_H=True))
    rows = np.setdiff1d(np.arange(M), [inf])
    Hr = X[rows].astype(np.float64) @ A.astype(np.float64)
    assert np.all(H[inf] == np.inf) and np.all(np.isinf(Y[inf]) | np.isnan(Y[inf]))
    assert np.all(H[zero] == 0) and np.all(Y[zero] == 0)
    part = [int(i) for i in range(0, len(rows), 37)] + [int(np.searchsorted(rows, t)) for t in (300, 305, 309, top)]
    for i in part:
        n = np.linalg.norm(Hr[i])
        assert np.linalg.norm(H[rows[i]] - Hr[i]) <= 1e-6 * n, rows[i]
    part = [i for i in part if rows[i] != top]                        # (its H times B overflows here and there)
    Yr = Hr[part] @ B.astype(np.float64)
    for i, y in zip(part, Yr):
        assert np.linalg.norm(Y[rows[i]] - y) <= 2e-6 * np.linalg.norm(y), rows[i]


def test_fp32_workspace_of_the_fp32_instructions_plans():
    """A workspace too small for operands in three parts, as large as the fp32 instructions' slabs, is enough: 6175232 bytes here."""
    import torch
    fhpc = _fhpc()
    M, K, r, N = 2050, 1032, 132, 4104
    X, A, B, dY = lowrank_inputs(11, M, K, r, N, bf16=False)
    Xd, Ad, Bd, dYd = (torch.from_numpy(a).cuda() for a in (X, A, B, dY))
    assert fhpc.workspace_bytes(fhpc.FHPC_OP_LOWRANK_BWD, M, K, r, N, fhpc.FHPC_F32) > 6175232
    ws = torch.full((6175232 + 4096,), 0xFF, dtype=torch.uint8, device="cuda")
    ws[:16384] = 0
    out = fhpc.lowrank_linear_bwd(Xd, Ad, Bd, dYd, workspace=ws[:6175232])
    assert int(ws[:16384].sum()) == 0 and bool((ws[6175232:] == 0xFF).all())
    _check_all("f32 tight", (None,) + out, (None,) + oracle.lowrank_bwd(X, A, B, dY), TOL_F32)
    with pytest.raises(fhpc.FhpcError):
        fhpc.lowrank_linear_bwd(Xd, Ad, Bd, dYd, workspace=ws[:2000000])
