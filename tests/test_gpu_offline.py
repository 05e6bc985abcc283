"""GPU tests of the offline pipeline (moe_lrc_offline_*) against oracle/compress.py.

Quantizer: codes, scales, zeros and the residual bit for bit (both sides work in fp64 and round the
scale and zero to fp16 before choosing codes).  Factors: what is unique about them — the singular
values, the product A B, the factors up to the sign of each pair — against the oracle's subspace
iteration on the same test matrix, and the approximation error against the exact SVD's optimum
(Eckart-Young).  Kurtosis to 1e-12.  End to end: a layer compressed on the device, loaded through the
C ABI and run, against the forward oracle on the same artefacts.
"""
import numpy as np
import pytest

from oracle import compress, fixtures
from oracle import moe_lrc_oracle as orc
from workload import configs, synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def amd():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    import paper_2512_17073_amd as amd
    amd.lib()
    return amd


def _dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _bits(t):
    return t.cpu().numpy().view(np.uint16)


@pytest.mark.parametrize("bits,group,K,N", [(2, 64, 512, 384), (3, 64, 256, 528), (4, 128, 512, 272), (3, 256, 768, 100)])
def test_quantizer_bit_exact(amd, bits, group, K, N):
    rng = np.random.default_rng(bits * 1000 + group)
    W = rng.standard_normal((K, N)) * 0.02
    W *= 1.0 + 4.0 * (rng.random((K, N)) < 0.01)            # heavy tails
    W[:group, 0] = 0.0                                      # a group of zeros
    W[:group, 1] = 0.3125                                   # a constant group
    W[group:2 * group, 2] *= 1e-9                           # a scale that rounds to zero in fp16
    W[:group, 3] *= 1e7                                     # a scale beyond fp16
    W[:group, 4] = np.linspace(-1.0, 1.0, group)            # exact ties between codes
    want = compress.quantize_groupwise(W, bits, group)
    codes, scale, zero, resid = amd.offline_quantize(_dev(W), bits, group)
    np.testing.assert_array_equal(codes.cpu().numpy(), want["codes"])
    np.testing.assert_array_equal(_bits(scale), want["scale"])
    np.testing.assert_array_equal(_bits(zero), want["zero"])
    E = W - compress.dequantize(want, group)
    np.testing.assert_array_equal(resid.cpu().numpy(), E)
    # what the quantizer promises: no code of a regular group is more than half a step off
    s = np.repeat(orc.f16_to_f64(want["scale"]), group, axis=0)
    regular = np.repeat(np.ptp(W.reshape(K // group, group, N), axis=1) < 6e4, group, axis=0)
    assert (np.abs(E)[regular] <= 0.5 * s[regular] * (1 + 2e-3) + 1e-12).all()


@pytest.mark.parametrize("bits,group", [(2, 64), (3, 64), (4, 128)])
def test_refined_quantizer_against_the_oracle(amd, bits, group):
    rng = np.random.default_rng(40 + bits)
    K, N = 512, 320
    W = rng.standard_normal((K, N)) * 0.02
    W *= 1.0 + 9.0 * (rng.random((K, N)) < 0.01)
    W[:group, 0] = 0.25                                     # a constant group
    want = compress.quantize_refined(W, bits, group)
    codes, scale, zero, resid = amd.offline_quantize(_dev(W), bits, group, refine={})
    codes, scale, zero = codes.cpu().numpy(), _bits(scale), _bits(zero)
    np.testing.assert_array_equal(scale, want["scale"])
    # The zero point comes out of twenty steps that call pow(); the two libraries' pow may differ in
    # the last bit, which can move a zero point that sits on a rounding boundary: allow one group in
    # ten thousand to differ by one fp16 step (and its codes by one), nothing else.
    dz = zero.astype(np.int64) - want["zero"].astype(np.int64)
    assert (np.abs(dz) <= 1).all() and (dz != 0).mean() <= 1e-4
    dc = codes.astype(np.int64) - want["codes"].astype(np.int64)
    assert (np.abs(dc) <= 1).all() and (dc != 0).mean() <= 1e-4
    got = {"codes": codes, "scale": scale, "zero": zero}
    lp = lambda q: (np.abs(W - compress.dequantize(q, group)) ** 0.7).sum()
    assert abs(lp(got) - lp(want)) <= 1e-6 * lp(want)
    assert lp(got) < lp(compress.quantize_groupwise(W, bits, group))
    np.testing.assert_array_equal(resid.cpu().numpy(), W - compress.dequantize(got, group))
    # no steps: the plain quantizer, bit for bit
    c0, s0, z0, _ = amd.offline_quantize(_dev(W), bits, group, refine={"iters": 0})
    base = compress.quantize_groupwise(W, bits, group)
    np.testing.assert_array_equal(c0.cpu().numpy(), base["codes"])
    np.testing.assert_array_equal(_bits(z0), base["zero"])


# odd widths (one column per lane), a single column, every register form and a group that has none
@pytest.mark.parametrize("bits,group,K,N", [(2, 32, 96, 63), (3, 64, 128, 129), (4, 128, 256, 1), (2, 256, 256, 65), (3, 48, 96, 70), (2, 32, 32, 2)])
def test_quantizer_at_the_edges(amd, bits, group, K, N):
    rng = np.random.default_rng(K * N + group)
    W = rng.standard_normal((K, N)) * 0.02
    W[:group, 0] = 0.0
    want = compress.quantize_groupwise(W, bits, group)
    codes, scale, zero, resid = amd.offline_quantize(_dev(W), bits, group)
    np.testing.assert_array_equal(codes.cpu().numpy(), want["codes"])
    np.testing.assert_array_equal(_bits(scale), want["scale"])
    np.testing.assert_array_equal(_bits(zero), want["zero"])
    np.testing.assert_array_equal(resid.cpu().numpy(), W - compress.dequantize(want, group))


# entries on both sides of the threshold below which shrink() is zero (beta = 10 puts it at 0.17: far
# above every error; 3e3 and 3e4 put it inside their range), with and without the register form
@pytest.mark.parametrize("group,beta", [(32, 10.0), (64, 3e3), (64, 3e4), (96, 3e3)])
def test_refined_quantizer_around_its_threshold(amd, group, beta):
    rng = np.random.default_rng(int(beta) + group)
    W = rng.standard_normal((192, 75)) * 0.02
    want = compress.quantize_refined(W, 3, group, beta=beta)
    codes, scale, zero, _ = amd.offline_quantize(_dev(W), 3, group, refine={"beta": beta})
    np.testing.assert_array_equal(_bits(scale), want["scale"])
    # as above: the last bit of pow() may move a value over a rounding boundary
    dz = _bits(zero).astype(np.int64) - want["zero"].astype(np.int64)
    assert (np.abs(dz) <= 1).all() and (dz != 0).sum() <= 1
    dc = codes.cpu().numpy().astype(np.int64) - want["codes"].astype(np.int64)
    assert (np.abs(dc) <= 1).all() and (dc != 0).sum() <= 2


@pytest.mark.parametrize("group", [32, 48, 64])
@pytest.mark.parametrize("beta,kappa,iters", [(1e-310, 1e155, 6), (1e-300, 1e100, 5), (1e300, 1.0, 3), (10.0, float("inf"), 3)])
def test_refined_quantizer_with_extreme_penalties(amd, group, beta, kappa, iters):
    """p = 1: the threshold is 1 / beta, which fp64 cannot hold for a subnormal beta, also after the penalty has grown
    to where the threshold matters."""
    W = np.random.default_rng(group).standard_normal((192, 70)) * 0.02
    want = compress.quantize_refined(W, 3, group, iters=iters, p=1.0, beta=beta, kappa=kappa)
    codes, scale, zero, _ = amd.offline_quantize(_dev(W), 3, group, refine={"iters": iters, "p": 1.0, "beta": beta, "kappa": kappa})
    np.testing.assert_array_equal(_bits(scale), want["scale"])
    np.testing.assert_array_equal(_bits(zero), want["zero"])
    np.testing.assert_array_equal(codes.cpu().numpy(), want["codes"])


def test_kurtosis(amd):
    rng = np.random.default_rng(3)
    for W in (rng.standard_normal((700, 513)), rng.laplace(size=(300, 1001)) * 0.05 + 0.01, rng.random((257, 129))):
        want = compress.kurtosis(W)
        got = amd.offline_kurtosis(_dev(W))
        assert abs(got - want) <= 1e-12 * want, (got, want)


def _aligned(A, B, A0, B0):
    sign = np.sign(np.sum(A * A0, axis=0))
    return A * sign[None, :], B * sign[:, None]


@pytest.mark.parametrize("power,rel", [(247, 1e-12), (-250, 1e-12), (-260, 1e-9)])
def test_kurtosis_of_very_large_and_very_small_values(amd, power, rel):
    """A ratio of moments does not change with the scale; while the fourth powers fit fp64 it is finite, whatever
    the number of entries (2^-1040, the fourth power of 2^-260, is a subnormal with 34 bits: 6e-11 each)."""
    W = np.random.default_rng(3).standard_normal((1024, 1031))
    want = compress.kurtosis(W)
    assert abs(amd.offline_kurtosis(_dev(W * 2.0 ** power)) - want) <= rel * want


@pytest.mark.parametrize("K,N", [(96, 70), (64, 129), (256, 130)])
def test_kurtosis_of_a_constant_matrix(amd, K, N):
    """0 / 0 up to rounding: never below 1, the least a kurtosis can be (or NaN where the mean is exact)."""
    assert not amd.offline_kurtosis(_dev(np.full((K, N), 0.3))) < 1.0


@pytest.mark.parametrize("K,N,r,bits", [(256, 512, 8, 3), (512, 768, 40, 2), (1024, 640, 16, 2), (384, 384, 128, 4)])
def test_residual_factors(amd, K, N, r, bits):
    rng = np.random.default_rng(K + N + r)
    W = rng.standard_normal((K, N)) * 0.02
    W *= 1.0 + 4.0 * (rng.random((K, N)) < 0.01)
    q = compress.quantize_groupwise(W, bits, 64)
    E = W - compress.dequantize(q, 64)
    seed, l = 11, r + 8
    omega = np.random.default_rng(seed).standard_normal((N, l))    # what the oracle's "randomized" method draws
    A0, B0, S0 = compress.residual_factors(E, r, method="randomized", seed=seed, power_iters=2)
    A, B, sigma, Ab, Bb = amd.offline_factors(_dev(E), r, _dev(omega), power_iters=2)
    A, B = A.cpu().numpy(), B.cpu().numpy()
    np.testing.assert_allclose(sigma, S0, rtol=1e-9)
    assert (np.diff(sigma) <= 0).all()
    assert orc.rel_frobenius(A @ B, A0 @ B0) <= 1e-8
    # Section 3.1 step 2's reparameterisation: A^T A = B B^T = diag(sigma)
    np.testing.assert_allclose(A.T @ A, np.diag(sigma), atol=1e-9 * sigma[0])
    np.testing.assert_allclose(B @ B.T, np.diag(sigma), atol=1e-9 * sigma[0])
    # the factors themselves, up to the sign of each pair (the singular values of a quantizer's
    # residual are close together, so single vectors are less well determined than the product)
    As, Bs = _aligned(A, B, A0, B0)
    assert orc.rel_frobenius(As, A0) <= 1e-5 and orc.rel_frobenius(Bs, B0) <= 1e-5
    # against the exact SVD: never better than the optimum, and as close to it as the oracle's iteration
    Sx = np.linalg.svd(E, compute_uv=False)
    best = np.sqrt((Sx[r:] ** 2).sum())
    err, err0 = np.linalg.norm(E - A @ B), np.linalg.norm(E - A0 @ B0)
    assert best * (1 - 1e-12) <= err <= err0 * (1 + 1e-9) and err <= best * 1.05
    # stored form: the same rounding to bf16 as the oracle's
    np.testing.assert_array_equal(_bits(Ab), compress.round_to_bf16_bits(A))
    np.testing.assert_array_equal(_bits(Bb), compress.round_to_bf16_bits(B))


# edges of the tiles and of the choice between the one-block and the many-launch SVD: l odd, l = 96 (the
# largest that fits one block's LDS) and 97, fewer than 32 rows in a transposed product, K and N that
# are no multiple of a chunk, a single pair
@pytest.mark.parametrize("K,N,r,over,iters", [(70, 97, 24, 9, 2), (131, 161, 88, 8, 1), (131, 161, 89, 8, 1), (33, 45, 3, 2, 2),
                                              (1000, 131, 8, 0, 0), (64, 64, 1, 0, 1), (129, 777, 40, 9, 2)])
def test_residual_factors_at_the_edges(amd, K, N, r, over, iters):
    rng = np.random.default_rng(K * N + r)
    E, omega = rng.standard_normal((K, N)), rng.standard_normal((N, r + over))
    Y = E @ omega
    for _ in range(iters):
        Y = E @ (E.T @ np.linalg.qr(Y)[0])
    Q = np.linalg.qr(Y)[0]
    U, S, Vt = np.linalg.svd(Q.T @ E, full_matrices=False)
    A, B, sigma, _, _ = amd.offline_factors(_dev(E), r, _dev(omega), power_iters=iters)
    np.testing.assert_allclose(sigma, S[:r], rtol=1e-9)
    assert orc.rel_frobenius(A.cpu().numpy() @ B.cpu().numpy(), (Q @ U[:, :r] * S[:r]) @ Vt[:r]) <= 1e-8


# products of a block per CU: two, three, four and seven chunks of 32 to a block, a last chunk that is partial, two groups of columns, fewer
# rows than a block takes; shares of the reduction that run over the end of a row block (6500 x 5000, 80 columns), and so many row
# blocks that they are not cut at all
@pytest.mark.parametrize("K,N,r,over,iters", [(4100, 129, 8, 8, 1), (1700, 3300, 24, 8, 1), (520, 3000, 40, 30, 1), (31, 8192, 16, 8, 1),
                                              (6500, 5000, 60, 20, 0), (131200, 40, 8, 4, 0)])
def test_residual_factors_cut_across_row_blocks(amd, K, N, r, over, iters):
    test_residual_factors_at_the_edges(amd, K, N, r, over, iters)


# ... with one group of columns: few row blocks, a last chunk that is partial; many row blocks, ten chunks each
@pytest.mark.parametrize("K,N,r,over,iters", [(8300, 4100, 8, 8, 0), (33000, 300, 8, 8, 1)])
def test_residual_factors_of_shares_across_row_blocks(amd, K, N, r, over, iters):
    test_residual_factors_at_the_edges(amd, K, N, r, over, iters)


def test_residual_factors_of_a_matrix_whose_gram_matrix_is_singular(amd):
    # ten singular values near 1, ten near 1e-12, and a test matrix that weighs them alike: Y is well
    # conditioned, Bm Bm^T is not positive definite in fp64
    rng = np.random.default_rng(9)
    U, V = np.linalg.qr(rng.standard_normal((64, 20)))[0], np.linalg.qr(rng.standard_normal((96, 20)))[0]
    S = np.concatenate([np.linspace(1.0, 0.5, 10), np.linspace(2e-12, 1e-12, 10)])
    E, omega = (U * S) @ V.T, V / S
    A, B, sigma, _, _ = amd.offline_factors(_dev(E), 20, _dev(omega), power_iters=0)
    np.testing.assert_allclose(sigma[:10], S[:10], rtol=1e-9)
    assert orc.rel_frobenius(A.cpu().numpy() @ B.cpu().numpy(), E) <= 1e-10


def test_low_rank_matrix_is_recovered(amd):
    # E of exact rank 6 plus nothing: the factors of rank 6 reproduce it (l = rank: no room to spare)
    rng = np.random.default_rng(8)
    E = rng.standard_normal((300, 6)) @ rng.standard_normal((6, 200))
    omega = rng.standard_normal((200, 6))
    A, B, sigma, _, _ = amd.offline_factors(_dev(E), 6, _dev(omega), power_iters=1)
    np.testing.assert_allclose(sigma, np.linalg.svd(E, compute_uv=False)[:6], rtol=1e-10)
    assert orc.rel_frobenius(A.cpu().numpy() @ B.cpu().numpy(), E) <= 1e-12
    # a sketch wider than the matrix's rank cannot be orthonormalised: reported, not computed
    with pytest.raises(amd.MoeLrcError) as ei:
        amd.offline_factors(_dev(E), 6, _dev(rng.standard_normal((200, 14))), power_iters=1)
    assert ei.value.code == -2


def test_layer_compressed_on_the_device_runs_through_the_hot_path(amd):
    cfg = configs.TINY.with_(tokens=40, name="offline_e2e")
    wg, bias = synth.make_gate(cfg)
    experts = []
    for e in range(cfg.n_experts):
        ex = {}
        for mat in (0, 1, 2):
            W = np.asarray(synth.make_expert_weight(cfg, e, mat), dtype=np.float64)
            codes, scale, zero, resid = amd.offline_quantize(_dev(W), cfg.bits, cfg.group)
            omega = np.random.default_rng(100 * e + mat).standard_normal((W.shape[1], cfg.rank + 8))
            A, B, sigma, Ab, Bb = amd.offline_factors(resid, cfg.rank, _dev(omega), power_iters=2)
            ex[mat] = {"codes": codes.cpu().numpy(), "scale": _bits(scale), "zero": _bits(zero), "A": _bits(Ab), "B": _bits(Bb)}
            # the compensated weights are closer to W than the quantized ones, by what Eckart-Young allows
            D = compress.dequantize(ex[mat], cfg.group)
            Sx = np.linalg.svd(W - D, compute_uv=False)
            gain = np.linalg.norm(W - D - A.cpu().numpy() @ B.cpu().numpy()) / np.linalg.norm(W - D)
            assert gain <= np.sqrt((Sx[cfg.rank:] ** 2).sum() / (Sx ** 2).sum()) * 1.05
        experts.append(ex)
    layer = {"wg": wg, "bias": bias, "experts": experts}
    L = amd.Layer.from_config(cfg)
    L.load(layer)
    x_bits = synth.make_tokens(cfg)
    ref = fixtures.oracle_forward(cfg, layer, x_bits)
    out = L.forward(amd.bf16_tensor(x_bits)).float().cpu().numpy().astype(np.float64)
    assert orc.rel_frobenius(out, ref["out"]) <= 5e-3
    L.close()
