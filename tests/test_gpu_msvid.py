"""GPU MSVID_l (paper Eq. "msvid-def") through the C ABI against the fp64 oracle (oracle/mdbf_quantizer.py): the sign
mask bit for bit; the envelope by what Theorem 1 fixes (Eq. "rankl-error": the error of the result is the tail of
|Z|'s spectrum, which the oracle's SVD gives in closed form), by exact recovery of members of the format, and,
where |Z|'s spectrum has a gap behind mode l, against the oracle's TSVD_l itself."""
import numpy as np
import pytest

from oracle import mdbf_oracle as orc
from oracle import mdbf_quantizer as qz
from paper_2512_24545_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2512_24545_amd import binding as mb
    mb.lib()
    return torch, mb


def _run(gpu, Z, l, iters=8, seed=1, ld_pad=0):
    torch, mb = gpu
    rows, cols = Z.shape
    b = mb.mdbf_msvid_block(l)
    X0 = synth.normal_block(cols, b, seed)              # the method's random start block: an input
    Zd = torch.zeros((rows, cols + ld_pad), dtype=torch.float32, device="cuda:0")
    Zd[:, :cols] = torch.from_numpy(np.ascontiguousarray(Z, dtype=np.float32))
    S, A, Q, sg = mb.mdbf_msvid(Zd[:, :cols], l, torch.from_numpy(X0).cuda(), iters=iters)
    torch.cuda.synchronize()
    return S.cpu().numpy(), A.cpu().numpy().astype(np.float64), Q.cpu().numpy().astype(np.float64), sg.cpu().numpy()


def _f32(Z):
    return np.asarray(Z, dtype=np.float32).astype(np.float64)


@pytest.mark.parametrize("shape,l", [((512, 384), 1), ((512, 384), 4), ((300, 200), 16), ((130, 77), 8), ((64, 24), 16)])
def test_mask_is_exact_and_error_is_the_spectral_tail(gpu, shape, l):
    """Gaussian Z: |Z| has one dominant singular value and a bulk without gaps, so the iteration cannot (and need
    not) find the oracle's individual singular vectors; what Theorem 1 fixes is the error of the projection,
    sqrt(sum_{i>l} sigma_i^2), and the result must be within 0.5 % of it after 8 passes (measured: 1.0000 for
    l = 1, 1.0002 for l = 4, 1.0013 for l = 16 on 512 x 384) and never below it."""
    Z = _f32(np.random.default_rng(10 + l).standard_normal(shape))
    Z[3, 5] = 0.0
    Z[4, 6] = -0.0                                     # sign(0) = +1, also for a negative zero
    S, A, Q, sg = _run(gpu, Z, l, ld_pad=8)
    np.testing.assert_array_equal(S, qz.sign_pm1(Z))
    sig = np.linalg.svd(np.abs(Z), compute_uv=False)
    opt = np.sqrt((sig[l:] ** 2).sum())
    err = np.linalg.norm(np.abs(Z) - A @ Q.T)
    assert opt * (1 - 1e-6) <= err <= opt * 1.005
    # the same through the mask: || Z - S o (A Q^T) ||_F is that error (the entries of S are +-1)
    assert np.linalg.norm(Z - S * (A @ Q.T)) == pytest.approx(err, rel=1e-12)
    # Ritz values: below the singular values (Cauchy interlacing), descending, and sigma_1 to fp32 accuracy
    assert np.all(sg[:l] <= sig[:l] * (1 + 1e-5)) and np.all(np.diff(sg) <= 1e-6 * sg[0])
    assert sg[0] == pytest.approx(sig[0], rel=1e-5)
    # the factors carry the Ritz values evenly: A^T A = Q^T Q = diag(sigma)
    np.testing.assert_allclose(A.T @ A, np.diag(sg[:l].astype(np.float64)), atol=2e-4 * sg[0])
    np.testing.assert_allclose(Q.T @ Q, np.diag(sg[:l].astype(np.float64)), atol=2e-4 * sg[0])


@pytest.mark.parametrize("rows,cols,l,iters", [(65, 40, 4, 3), (1025, 130, 16, 3), (191, 700, 8, 4), (24, 2049, 16, 5),
                                               (16384, 32, 8, 3), (16385, 33, 16, 3), (70, 16500, 1, 3)])
def test_later_passes_normalise_behind_the_product(gpu, rows, cols, l, iters):
    """From the third pass on the inverse Cholesky factor is worked out beside the product and applied to its sums, for up to
    256 row groups of 64 (16384 and 16385 rows, 16500 columns: the two sides of that line); blocks of both widths.  Against the
    same iteration in fp64: Ritz values and envelope are those of the same subspace, whatever basis is taken on the way."""
    Z = _f32(np.random.default_rng(rows + cols).standard_normal((rows, cols)))
    S, A, Q, sg = _run(gpu, Z, l, iters=iters)
    np.testing.assert_array_equal(S, qz.sign_pm1(Z))
    M, V = np.abs(Z), synth.normal_block(cols, 16 if l <= 8 else 24, 1).astype(np.float64)
    for _ in range(iters):
        V = M.T @ np.linalg.qr(M @ V)[0]
    V = np.linalg.qr(V)[0]
    U, sig, Wt = np.linalg.svd(M @ V, full_matrices=False)
    best = (U[:, :l] * sig[:l]) @ (V @ Wt[:l].T).T
    # fp32 products of 2 iters steps, each 2^-24 of the block per entry, added up at random signs (2e-7 measured at most)
    assert np.abs(sg - sig).max() <= 2e-6 * sig[0]
    assert np.linalg.norm(A @ Q.T - best) <= 5e-6 * np.linalg.norm(best)


@pytest.mark.parametrize("start", ["first", "half", "lengths", "centred"])
@pytest.mark.parametrize("l,iters", [(4, 3), (16, 3), (16, 5), (16, 8)])
def test_start_blocks_that_hide_the_leading_mode(gpu, start, l, iters):
    """|Z| with one mode some hundred times the others, and start blocks whose first column, or half of the columns, are orthogonal to it,
    of lengths from 1e6 to 1e-6, or all centred: as accurate as from any other block, against the same iteration in fp64."""
    torch, mb = gpu
    rng = np.random.default_rng(l + iters)
    rows, cols, b = 400, 300, mb.mdbf_msvid_block(l)
    Z = _f32(np.where(rng.random((rows, cols)) < 0.5, -1, 1) * (1 + 0.01 * rng.standard_normal((rows, cols))))
    M, X0 = np.abs(Z), rng.standard_normal((cols, b))
    lead = np.linalg.svd(M, full_matrices=False)[2][0]
    hidden = X0 - np.outer(lead, lead @ X0)
    if start == "centred":
        X0 -= X0.mean(0)
    else:
        X0[:, :b // 2 if start == "half" else 1] = hidden[:, :b // 2 if start == "half" else 1]
    if start == "lengths":
        X0 *= np.logspace(6, -6, b)
    X0 = X0.astype(np.float32)
    V = X0.astype(np.float64)
    for _ in range(iters):
        V = M.T @ np.linalg.qr(M @ V)[0]
    V = np.linalg.qr(V)[0]
    U, sig, Wt = np.linalg.svd(M @ V, full_matrices=False)
    best = (U[:, :l] * sig[:l]) @ (V @ Wt[:l].T).T
    _, A, Q, _ = [x.cpu().numpy().astype(np.float64) for x in
                  mb.mdbf_msvid(torch.from_numpy(Z.astype(np.float32)).cuda(), l, torch.from_numpy(X0).cuda(), iters=iters)]
    # rounding of fp32 products, 2^-24 of the block per entry and step at random signs: 4e-7 measured at most, and 5e-6 to 1.2e-5 where
    # the columns that share the leading mode are told apart after a product has magnified it
    assert np.linalg.norm(A @ Q.T - best) <= 1.5e-6 * np.linalg.norm(best)


@pytest.mark.parametrize("l", [1, 3, 8, 16])
def test_members_of_the_format_are_fixed_points(gpu, l):
    """Z = S o (A0 Q0^T) with a non-negative envelope of rank l: |Z| has rank l, so MSVID_l returns Z itself
    (Theorem 1 with an empty tail), already after one pass."""
    rng = np.random.default_rng(20 + l)
    A0, Q0 = np.abs(rng.standard_normal((260, l))) + 0.1, np.abs(rng.standard_normal((190, l))) + 0.1
    S0 = qz.sign_pm1(rng.standard_normal((260, 190)))
    Z = _f32(S0 * (A0 @ Q0.T))
    for iters in (1, 4):
        S, A, Q, sg = _run(gpu, Z, l, iters=iters)
        np.testing.assert_array_equal(S, S0)
        assert np.linalg.norm(Z - S * (A @ Q.T)) <= 2e-6 * np.linalg.norm(Z)
    # and the oracle's projection of that Z is Z as well
    assert np.linalg.norm(Z - qz.msvid_value(Z, l)) <= 1e-6 * np.linalg.norm(Z)


@pytest.mark.parametrize("l", [1, 4, 16])
def test_envelope_equals_the_oracles_where_the_spectrum_has_a_gap(gpu, l):
    """Z with a geometrically decaying spectrum (the shape a factor U_0 = U_R Sigma_R^(1/2) of a weight matrix has,
    Eq. "mesvid-balanced"): behind mode l the singular values of |Z| fall by a visible ratio, the iteration
    converges to the dominant subspace and A Q^T equals the oracle's TSVD_l(|Z|) to fp32 accuracy."""
    rng = np.random.default_rng(30)
    Z = _f32((rng.standard_normal((600, 40)) * (0.7 ** np.arange(40))) @ rng.standard_normal((40, 300)))
    So, Ao, Qo = qz.msvid(Z, l)
    S, A, Q, sg = _run(gpu, Z, l, iters=16)
    np.testing.assert_array_equal(S, So)
    E, Eo = A @ Q.T, Ao @ Qo.T
    assert np.linalg.norm(E - Eo) <= 2e-5 * np.linalg.norm(Eo)
    sig = np.linalg.svd(np.abs(Z), compute_uv=False)
    np.testing.assert_allclose(sg[:l], sig[:l], rtol=2e-5)


@pytest.mark.parametrize("rows,cols,pad,l", [(257, 321, 3, 16), (64, 256, 0, 8), (63, 65, 1, 1), (1030, 130, 2, 4), (24, 700, 0, 16)])
def test_edges_of_the_product_kernel(gpu, rows, cols, pad, l):
    """Sizes around its 64-output strips, 64-entry waves and 256-entry chunks, rows at any element's address: the
    Ritz values equal those of the same iteration in fp64 from the same start block (they depend on the span only;
    fp32 products: 1e-5), and a padded leading dimension changes no bit."""
    torch, mb = gpu
    rng = np.random.default_rng(rows + cols)
    Z = _f32(rng.standard_normal((rows, cols)))
    b, iters = mb.mdbf_msvid_block(l), 2
    X0 = synth.normal_block(cols, b, 3)
    V = X0.astype(np.float64)
    for _ in range(iters):
        V = np.abs(Z).astype(np.float64).T @ np.linalg.qr(np.abs(Z) @ V)[0]
    want = np.linalg.svd(np.abs(Z) @ np.linalg.qr(V)[0], compute_uv=False)
    wide = torch.full((rows, cols + pad), float("nan"), device="cuda:0")
    wide[:, :cols] = torch.from_numpy(Z).cuda()
    X0d = torch.from_numpy(X0).cuda()
    got = mb.mdbf_msvid(wide[:, :cols], l, X0d, iters=iters)
    np.testing.assert_array_equal(got[0].cpu().numpy(), np.where(Z < 0, -1, 1))
    np.testing.assert_allclose(got[3].cpu().numpy(), want, rtol=1e-5)
    for x, y in zip(got, mb.mdbf_msvid(wide[:, :cols].contiguous(), l, X0d, iters=iters)):
        assert torch.equal(x, y)


@pytest.mark.parametrize("bad", [float("nan"), float("inf"), -float("inf")])
@pytest.mark.parametrize("l,iters", [(4, 0), (4, 2), (16, 0), (16, 3)])
def test_non_finite_input_gives_the_same_defined_result_every_time(gpu, bad, l, iters):
    """One NaN or infinity in Z spoils the whole Gram matrix: no eigenvalue compares with another, and the Ritz step
    still has to order them.  The mask is right, nothing finite but zeros comes out, and a call whose workspace held
    other bytes, after calls on other matrices, returns the same."""
    torch, mb = gpu
    rows, cols = 130, 77
    good = torch.from_numpy(_f32(np.random.default_rng(l).standard_normal((rows, cols))).astype(np.float32)).cuda()
    start = {k: torch.from_numpy(synth.normal_block(cols, mb.mdbf_msvid_block(k), 3)).cuda() for k in (4, 16)}
    Z = good.clone()
    Z[71, 40] = bad
    got = []
    for fill in (0, 255, 63):
        ws = torch.full((8 << 20,), fill, dtype=torch.uint8, device="cuda:0")
        got.append([x.cpu() for x in mb.mdbf_msvid(Z, l, start[l], iters=iters, workspace=ws)])
        mb.mdbf_msvid(good, 20 - l, start[20 - l], iters=1)
    S, A, Q, sg = got[0]
    np.testing.assert_array_equal(S.numpy(), np.where(Z.cpu().numpy() < 0, -1, 1))
    for E in (A, Q):
        assert not (torch.isinf(E) | (torch.isfinite(E) & (E != 0))).any()
    assert ((sg == 0) | torch.isinf(sg)).all()
    for other in got[1:]:
        for x, y in zip(got[0], other):
            np.testing.assert_array_equal(x.numpy(), y.numpy())         # (NaNs at the same places count as equal)


@pytest.mark.parametrize("iters", [2, 4])
@pytest.mark.parametrize("l", [4, 16])
def test_modes_far_below_the_largest_are_told_apart(gpu, l, iters):
    """Two blocks, one 2^-52 of the other, and a start block whose columns lie in one of them each: the Gram matrix has two blocks as
    well, one 2^-104 of the other, and the Ritz step diagonalises both.  All b Ritz values against the same iteration in fp64."""
    torch, mb = gpu
    rng = np.random.default_rng(l)
    b = mb.mdbf_msvid_block(l)
    rows, cols, r0, c0, b0 = 300, 200, 170, 110, b // 2
    Z, X0 = np.zeros((rows, cols)), np.zeros((cols, b))
    Z[:r0, :c0], Z[r0:, c0:] = rng.standard_normal((r0, c0)), rng.standard_normal((rows - r0, cols - c0)) * 2.0 ** -52
    X0[:c0, :b0], X0[c0:, b0:] = rng.standard_normal((c0, b0)), rng.standard_normal((cols - c0, b - b0))
    Z, X0 = Z.astype(np.float32), X0.astype(np.float32)
    want = []
    for z, V in ((Z[:r0, :c0], X0[:c0, :b0]), (Z[r0:, c0:], X0[c0:, b0:])):
        M, V = np.abs(z.astype(np.float64)), V.astype(np.float64)
        for _ in range(iters):
            V = M.T @ np.linalg.qr(M @ V)[0]
        want.append(np.linalg.svd(M @ np.linalg.qr(V)[0], compute_uv=False))
    sg = mb.mdbf_msvid(torch.from_numpy(Z).cuda(), l, torch.from_numpy(X0).cuda(), iters=iters)[3]
    np.testing.assert_allclose(sg.cpu().numpy().astype(np.float64), np.concatenate(want), rtol=1e-5)     # (fp32 products)


def test_error_falls_with_l_and_with_the_number_of_passes(gpu):
    """Monotone in l (nested feasible sets, Sec. 4.2) and non-increasing in the number of passes."""
    Z = _f32(np.random.default_rng(40).standard_normal((256, 160)))
    errs = []
    for l in (1, 2, 4, 8, 16):
        S, A, Q, _ = _run(gpu, Z, l)
        errs.append(np.linalg.norm(Z - S * (A @ Q.T)))
    assert all(a > b for a, b in zip(errs, errs[1:]))
    by_iters = []
    for iters in (0, 1, 2, 4, 8):
        S, A, Q, _ = _run(gpu, Z, 8, iters=iters)
        by_iters.append(np.linalg.norm(Z - S * (A @ Q.T)))
    assert all(a >= b * (1 - 1e-6) for a, b in zip(by_iters, by_iters[1:]))


def test_repeatable_and_idempotent(gpu):
    Z = _f32(np.random.default_rng(50).standard_normal((200, 150)))
    r1 = _run(gpu, Z, 4)
    r2 = _run(gpu, Z, 4)
    for x, y in zip(r1, r2):
        np.testing.assert_array_equal(x, y)                  # fixed summation orders: the same bits
    S, A, Q, _ = r1
    Y = _f32(S * (A @ Q.T))
    if np.all(A @ Q.T > 0):                                  # then |Y| = A Q^T has rank 4 and Y is a fixed point
        S2, A2, Q2, _ = _run(gpu, Y, 4, iters=2)
        assert np.linalg.norm(Y - S2 * (A2 @ Q2.T)) <= 5e-6 * np.linalg.norm(Y)


def test_projected_factors_run_through_the_forward_kernels(gpu):
    """The quantizer's initialisation on the GPU (Eq. "mesvid-init-compact"): MSVID_l of the balanced factors
    U_0 (N x R), V_0 (M x R) gives S_a, A, Q and S_b, B, G; packed and run through mdbf_forward they must give
    what the forward oracle gives for the same factors, and W_hat must approximate W about as well as the
    oracle's own initialisation does."""
    torch, mb = gpu
    rng = np.random.default_rng(60)
    N, M, R, l = 384, 320, 96, 8
    W = (rng.standard_normal((N, 64)) * (0.9 ** np.arange(64))) @ rng.standard_normal((64, M))
    U0, V0 = qz.balanced_factors(W, R)
    Sa, A, Q, _ = _run(gpu, _f32(U0), l, iters=12)
    Sb, B, G, _ = _run(gpu, _f32(V0), l, iters=12, seed=2)
    h = lambda x: np.asarray(x, dtype=np.float16)
    L = {"m": N, "n": M, "k": R, "l": l, "SA": Sa.astype(np.int8), "SB": np.ascontiguousarray(Sb.T).astype(np.int8),
         "A": h(A), "Q": h(Q), "G": h(G), "B": h(B), "env_dtype": "f16"}
    X = synth.make_activations(M, 1, seed=61, x_dtype="f16")
    ref = orc.forward_factored(L["SA"], L["SB"], L["A"], L["Q"], L["G"], L["B"], X)
    dl = mb.DeviceLayer.from_host(L)
    Y = mb.mdbf_forward(dl, torch.from_numpy(X).cuda(), y_dtype="f32")
    torch.cuda.synchronize()
    assert orc.max_rel_error(Y.cpu().numpy(), ref) <= 2e-3
    What = (Sa * (A @ Q.T)) @ (Sb * (B @ G.T)).T
    Lo = qz.quantize(W, R, l, outer=0)
    What_o = orc.dense_reconstruct(Lo["SA"], Lo["SB"], Lo["A"], Lo["Q"], Lo["G"], Lo["B"])
    e_gpu, e_orc = qz.relative_error(W, What), qz.relative_error(W, What_o)
    assert e_gpu <= e_orc * 1.02 + 1e-6
