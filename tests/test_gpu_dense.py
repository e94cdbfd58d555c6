"""GPU parity of the dense ChFSI steps (Gram products, Lanczos bound,
Cholesky-QR, Rayleigh-Ritz, one full ChFSI iteration) against the FP64
oracle, through the C ABI.

Tolerances: FP64 Gram 1e-13 relative (the products are exact dot products in
a different summation order); FP32 Gram 2e-6 of n (the scale of the diagonal):
FP32 accumulation within row slices of about 4100-5000 rows here,
eps_32 * sqrt(R) ~ 4e-6 random-walk relative error per slice sum, the slice
partials added in FP64 (for the 70000-row case 17 slices, averaging the
slice errors down by ~sqrt(17)).  Eigenvalues from FP64 paths 1e-10 Ha.
"""
import numpy as np
import pytest

from oracle import chfsi as OC
from synth.cluster import random_block

from gpu_system import build, from_rows, relerr, to_rows

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def system():
    s = build()
    s["ctx"] = s["B"].Context(0)
    return s


@pytest.mark.parametrize("n,m,k,same", [(5003, 70, 45, False), (4000, 130, 130, True), (100000, 64, 64, True),
                                        (300, 17, 3, False)])
def test_gram_f64(system, n, m, k, same):
    B = system["B"]
    rng = np.random.default_rng(n + m)
    A = rng.standard_normal((n, m))
    Bm = A if same else rng.standard_normal((n, k))
    At = torch.from_numpy(A).cuda()
    Bt = At if same else torch.from_numpy(Bm).cuda()
    S = torch.zeros((m, Bm.shape[1]), dtype=torch.float64, device="cuda")
    B.gram(system["ctx"], At, Bt, S)
    assert relerr(S.cpu().numpy(), A.T @ Bm) < 1e-13


@pytest.mark.parametrize("n,m", [(70000, 96), (5000, 33)])
def test_gram_f32(system, n, m):
    B = system["B"]
    rng = np.random.default_rng(5)
    A32 = rng.standard_normal((n, m)).astype(np.float32)
    At = torch.from_numpy(A32).cuda()
    S = torch.zeros((m, m), dtype=torch.float64, device="cuda")
    B.gram(system["ctx"], At, At, S)
    ref = A32.astype(np.float64).T @ A32.astype(np.float64)
    assert float(np.abs(S.cpu().numpy() - ref).max() / n) < 2e-6
    assert np.array_equal(S.cpu().numpy(), S.cpu().numpy().T)


@pytest.mark.parametrize("dtype,tol", [(torch.float64, 1e-15), (torch.float32, 1e-7)])
@pytest.mark.parametrize("m,k", [(1, 0), (16, 0), (17, 0), (32, 0), (33, 0), (64, 0), (65, 0), (128, 0), (129, 0), (257, 0),
                                 (1, 1), (3, 64), (65, 16), (130, 5), (5, 130), (64, 33)])
@pytest.mark.parametrize("n", [1, 31, 257, 9001])
def test_gram_tile_edges(system, dtype, tol, m, k, n):
    # widths at the edges of the 16, 32, 64 and 128 column pieces, row counts
    # around the unrolled steps and slices; the blocks are columns of wider ones,
    # off any alignment and with NaN beside them.  A sum of n products of N(0, 1)
    # pairs in one order is off by eps sqrt(n) per term of a random walk: below
    # 8 eps max(n, 8) by far.
    B = system["B"]
    rng = np.random.default_rng(m + 7 * k + n)

    def block(w, pad, off):
        X = torch.full((n, w + pad), float("nan"), dtype=dtype, device="cuda")
        X[:, off:off + w] = torch.from_numpy(rng.standard_normal((n, w))).to(device="cuda", dtype=dtype)
        return X[:, off:off + w]

    for pad, off in ((0, 0), (3, 1), (4, 4), (8, 0)):
        At = block(m, pad, off)
        Bt = block(k, 5, 2) if k else At
        S = torch.full((m, Bt.shape[1] + 1), -7.0, dtype=torch.float64, device="cuda")
        B.gram(system["ctx"], At, Bt, S[:, :-1])
        ref = At.double().cpu().numpy().T @ Bt.double().cpu().numpy()
        got = S.cpu().numpy()
        assert np.abs(got[:, :-1] - ref).max() < 8 * tol * max(n, 8), (pad, off)
        assert (got[:, -1] == -7.0).all()
        if not k:
            assert np.array_equal(got[:, :-1], got[:, :-1].T)


def test_gram_f32_wide_block_norms_unbiased(system):
    """FP32 Gram of a wide block over many rows (1,048,576 x 8192, unit
    columns): the diagonal, the columns' squared norms, is what FP32
    Cholesky-QR leaves in the length of every column and so in the charge of
    the SCF density.  The FP32 MFMA sums of the BLAS kernels come out low by
    an amount that grows with the rows one sum runs over (measured on the
    MI355X: -8.6e-6 relative over ~284k-row slices, -3.6e-7 over 8192-row
    slices); the slices are kept short whatever the width, so the mean
    error of the diagonal stays below 1e-6 (a long-slice Gram fails)."""
    B = system["B"]
    n, m = 1 << 20, 8192
    print(f"case: FP32 Gram {n} x {m}", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(11)
    X = torch.randn((n, m), generator=gen, dtype=torch.float32, device="cuda")
    true = torch.empty(m, dtype=torch.float64, device="cuda")
    for c in range(0, m, 512):
        true[c:c + 512] = (X[:, c:c + 512].double() ** 2).sum(0)
    X /= true.sqrt().float()[None, :]
    for c in range(0, m, 512):
        true[c:c + 512] = (X[:, c:c + 512].double() ** 2).sum(0)
    S = torch.empty((m, m), dtype=torch.float64, device="cuda")
    B.gram(system["ctx"], X, X, S)
    d = (torch.diagonal(S) - true).cpu().numpy()
    del X, S
    torch.cuda.empty_cache()
    print(f"diagonal error: mean {d.mean():.3e}, max |.| {np.abs(d).max():.3e}")
    assert abs(d.mean()) < 1e-6 and np.abs(d).max() < 3e-6


def test_lanczos_bound(system):
    s = system
    v0 = random_block(s["g"].n, 1, 3001)[:, 0]
    ref = OC.lanczos_bound(s["Ho"].apply, v0, 10)
    got = s["Hg"].lanczos_bound(s["ctx"], to_rows(s, v0, torch.float64), 10)
    assert np.allclose(got, ref, rtol=1e-10, atol=1e-10)


@pytest.mark.parametrize("k", [2, 7, 32])
@pytest.mark.parametrize("ordering", ["hilbert", "lexicographic"])
@pytest.mark.parametrize("radius,scale", [(2.0, 1.0), (9.0, 1e-150), (9.0, 1e150)])
def test_lanczos_bound_small_grids(k, ordering, radius, scale):
    # both loops (all steps on the device; the general one for the
    # lexicographic layout), from a grid with fewer 512-row runs than
    # workgroups, at the ends of k and of the start vector's norm.  Without
    # reorthogonalisation rounding is amplified as Ritz values converge, so
    # beyond a few steps the extreme values are compared to 1e-8.
    from oracle import grid as G
    from oracle import hamiltonian as OH
    from paper_2303_00790_amd import binding as B
    pos, spc = np.array([[0.1, -0.2, 0.3], [1.5, 0.4, -0.8]]), np.zeros(2, np.int32)
    pp = OH.PseudoParams(h_s=2.0, h_p=0.5)
    lex = ordering == "lexicographic"
    g = G.build_grid(radius, 0.7, G.ORDER_LEX if lex else G.ORDER_HILBERT)
    Ho = OH.build_hamiltonian(g, pos, spc, pp)
    H = B.Hamiltonian(pos, spc, pp, 0.7, radius, B.ORDER_LEX if lex else B.ORDER_HILBERT)
    ctx = B.Context(0)
    v0 = random_block(g.n, 1, 3002)[:, 0]
    vec = torch.zeros(H.n_rows, dtype=torch.float64, device="cuda")
    vec[slice(0, g.n) if lex else torch.from_numpy(g.row_of_rank).cuda()] = torch.from_numpy(v0 * scale).cuda()
    b, tmin, tmax = H.lanczos_bound(ctx, vec, k)
    rb, rmin, rmax = OC.lanczos_bound(Ho.apply, v0, k)
    tol = 1e-10 if k < 10 else 1e-8
    assert abs(tmin - rmin) < tol * rmax and abs(tmax - rmax) < tol * rmax
    if k < 10:
        assert abs(b - rb) < tol * rb
    with pytest.raises(B.ChfError):
        H.lanczos_bound(ctx, torch.zeros_like(vec), k)


def test_orthonormalize_f64(system):
    s = system
    X = random_block(s["g"].n, 96, 2400)
    Q, R = OC.cholesky_qr(X)
    Xg = to_rows(s, X, torch.float64)
    fb = s["B"].orthonormalize(s["ctx"], Xg)
    assert fb == 0
    assert relerr(from_rows(s, Xg, 96), Q) < 1e-11
    G = (Xg.T @ Xg).cpu().numpy()
    assert np.abs(G - np.eye(96)).max() < 1e-12
    pad = torch.ones(s["Hg"].n_rows, dtype=torch.bool, device="cuda")
    pad[s["rows"]] = False
    assert float(Xg[pad].abs().max()) == 0.0


def test_orthonormalize_f32(system):
    s = system
    X = random_block(s["g"].n, 64, 2401)
    Xg = to_rows(s, X, torch.float32)
    s["B"].orthonormalize(s["ctx"], Xg)
    G = (Xg.double().T @ Xg.double()).cpu().numpy()
    assert np.abs(G - np.eye(64)).max() < 5e-5


@pytest.fixture(scope="module")
def filtered_block(system):
    # a block as the SCF filters it: Ritz vectors after two oracle ChFSI
    # iterations, filtered with degree 12 between their own bounds; the
    # columns stay nearly orthogonal but their norms spread by |T_12(t0)|, a
    # condition number of ~1.4e2 (one FP32 Cholesky-QR pass would leave
    # kappa^2 u_32 ~ 1e-3 of orthogonality error)
    s = system
    v0 = random_block(s["g"].n, 1, 3001)[:, 0]
    b, tmin, _ = OC.lanczos_bound(s["Ho"].apply, v0)
    a0, a = tmin, tmin + 0.1 * (b - tmin)
    X = random_block(s["g"].n, 64, 2410)
    for _ in range(2):
        lam, X = OC.chfsi_iteration(s["Ho"].apply, X, 10, a, b, a0)
        a, a0 = lam[-1], lam[0]
    Y = OC.chebyshev_filter(s["Ho"].apply, X, 12, a, b, a0)
    return Y / np.abs(Y).max()


@pytest.mark.parametrize("gram_dtype", ["f32", "f64"])
def test_orthonormalize_f32_filtered_block_matches_oracle(system, filtered_block, gram_dtype):
    # FP32 Cholesky-QR (two passes) of a freshly filtered block against the
    # oracle's one exact pass on the same FP32-rounded block: Q of a full-rank
    # block is unique (positive diagonal of R), and the two-pass product of
    # triangular factors is again such an R.  Q moves by about kappa(X) times
    # the FP32 rounding of the block and of the updates (kappa here ~1.4e2),
    # so 2e-4 of max |Q|; orthonormality to 1e-6; the Ritz values of the FP32
    # Rayleigh-Ritz on the result against the oracle's within 2e-5 of the
    # spectrum's scale (the FP32 H X and Gram products).
    s = system
    B = s["B"]
    X32 = filtered_block.astype(np.float32).astype(np.float64)
    Q, _ = OC.cholesky_qr(X32)
    assert np.linalg.cond(X32) > 100
    Xg = to_rows(s, X32, torch.float32)
    fb = B.orthonormalize(s["ctx"], Xg, gram_dtype=B.CHF_F32 if gram_dtype == "f32" else B.CHF_F64)
    assert fb == 0
    got = from_rows(s, Xg, 64)
    assert relerr(got, Q) < 2e-4
    G = (Xg.double().T @ Xg.double()).cpu().numpy()
    assert np.abs(G - np.eye(64)).max() < 1e-6
    lam, _ = OC.rayleigh_ritz(s["Ho"].apply, Q)
    W = torch.zeros_like(Xg)
    eig = B.rayleigh_ritz(s["Hg"], s["ctx"], Xg, W)
    assert np.abs(eig - lam).max() < 2e-5 * max(1.0, np.abs(lam).max())


def test_orthonormalize_f32_retries_with_fp64_gram(system):
    # a column dependent on the others to ~3e-4 (pivot ratio ~1e-7, below what
    # an FP32 Gram resolves): the first pass is redone with an FP64 Gram
    # (one retry) and the result is orthonormal and spans the same columns
    s = system
    B = s["B"]
    X = random_block(s["g"].n, 32, 2411)
    X = X / np.abs(X).max()
    X[:, 7] = X[:, 3] + 3e-4 * X[:, 7]
    X32 = X.astype(np.float32).astype(np.float64)
    Xg = to_rows(s, X32, torch.float32)
    fb = B.orthonormalize(s["ctx"], Xg)
    assert fb == 1
    got = from_rows(s, Xg, 32)
    assert np.abs(got.T @ got - np.eye(32)).max() < 1e-6
    # span: X32 = got (got^T X32)
    assert relerr(got @ (got.T @ X32), X32) < 1e-5


def test_orthonormalize_rejects_fp64_block_with_fp32_gram(system):
    s = system
    B = s["B"]
    Xg = to_rows(s, random_block(s["g"].n, 8, 2412), torch.float64)
    with pytest.raises(B.ChfError) as e:
        B.orthonormalize(s["ctx"], Xg, gram_dtype=B.CHF_F32)
    assert e.value.code == -1


@pytest.mark.parametrize("dtype,tol", [(torch.float64, 1e-12), (torch.float32, 1e-5)])
def test_rayleigh_ritz_narrow_work_matches_full_width(system, dtype, tol):
    # W = H X in column blocks and X <- X Q in row panels through a work block
    # of 32 columns for 64 vectors: the same result as a full-width work block
    # up to the summation order of the products
    s = system
    X, _ = OC.cholesky_qr(random_block(s["g"].n, 64, 2413))
    Xa = to_rows(s, X, dtype)
    Xb = Xa.clone()
    ea = s["B"].rayleigh_ritz(s["Hg"], s["ctx"], Xa, torch.zeros_like(Xa))
    eb = s["B"].rayleigh_ritz(s["Hg"], s["ctx"], Xb, torch.zeros((s["Hg"].n_rows, 32), dtype=dtype, device="cuda"))
    assert np.abs(ea - eb).max() < tol * np.abs(ea).max()
    gaps = np.minimum(np.diff(ea, prepend=-np.inf), np.diff(ea, append=np.inf))
    ok = torch.from_numpy(gaps > 1e-6).cuda()
    da = Xa[:, ok].double()
    db = Xb[:, ok].double()
    sign = torch.sign((da * db).sum(0))
    assert float((da - db * sign).abs().max() / da.abs().max()) < (1e-10 if dtype == torch.float64 else 1e-3)


def test_rayleigh_ritz_rejects_more_vectors_than_grid_points():
    # a block wider than the grid cannot be orthonormal; the call refuses it
    # before any device work (it would also not fit the rotation's row panels
    # in a one-column work block)
    from paper_2303_00790_amd import binding as B
    from synth.workloads import MODEL_PP
    H = B.Hamiltonian(np.zeros((1, 3)), np.array([1], np.int32), MODEL_PP, 0.7, 2.5, B.ORDER_HILBERT)
    assert H.n_points < H.n_rows
    ctx = B.Context(0)
    X = torch.zeros((H.n_rows, H.n_points + 1), dtype=torch.float64, device="cuda")
    W = torch.zeros((H.n_rows, 1), dtype=torch.float64, device="cuda")
    with pytest.raises(B.ChfError) as e:
        B.rayleigh_ritz(H, ctx, X, W)
    assert e.value.code == -1 and "grid points" in str(e.value)


def test_orthonormalize_rank_deficient_falls_back(system):
    s = system
    X = random_block(s["g"].n, 32, 2402)
    X[:, 5] = X[:, 4]                     # exactly dependent columns
    Xg = to_rows(s, X, torch.float64)
    try:
        fb = s["B"].orthonormalize(s["ctx"], Xg)
        assert fb == 1
    except s["B"].ChfError as e:
        assert e.code == -4


@pytest.mark.parametrize("dtype,tol", [(torch.float64, 1e-10), (torch.float32, 2e-5)])
def test_rayleigh_ritz(system, dtype, tol):
    s = system
    X, _ = OC.cholesky_qr(random_block(s["g"].n, 64, 2403))
    lam, Xr = OC.rayleigh_ritz(s["Ho"].apply, X)
    Xg = to_rows(s, X, dtype)
    W = torch.zeros_like(Xg)
    eig = s["B"].rayleigh_ritz(s["Hg"], s["ctx"], Xg, W)
    assert np.abs(eig - lam).max() < tol * max(1.0, np.abs(lam).max())
    if dtype == torch.float64:
        got = from_rows(s, Xg, 64)
        sign = np.sign((got * Xr).sum(0))
        gaps = np.minimum(np.diff(lam, prepend=-np.inf), np.diff(lam, append=np.inf))
        ok = gaps > 1e-6
        assert relerr((got * sign)[:, ok], Xr[:, ok]) < 1e-8


def test_chfsi_iteration_f64(system):
    s = system
    X = random_block(s["g"].n, 64, 2404)
    v0 = random_block(s["g"].n, 1, 3001)[:, 0]
    b, tmin, _ = OC.lanczos_bound(s["Ho"].apply, v0)
    a0, a = tmin, tmin + 0.1 * (b - tmin)
    Xo = X
    Xg = to_rows(s, X, torch.float64)
    W = torch.zeros_like(Xg)
    for _ in range(3):
        lam, Xo = OC.chfsi_iteration(s["Ho"].apply, Xo, 10, a, b, a0)
        s["Hg"].filter(Xg, W, 10, a, b, a0)
        s["B"].orthonormalize(s["ctx"], Xg)
        eig = s["B"].rayleigh_ritz(s["Hg"], s["ctx"], Xg, W)
        assert np.abs(eig - lam).max() < 1e-9
        a, a0 = lam[-1], lam[0]


def test_reserved_workspace_makes_later_calls_allocation_free(system):
    """After chf_reserve for an operation, calling it at that size allocates
    no device memory in the library (the counter of its allocations stays)."""
    s = system
    B = s["B"]
    H = s["Hg"]
    ctx = B.Context(0)
    X = to_rows(s, random_block(s["g"].n, 48, 2403), torch.float64)
    W = torch.zeros_like(X)
    v0 = to_rows(s, random_block(s["g"].n, 1, 3003)[:, 0], torch.float64)
    # the query is consistent and non-trivial
    hb, cb = B.workspace_bytes(H, B.WS_ORTHONORMALIZE, B.CHF_F64, 48)
    assert hb == 0 and cb >= 48 * 48 * 12
    hb, cb = B.workspace_bytes(H, B.WS_FILTER, B.CHF_F64, 48)
    assert hb >= 4 * H.n_proj * 48 * 8 and cb == 0
    with pytest.raises(B.ChfError):
        B.workspace_bytes(H, 7, B.CHF_F64, 48)
    for op, ldw in ((B.WS_FILTER, 0), (B.WS_ORTHONORMALIZE, 0), (B.WS_RAYLEIGH_RITZ, 48), (B.WS_LANCZOS, 0)):
        B.reserve(H, ctx, op, B.CHF_F64, 48, ldw)
    before = B.device_allocations()
    b, tmin, _ = H.lanczos_bound(ctx, v0, 10)
    H.apply(X, W)
    H.filter(X, W, 4, tmin + 0.1 * (b - tmin), b, tmin - 1.0)
    B.orthonormalize(ctx, X)
    B.rayleigh_ritz(H, ctx, X, W)
    torch.cuda.synchronize()
    assert B.device_allocations() == before


def test_absurd_reservation_reports_out_of_memory(system):
    """A workspace far beyond the device (2^30 FP64 vectors of KB
    coefficients) fails with CHF_ENOMEM and leaves the handle usable."""
    s = system
    B = s["B"]
    with pytest.raises(B.ChfError) as e:
        B.reserve(s["Hg"], None, B.WS_FILTER, B.CHF_F64, 1 << 30)
    assert e.value.code == -2
    X = to_rows(s, random_block(s["g"].n, 8, 2404), torch.float64)
    Y = torch.zeros_like(X)
    s["Hg"].apply(X, Y)
    torch.cuda.synchronize()
    assert bool(torch.isfinite(Y).all())


@pytest.mark.parametrize("dtype,tol", [(torch.float64, 1e-13), (torch.float32, 2e-6)])
@pytest.mark.parametrize("n,m", [(40, 1), (131, 16), (500, 17), (1000, 127), (1000, 128), (1000, 129), (3001, 257), (5000, 400)])
def test_orthonormalize_panel_edges(system, dtype, tol, n, m):
    # widths around the 16 columns of a product and the 128 of a panel, rows not
    # a multiple of a wave's 32, a leading dimension off any alignment with NaN
    # in the columns beside the block, which stay.  A well-conditioned block: Q
    # R = X and Q^T Q = 1 to the rounding of sums of up to m terms of the last
    # pass, eps (sqrt(m) + 2) and a factor of 4 for the condition number (~3).
    B = system["B"]
    rng = np.random.default_rng(n + m)
    X = rng.standard_normal((n, m)) * np.exp(rng.uniform(-3, 3, m))
    Xg = torch.full((n, m + 3), float("nan"), dtype=dtype, device="cuda")
    Xg[:, 1:1 + m] = torch.from_numpy(X).to(device="cuda", dtype=dtype)
    X = Xg[:, 1:1 + m].double().cpu().numpy()
    B.orthonormalize(system["ctx"], Xg[:, 1:1 + m])
    Q = Xg[:, 1:1 + m].double().cpu().numpy()
    ref, R = np.linalg.qr(X)
    ref *= np.sign(np.diag(R))
    assert np.abs(Q.T @ Q - np.eye(m)).max() < tol * (np.sqrt(m) + 2)
    assert np.abs(Q - ref).max() < 4 * tol * (np.sqrt(m) + 2) * np.abs(ref).max()
    assert bool(torch.isnan(Xg[:, 0]).all()) and bool(torch.isnan(Xg[:, 1 + m:]).all())


@pytest.mark.parametrize("m", [1, 2, 3, 4, 16, 63, 64, 65, 127, 128, 129, 191, 192, 193])
@pytest.mark.parametrize("kind", ["random", "invariant"])
def test_rayleigh_ritz_eigensolver_edges(system, m, kind):
    # the own reduction to tridiagonal form (M <= 192) at the edges of its
    # variants and the library's beyond.  "invariant":
    # unit vectors far apart, whose projected matrix is (nearly) diagonal with
    # many close entries, so that reflectors vanish.  Eigenvalues to
    # 1e-13 of the matrix norm times m (backward error of the reduction and
    # of divide and conquer, ~m eps), columns orthonormal to the same.
    s = system
    n = s["g"].n
    if kind == "random":
        X = np.linalg.qr(np.random.default_rng(m).standard_normal((n, m)))[0]
    else:
        X = np.zeros((n, m))
        X[np.linspace(0, n - 1, m).astype(int), np.arange(m)] = 1.0
    P = X.T @ s["Ho"].apply(X)
    P = 0.5 * (P + P.T)
    ref = np.linalg.eigvalsh(P)
    Xg = to_rows(s, X, torch.float64)
    W = torch.zeros_like(Xg)
    eig = s["B"].rayleigh_ritz(s["Hg"], s["ctx"], Xg, W)
    Q = from_rows(s, Xg, m)
    tol = 1e-13 * max(m, 10)
    assert np.abs(np.asarray(eig) - ref).max() < tol * np.abs(ref).max()
    assert np.abs(Q.T @ Q - np.eye(m)).max() < tol
    assert np.abs(Q.T @ s["Ho"].apply(Q) - np.diag(np.asarray(eig))).max() < tol * max(np.abs(P).max(), np.abs(ref).max())


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("col", [0, 15, 16, 127, 128, 200])
def test_orthonormalize_reports_the_failing_column(system, dtype, col):
    # a zero column has no direction: every pass's factorisation stops at it,
    # in whichever 16 x 16 or 128-column block it lies
    B = system["B"]
    X = np.random.default_rng(col).standard_normal((2000, 201))
    X[:, col] = 0.0
    Xg = torch.from_numpy(X).to(device="cuda", dtype=dtype)
    with pytest.raises(B.ChfError, match=rf"minor {col + 1}\b"):
        B.orthonormalize(system["ctx"], Xg)


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("m", [1, 16, 129])
def test_orthonormalize_stops_at_an_infinite_pivot(system, dtype, m):
    """an infinite value makes its column's norm infinite, and with the shift of
    the last attempt every pivot: the first one is named, also of a single column
    (behind whose square there is no second one)"""
    B = system["B"]
    X = torch.from_numpy(np.random.default_rng(m).standard_normal((400, m))).to("cuda", dtype)
    X[7, m - 1] = float("inf")
    with pytest.raises(B.ChfError, match=r"CHF_ENOTPD: .*minor 1\)"):
        B.orthonormalize(system["ctx"], X)


@pytest.mark.parametrize("dtype,tol", [(torch.float64, 1e-13), (torch.float32, 2e-6)])
@pytest.mark.parametrize("m", [1, 15, 17, 31, 97, 128, 129])
def test_rayleigh_ritz_rotation_in_place(system, dtype, tol, m):
    # the rotation of up to 128 columns in place, and the panels beyond, on
    # columns off any alignment with NaN beside them, which stay: X Q from the
    # Q that takes X to the result, sums of m products of unit columns
    s, B = system, system["B"]
    X, _ = np.linalg.qr(np.random.default_rng(m).standard_normal((s["g"].n, m)))
    Xg = torch.full((s["Hg"].n_rows, m + 3), float("nan"), dtype=dtype, device="cuda")
    Xg[:, 1:1 + m] = to_rows(s, X, dtype)
    X = from_rows(s, Xg[:, 1:1 + m].contiguous(), m)
    W = torch.zeros((s["Hg"].n_rows, m), dtype=dtype, device="cuda")
    B.rayleigh_ritz(s["Hg"], s["ctx"], Xg[:, 1:1 + m], W)
    got = from_rows(s, Xg[:, 1:1 + m].contiguous(), m)
    Q = np.linalg.lstsq(X, got, rcond=None)[0]
    assert np.abs(X @ Q - got).max() < 8 * tol * (np.sqrt(m) + 2) * np.abs(got).max()
    assert np.abs(Q.T @ Q - np.eye(m)).max() < 8 * tol * (np.sqrt(m) + 2)
    assert bool(torch.isnan(Xg[:, 0]).all()) and bool(torch.isnan(Xg[:, 1 + m:]).all())
    assert not bool(torch.isnan(Xg[:, 1:1 + m]).any())


@pytest.mark.parametrize("m", [97, 260, 400])
def test_orthonormalize_f64_rounds_like_a_blocked_solve(system, m):
    # Whole numbers: the Gram matrix is exact, and the columns are nearly orthogonal,
    # so what is left is the rounding of the factorisation and of the solve.  Against
    # 80 bits, without each column's common factor (the rounding of its pivot).  The
    # sums over blocks of 128 columns round a few times at the size of the column:
    # 1.1 eps in an emulation of their order, half of that again for R; twice their
    # sum is allowed.  One chain over all columns rounds at every one of them: 4.8
    # eps in the second panel and growing.
    n = 4096
    X = np.random.default_rng(m).integers(-8, 9, (n, m)).astype(np.float64)
    Xl = X.astype(np.longdouble)
    S = Xl.T @ Xl
    R = np.zeros_like(S)
    for k in range(m):
        R[k, k:] = S[k, k:] / np.sqrt(S[k, k])
        S[k + 1:, k + 1:] -= np.outer(R[k, k + 1:], R[k, k + 1:])
    Q = np.zeros_like(Xl)
    for j in range(m):
        Q[:, j] = (Xl[:, j] - Q[:, :j] @ R[:j, j]) / R[j, j]
    Xg = torch.from_numpy(X).cuda()
    system["B"].orthonormalize(system["ctx"], Xg)
    err = (Xg.cpu().numpy() - Q).astype(np.float64)
    Q = Q.astype(np.float64)
    err -= Q * ((err * Q).sum(0) / (Q * Q).sum(0))
    for c in range(0, m, 128):
        rms = np.sqrt((err[:, c:c + 128] ** 2).mean() / (Q * Q).mean()) / 2.0 ** -53
        print(f"columns from {c}: {rms:.2f} eps")
        assert rms < 3.2, c


@pytest.mark.parametrize("same", [True, False])
def test_gram_of_very_wide_blocks(system, same):
    # more pieces of 32 columns than a launch has workgroups: every entry of S is
    # written.  Sums of 3 products of N(0, 1) pairs in FP32.
    B = system["B"]
    m = 23200
    gen = torch.Generator(device="cuda")
    gen.manual_seed(12)
    At = torch.randn((3, m), generator=gen, dtype=torch.float32, device="cuda")
    Bt = At if same else torch.randn((3, m), generator=gen, dtype=torch.float32, device="cuda")
    S = torch.full((m, m), float("nan"), dtype=torch.float64, device="cuda")
    B.gram(system["ctx"], At, Bt, S)
    err = [float((S[r:r + 2320] - At[:, r:r + 2320].double().T @ Bt.double()).abs().max()) for r in range(0, m, 2320)]
    del S
    torch.cuda.empty_cache()
    assert all(e < 8e-7 * 8 for e in err), err


@pytest.mark.parametrize("dtype,tol", [(torch.float64, 1e-12), (torch.float32, 1e-5)])
def test_orthonormalize_of_the_longest_blocks(system, dtype, tol):
    # one column of the most rows the call takes, where a launch over all of them
    # would have 2^32 threads: it is scaled to length one
    B = system["B"]
    n = (1 << 31) - 1
    X = torch.full((n, 1), 3.0, dtype=dtype, device="cuda")
    assert B.orthonormalize(system["ctx"], X) == 0
    lo, hi = float(X.min()), float(X.max())
    del X
    torch.cuda.empty_cache()
    assert abs(lo * n ** 0.5 - 1) < tol and abs(hi * n ** 0.5 - 1) < tol


def test_reserved_workspace_covers_smaller_calls(system):
    # the scratch of an operation is not largest at its largest size: at 128 columns
    # a Gram matrix is one piece in 1.1 times the bytes of 129, and up to 192 columns
    # the eigensolver is the library's own
    from oracle import hamiltonian as OH
    B = system["B"]
    helper, ctx = B.Context(0), B.Context(0)
    B.reserve(system["Hg"], ctx, B.WS_RAYLEIGH_RITZ, B.CHF_F64, 193, 193)
    for m, ldw in ((193, 193), (192, 192), (130, 3), (129, 128), (128, 100), (65, 65), (17, 16)):
        X = to_rows(system, random_block(system["g"].n, m, 2420 + m), torch.float64)
        W = torch.empty((X.shape[0], ldw), dtype=torch.float64, device="cuda")
        B.orthonormalize(helper, X)
        before = B.device_allocations()
        B.rayleigh_ritz(system["Hg"], ctx, X, W)
        assert B.device_allocations() == before, (m, ldw)
    H = B.Hamiltonian(np.zeros((1, 3)), np.zeros(1, np.int32), OH.PseudoParams(h_s=2.0, h_p=0.5), 0.7, 27.0,
                      B.ORDER_HILBERT)
    ctx = B.Context(0)
    B.reserve(H, ctx, B.WS_ORTHONORMALIZE, B.CHF_F64, 129)
    before = B.device_allocations()
    for m in (129, 128, 64, 32, 16, 1):
        X = torch.randn((H.n_rows, m), dtype=torch.float64, device="cuda")
        B.orthonormalize(ctx, X)
        assert B.device_allocations() == before, m


@pytest.mark.parametrize("gram_dtype", ["f32", "f64"])
def test_reserved_workspace_covers_the_fp64_gram_of_an_fp32_block(system, gram_dtype):
    # its partials are twice as large; with an FP32 Gram a dependent column (see the
    # retry's test) makes the call redo the product in FP64
    B = system["B"]
    X = random_block(system["g"].n, 32, 2411)
    X = X / np.abs(X).max()
    X[:, 7] = X[:, 3] + 3e-4 * X[:, 7]
    Xg = to_rows(system, X, torch.float32)
    ctx = B.Context(0)
    B.reserve(system["Hg"], ctx, B.WS_ORTHONORMALIZE, B.CHF_F32, 32)
    before = B.device_allocations()
    fb = B.orthonormalize(ctx, Xg, gram_dtype=B.CHF_F32 if gram_dtype == "f32" else B.CHF_F64)
    assert fb == (1 if gram_dtype == "f32" else 0)
    assert B.device_allocations() == before


def test_rayleigh_ritz_rejects_overlapping_work(system):
    # H X would overwrite columns of X that the projection and the rotation still read
    s, B = system, system["B"]
    buf = to_rows(s, random_block(s["g"].n, 24, 2430), torch.float64)
    kept = buf.clone()
    for X, W in ((buf[:, :16], buf[:, 8:]), (buf[:, :16], buf[:, :16]), (buf[:, 4:8], buf[:, :1])):
        with pytest.raises(B.ChfError) as e:
            B.rayleigh_ritz(s["Hg"], s["ctx"], X, W)
        assert e.value.code == -1 and "overlap" in str(e.value)
    assert torch.equal(buf, kept)
