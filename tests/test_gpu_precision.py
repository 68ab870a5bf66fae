"""GPU: how far the fp16-piece products are from float64, where a plain fp32 evaluation would be, at
shapes that reach every tile size and remainder.  References are float64 on the GPU."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_2501_12956_amd import binding
    c = binding.Context(0)
    yield c
    c.close()


def _target_error(ctx, m, J, K, kind, seed):
    """Mean |error| of the S-update's targets in units of 2^-24 of their size, over m x J of them.

    The K columns on the right have a diagonal L among themselves, so their residuals E are those of
    plain rounding; the J columns on the left see nothing but the sums over these K.  A column's target
    W_ij + (E_i L_j) / L_jj is placed within +-D of the boundary between codes 7 and 8 (zero): the share
    of targets that fall on the wrong side is E|error| / (2 D)."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    step, size = 0.01, 0.02
    T = ((torch.arange(16, device="cuda") - 7.5) * step).repeat(m, 1).contiguous()
    Ws = torch.randn(m, K, generator=g, device="cuda") * 0.03
    A = torch.randn(K, J, generator=g, device="cuda")
    if kind != "gauss":          # heavy tails; the features that dominate stand anywhere, or nearest to the targets
        A = torch.sign(A) * A.abs() ** 1.5
        big = torch.rand(K, generator=g, device="cuda") < 0.005 if kind == "heavy" else torch.arange(K, device="cuda") < K // 200
        A[big] *= 30.0
    E = Ws - torch.gather(T, 1, (Ws / step + 7.5).round().clamp(0, 15).long())
    S = E.double() @ A.double()
    diag = torch.exp2(torch.round(torch.log2(S.square().mean(0).sqrt() / size))).float()
    D = 2.0 ** -18 * size
    near = D * (2 * torch.rand(m, J, generator=g, device="cuda", dtype=torch.float64) - 1)
    W = torch.cat([(near - S / diag.double()).float(), Ws], 1).contiguous()
    L = torch.zeros(J + K, J + K, device="cuda")
    L[J:, :J] = A
    L.diagonal()[:J] = diag
    L.diagonal()[J:] = 1.0
    Q, Eo = ctx.update_S(W, L, T, 4, want_E=True)
    true = W[:, :J].double() + (Eo[:, J:].double() @ A.double()) / diag.double()
    used = true.abs() < 2 * D               # not so in the few rows where a source column sits on a tie
    assert used.double().mean().item() > 0.98
    wrong = ((Q[:, :J] >= 8) != (true > 0)) & used
    return wrong.double().sum().item() / used.double().sum().item() * 2 * D / size * 2.0 ** 24


@pytest.mark.parametrize("m,J,K,kind", [(5900, 1024, 5000, "gauss"), (5900, 1024, 5000, "heavy"), (5900, 1024, 5000, "near"),
                                        (300, 1024, 1024, "near"), (520, 300, 2901, "gauss"), (1100, 1024, 9000, "near")])
def test_update_S_sums(ctx, m, J, K, kind):
    """An accumulator of the products sums 256 columns (16 roundings, of a sixteenth of the total in the
    mean) and K / 256 of them are added (one rounding of the running total each): about
    0.29 (sqrt(K / 256) + 2) 2^-24 of the target's size, twice that for the spread over targets.  Sums of
    thousands of columns in one fp32 accumulator are at 3 to 8 here."""
    err = _target_error(ctx, m, J, K, kind, seed=K)
    bound = 0.58 * ((K / 256) ** 0.5 + 2)
    print("mean |error| %.2f x 2^-24 of the targets (bound %.2f)" % (err, bound))
    assert err <= bound


def _gram(n, p, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    X = torch.randn(n, p, generator=g, device="cuda").double()
    return (X @ X.t()).float()


def test_cholesky_pivots_are_not_biased(ctx):
    """More than 4096 rows below a panel: the trailing update is a split product.  A product of low pieces
    left out of its diagonal is a sum of squares, 2^-22 / 12 to 2^-22 / 3 of an entry's own square, that no
    pivot gets rid of.  The mean over the rows of (L L^T - H)_jj / H_jj has a standard error of
    2e-7 / sqrt(n) = 2e-9 here; the bias was 1.5e-8."""
    n = 8192
    for seed in (0, 1):
        H = _gram(n, n + n // 16, seed)
        L, info = ctx.cholesky(H)
        assert info == 0
        d = torch.diagonal(H).double()
        bias = ((torch.tril(L).double().square().sum(1) - d) / d).mean().item()
        print("mean of (L L^T - H)_jj / H_jj: %.2e" % bias)
        assert abs(bias) <= 7e-9


@pytest.mark.parametrize("n,p", [(4480, 4400), (4500, 4490), (8192, 8000)])
def test_cholesky_reports_a_singular_matrix_beyond_the_split_update(ctx, n, p):
    """Fewer tokens than features where the first trailing updates are split products: the pivots from p on
    are rounding noise (those right before it hardly more), and one of the first must be reported; AUTO
    then factors the preconditioned matrix."""
    from paper_2501_12956_amd import binding as b
    H = _gram(n, p, n)
    _, info = ctx.cholesky(H, b.PRECOND_NONE, raise_on_fail=False)
    assert p - 8 < info <= p + 8, info
    L, info = ctx.cholesky(H, b.PRECOND_AUTO)
    assert info == 0
    Hd = H.double()
    delta = (Hd.abs().sum(1) - 2 * torch.diagonal(Hd)).clamp(min=1e-8)
    Hp = Hd + torch.diag(delta)
    R = torch.tril(L).double() @ torch.tril(L).double().t() - Hp
    assert R.norm().item() <= 2e-6 * Hp.norm().item()


@pytest.mark.parametrize("where", ["column", "diagonal", "nan"])
def test_cholesky_reports_the_first_bad_pivot_beyond_the_split_update(ctx, where):
    """Not finite below the first panel, or an exact copy of a feature: the pivot of that row is the first
    that fails, as it is in smaller matrices."""
    from paper_2501_12956_amd import binding as b
    n, k = 4500, 4321
    g = torch.Generator(device="cuda").manual_seed(3)
    X = torch.randn(n, 2 * n, generator=g, device="cuda").double()
    if where == "column":
        X[k] = X[17]
    H = (X @ X.t()).float()
    if where == "diagonal":
        H[k, 40] = H[40, k] = float("inf")
    if where == "nan":
        H[k, 4300] = H[4300, k] = float("nan")
    _, info = ctx.cholesky(H, b.PRECOND_NONE, raise_on_fail=False)
    assert info == k + 1


def test_large_tiles_with_remainders_in_every_direction(ctx):
    """G = W H and F = E H take 256 x 256 tiles from 192 of them on; here 15 x 15 with 17 rows and 29
    columns in the last ones and a last step of 29 columns.  Row losses against float64, and the codebooks
    of the prepared T-update on the rows around the last tile's edge."""
    m, n, nbits = 3601, 3613, 3
    g = torch.Generator(device="cuda").manual_seed(4)
    H = _gram(n, 2 * n, 5)
    W = torch.randn(m, n, generator=g, device="cuda") * 0.02
    W[torch.rand(m, n, generator=g, device="cuda") < 0.003] *= 10
    T = ctx.init_codebooks(W, nbits)
    Q = torch.empty(m, n, dtype=torch.uint8, device="cuda")
    for r in range(0, m, 256):
        Q[r:r + 256] = (W[r:r + 256, :, None] - T[r:r + 256, None, :]).abs().argmin(2).to(torch.uint8)
    total, rows = ctx.layer_loss(W, H, T, Q, nbits, want_rows=True)
    E = (W - torch.gather(T, 1, Q.long())).double()
    want = ((E @ H.double()) * E).sum(1)
    rel = ((rows.double() - want) / want).abs()
    print("row losses: rms %.2e, max %.2e" % (rel.square().mean().sqrt().item(), rel.max().item()))
    # about sqrt(3 n / 16) roundings of 2^-24 in a product's chain, summed over a row with random signs
    assert rel.max().item() <= 5e-6 and abs(total - want.sum().item()) <= 1e-6 * want.sum().item()
    T2 = T.clone()
    ctx.update_T_prepare(W, H, nbits)
    ctx.update_T(W, H, Q, T2, nbits)
    ctx.update_T_prepare(None, None, nbits)
    C = 1 << nbits
    for i in list(range(0, 8)) + list(range(3580, 3601)):
        S = torch.nn.functional.one_hot(Q[i].long(), C).double()
        used = S.sum(0) > 0
        A = (S.t() @ (H.double() @ S))[used][:, used]
        t = torch.linalg.solve(A, ((W[i].double() @ H.double()) @ S)[used])
        err = (T2[i].double()[used] - t).abs().max().item() / t.abs().max().item()
        assert err <= 1e-4, (i, err)


def _synthetic_factor(n, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    L = torch.randn(n, n, generator=g, device="cuda").tril_(-1) * (0.3 / n ** 0.5)
    L.diagonal().copy_(0.5 + torch.rand(n, generator=g, device="cuda"))
    return L


@pytest.mark.parametrize("m,n,nbits", [(5900, 2113, 4), (4097, 3203, 3), (133, 10411, 4), (4225, 5003, 2)])
def test_update_S_choices_with_remainders_in_every_direction(ctx, m, n, nbits):
    """One and two k-splits, rows, columns and steps that fill no tile: every choice on rows around the
    tiles' edges is the nearest code of its float64 target, or a near tie."""
    L = _synthetic_factor(n, n)
    W = torch.randn(m, n, generator=torch.Generator(device="cuda").manual_seed(m), device="cuda") * 0.02
    T = ctx.init_codebooks(W, nbits)
    Q = ctx.update_S(W, L, T, nbits)
    rows = sorted({r for e in range(0, m + 1, 128) for r in (e - 1, e) if 0 <= r < m} | {m - 1})
    Wd, Td, Qr = W[rows].double(), T[rows].double(), Q[rows].long()
    chosen = torch.gather(Td, 1, Qr)
    Ld = L.double()
    tgt = Wd + ((Wd - chosen) @ torch.tril(Ld, -1)) / torch.diagonal(Ld)
    gap = (tgt - chosen).abs()
    best = torch.stack([(tgt - Td[:, s:s + 1]).abs() for s in range(1 << nbits)]).amin(0)
    rel = (gap - best) / Td.abs().amax(1, keepdim=True)
    assert rel.max().item() < 1e-6


@pytest.mark.parametrize("n", [300, 2100])
def test_update_S_follows_the_scale_of_a_row(ctx, n):
    """Scaling a row of W and of T by a power of two scales its targets exactly, so its choices stay, up to
    rows whose largest weight and code add up to more than fp32 holds."""
    m, nbits = 6, 4
    g = torch.Generator(device="cuda").manual_seed(n)
    W1 = torch.randn(1, n, generator=g, device="cuda")
    W1 = W1 / W1.abs().max() * 1.9
    L = torch.randn(n, n, generator=g, device="cuda").tril_(-1) * (0.3 / n ** 0.5)
    L.diagonal().fill_(1.0)
    T1 = ctx.init_codebooks(W1, nbits)
    T1 = T1.clamp(-0.95, 0.95)              # the midpoint of two codes forms their sum, which stays in range
    T1[0, 0], T1[0, 15] = -1.0, 1.0
    k = torch.tensor([0.0, -90.0, -20.0, 60.0, 126.0, 127.0], device="cuda", dtype=torch.float64)
    s = torch.exp2(k)[:, None]
    W, T = (W1.double() * s).float().contiguous(), (T1.double() * s).float().contiguous()
    Q = ctx.update_S(W, L, T, nbits)
    assert bool(torch.isfinite(W).all()) and bool(torch.isfinite(T).all())
    for i in range(1, m):
        assert torch.equal(Q[i], Q[0]), i
