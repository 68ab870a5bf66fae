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
