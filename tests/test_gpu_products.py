"""The complex FP64 product kernels (both tile sizes and the rule between them) through the inverse and the Newton
iteration, against LAPACK: 1e-12 relative, as the condition numbers here are below 10."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def gw():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1810_07772_amd as gw
    gw.load()
    return gw


def matrix(n):
    rng = np.random.default_rng(n)
    x = rng.standard_normal((n, 2 * n)) + 1j * rng.standard_normal((n, 2 * n))
    return np.eye(n) + x @ x.conj().T / (4 * n)


# One panel of 128 columns and the values beside it; several panels with a ragged last one; a size whose products take
# small tiles throughout (640), one that takes both sizes (2000).  The workspace holds NaN from a call before.
@pytest.mark.parametrize("n", [127, 128, 129, 163, 300, 640, 2000])
def test_inverse(gw, n):
    ctx = gw.Context(0)
    bad = torch.full((n, n), float("nan"), dtype=torch.complex128, device="cuda:0")
    with pytest.raises(gw.GwError):
        gw.hpd_inverse(bad, ctx=ctx)
    a = matrix(n)
    print(f"[case] n={n}", flush=True)
    got = gw.hpd_inverse(torch.from_numpy(a).cuda(), ctx=ctx).cpu().numpy()
    ref = np.linalg.inv(a)
    assert np.linalg.norm(got - ref) < 1e-12 * np.linalg.norm(ref)
    assert np.array_equal(np.triu(got, 1), np.tril(got, -1).conj().T)     # the mirrored triangle


# The factorisation of one 32-wide block: a single entry, part of one 16-column half, a block short of or beyond its
# edge, and blocks after one to three earlier ones of the same panel.  Turning one pivot negative names that one,
# also in the last (padded) block.  A = Lu D Lu^H with Lu unit lower, so the pivots are D.
@pytest.mark.parametrize("n", [1, 2, 16, 17, 31, 33, 50, 80, 111])
def test_diagonal_blocks(gw, n):
    ctx = gw.Context(0)
    a = matrix(n)
    print(f"[case] n={n}", flush=True)
    got = gw.hpd_inverse(torch.from_numpy(a).cuda(), ctx=ctx).cpu().numpy()
    ref = np.linalg.inv(a)
    assert np.linalg.norm(got - ref) < 1e-12 * np.linalg.norm(ref)
    c = np.linalg.cholesky(a)
    lu = c / np.diag(c)
    for bad in sorted({1, n // 2 + 1, n}):
        d = np.diag(c).real ** 2
        d[bad - 1] *= -1
        with pytest.raises(gw.GwError) as e:
            gw.hpd_inverse(torch.from_numpy(lu * d @ lu.conj().T).cuda(), ctx=ctx)
        assert e.value.status == 4 and f"pivot {bad} " in str(e.value)


@pytest.mark.parametrize("n", [33, 65, 500, 900])
def test_newton(gw, n):
    a = matrix(n)
    got, its, _ = gw.newton_inverse(torch.from_numpy(a).cuda())
    ref = np.linalg.inv(a)
    assert np.linalg.norm(got.cpu().numpy() - ref) < 1e-12 * np.linalg.norm(ref)


def test_inverse_rounds_once_per_step(gw):
    """An entry of the factor's diagonal block is rounded once per elimination step and once for the columns applied
    to it.  Against inverses refined in extended precision, three dielectric matrices of 130 rows come to 4.7e-16 so on
    the mean, and to 5.5e-16 with two roundings a step; the bound lies between."""
    err = []
    for seed in range(3):
        n, rng = 130, np.random.default_rng(130000 + seed)
        x = (rng.standard_normal((n, 2 * n)) + 1j * rng.standard_normal((n, 2 * n))) / np.sqrt(2)
        d = 2.0 / (0.3 + np.sort(rng.uniform(0.05, 12.0, n))) ** 0.75
        h = x @ x.conj().T / (2 * n)
        a = np.eye(n) + d[:, None] * (0.5 * (h + h.conj().T)) * d[None, :]
        got = gw.hpd_inverse(torch.from_numpy(a).to("cuda:0")).cpu().numpy()
        ref = np.linalg.inv(a).astype(np.clongdouble)
        ref = ref @ (2 * np.eye(n, dtype=np.clongdouble) - a.astype(np.clongdouble) @ ref)
        err.append(float(np.sqrt(np.sum(np.abs(got - ref) ** 2) / np.sum(np.abs(ref) ** 2))))
    print(f"relative errors {err}")
    assert np.mean(err) < 5.1e-16
