"""GPU parity of the plasmon-pole model against the FP64 oracle: mode strengths, vectors and sum-rule
frequencies from the block iteration (small, full-space and 410-vector cases), the homogeneous-gas
closed form, the pole-form eps^-1(w) with its mode convergence (the synthetic analogue of the
paper's 410 x 410 silicon figure), and the iteration limit."""
import numpy as np
import pytest

import gwsynth as gs
import oracle as orc
from oracle import pp_oracle as pp

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def gw():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1810_07772_amd as gw
    gw.load()
    return gw


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).to("cuda:0")


def gpu_eps_inv(gw, s):
    """eps^-1 by the library, for a system whose orbitals are already complex64-exact."""
    pv, pc = dev(s.psi_v.astype(np.complex64)), dev(s.psi_c.astype(np.complex64))
    pgg = gw.polarizability(pv, pc, s.e_v, s.e_c, s.n, s.a_bohr, s.q, s.miller)
    return gw.eps_inverse(pgg, s.n, s.a_bohr, s.q, s.miller), pv


def compare(gw, s, ei, pv, n_modes, occ=1.0, tol=1e-10):
    sig, om, a, its, res = gw.plasmon_pole(ei, s.n, s.a_bohr, s.q, s.miller, pv, occ, n_modes, tol=tol)
    torch.cuda.synchronize()
    sv = orc.coulomb_sqrt(s.n, s.a_bohr, s.q, s.miller)
    e = ei.cpu().numpy()
    s_ref, o_ref, a_ref = pp.plasmon_pole(e, s.n, s.a_bohr, s.q, s.miller, sv, s.psi_v, occ, n_modes)
    sig, om, a = sig.cpu().numpy(), om.cpu().numpy(), a.cpu().numpy()
    e_sig = np.max(np.abs(sig - s_ref)) / abs(s_ref[0])
    e_om = np.max(np.abs(om - o_ref) / o_ref)
    overlap = np.abs(np.sum(np.conj(a_ref) * a, axis=0))         # |<a_ref, a>| per mode (phases are free)
    print(f"ng={len(sv)} modes={n_modes}: {its} iterations, residual {res:.1e}; sigma {e_sig:.1e}, "
          f"omega {e_om:.1e}, 1-overlap {np.max(1 - overlap):.1e}")
    return e_sig, e_om, overlap, its, (sig, om, a, s_ref, o_ref, a_ref, sv, e)


def test_small_system_modes(gw):
    s = gs.make_system(8, 6, 40, r2_psi=6.0, q=(0.2, 0.1, 0.05), seed=4).as_c64()
    ei, pv = gpu_eps_inv(gw, s)
    for nm in (1, 5, 8, 16):
        e_sig, e_om, ov, its, _ = compare(gw, s, ei, pv, nm, occ=2.0)
        # the residual bound 1e-10 gives eigenvalues to about its square and vectors to about 1e-10 / gap
        assert e_sig < 1e-12 and e_om < 1e-8 and np.min(ov) > 1 - 1e-8


def test_full_space_block_is_exact_in_one_iteration(gw):
    s = gs.make_system(6, 4, 20, r2_psi=4.0, q=(0.1, 0.2, 0.3), ng=30, seed=2).as_c64()
    ei, pv = gpu_eps_inv(gw, s)
    e_sig, e_om, ov, its, _ = compare(gw, s, ei, pv, 12)
    assert its == 1 and e_sig < 1e-13 and e_om < 1e-10 and np.min(ov) > 1 - 1e-10


def test_homogeneous_gas_closed_form(gw):
    n = (6, 6, 6)
    q = np.array([0.13, 0.07, 0.03])
    mv = np.array([[0, 0, 0], [1, 0, 0], [0, -1, 0]])
    mc = np.array([[1, 1, 0], [-1, 0, 2], [0, 0, 1], [2, -1, 1], [0, 2, -1], [-2, 1, 0], [1, -2, 2]])
    e_v = np.array([-0.31, -0.22, -0.12])
    e_c = np.array([0.15, 0.21, 0.33, 0.41, 0.52, 0.6, 0.75])
    a = gs.cell_side(6)
    miller = gs.sphere(n, r2=5.0, q=q)
    pv = dev(gs.plane_wave_orbitals(n, mv).astype(np.complex64))
    pc = dev(gs.plane_wave_orbitals(n, mc).astype(np.complex64))
    pgg = gw.polarizability(pv, pc, e_v, e_c, n, a, q, miller)
    ei = gw.eps_inverse(pgg, n, a, q, miller)
    occ, nm = 2.0, 6
    sig, om, modes, its, _ = gw.plasmon_pole(ei, n, a, q, miller, pv, occ, nm)
    sv = orc.coulomb_sqrt(n, a, q, miller)
    ptd = np.real(np.diag(pgg.cpu().numpy().astype(np.complex128)))
    eps_d = 1.0 - sv ** 2 * ptd
    sig_closed = np.sort(sv ** 2 * (1.0 / eps_d - 1.0))[:nm]
    sig = sig.cpu().numpy()
    assert np.max(np.abs(sig - sig_closed)) < 1e-10 * np.max(np.abs(sig_closed))
    idx = np.argmax(np.abs(modes.cpu().numpy()), axis=0)
    w2 = 4 * np.pi / a ** 3 * occ * 3 / (1.0 - 1.0 / eps_d[idx])
    # the density comes from complex64 orbitals: relative error at the FP32 level
    assert np.max(np.abs(om.cpu().numpy() ** 2 - w2) / w2) < 1e-6


def test_silicon_analogue_410_pole_form(gw):
    """410 G, q = pi/a (1,1,-1): modes and eps^-1(w) of the pole form with 1 and 5 modes against all
    410 (the oracle's full eigendecomposition), at frequencies below, between and above the poles."""
    s = gs.make_system(12, 8, 64, r2_psi=10.0, r2_p=25.0, q=(0.5, 0.5, -0.5), ng=410, seed=4).as_c64()
    ei, pv = gpu_eps_inv(gw, s)
    e_sig, e_om, ov, its, (sig, om, a, s_ref, o_ref, a_ref, sv, e) = compare(gw, s, ei, pv, 5)
    assert e_sig < 1e-12 and e_om < 1e-8 and np.min(ov) > 1 - 1e-8
    freqs = np.array([0.0, 0.3 * o_ref.min(), 0.5 * (o_ref[0] + o_ref[1]), 3.0 * o_ref.max()])
    got = gw.pp_eps_inverse(ei, s.n, s.a_bohr, s.q, s.miller, dev(a), dev(sig), dev(om), freqs).cpu().numpy()
    ref = pp.pp_eps_inverse(e, sig, om, a, sv, freqs)          # the same modes through the oracle's formula
    assert np.max(np.abs(got - ref)) < 1e-12 * np.max(np.abs(ref))
    s_all, o_all, a_all = pp.plasmon_pole(e, s.n, s.a_bohr, s.q, s.miller, sv, s.psi_v, 1.0, len(sv))
    g = int(np.argmax(np.abs(1.0 - np.diag(e))))
    lo = freqs[:2]
    all_modes = pp.pp_eps_inverse(e, s_all, o_all, a_all, sv, lo)[:, g, g]
    one = pp.pp_eps_inverse(e, s_ref[:1], o_ref[:1], a_ref[:, :1], sv, lo)[:, g, g]
    five = got[:2, g, g]
    print(f"eps^-1(w)[{g},{g}] at w = {lo}: all {all_modes.real}, 1 mode {one.real}, 5 modes {five.real}")
    assert np.all(np.abs(five - all_modes) < np.abs(one - all_modes) + 1e-15)
    assert abs(got[0, g, g] - e[g, g]) < 0.5 * abs(1.0 - e[g, g])      # 5 modes hold most of the static screening


def test_iteration_limit(gw):
    s = gs.make_system(8, 6, 40, r2_psi=6.0, q=(0.2, 0.1, 0.05), seed=4).as_c64()
    ei, pv = gpu_eps_inv(gw, s)
    with pytest.raises(gw.GwError, match="did not reach tol"):
        gw.plasmon_pole(ei, s.n, s.a_bohr, s.q, s.miller, pv, 1.0, 8, tol=1e-14, max_iter=2)


# Block sizes of the iteration against LAPACK: one workgroup's worth of rows and less, odd blocks (the Jacobi
# rounds' padding index), sizes around the thin product's 64 rows, the Gram chunks (48 rows) and its splits of K,
# and a matrix of rank one, whose dependent directions are dropped.  Tolerances as above: sigma to 1e-12 of
# |sigma_0|, every mode to 1e-9; omega follows from the modes.
@pytest.mark.parametrize("ng,nm,rank", [(1, 1, 0), (2, 2, 0), (7, 5, 0), (31, 16, 0), (33, 8, 0), (47, 4, 0), (65, 24, 0),
                                        (130, 16, 0), (515, 24, 0), (1100, 8, 0), (60, 1, 1)])
def test_block_sizes(gw, ng, nm, rank):
    rng = np.random.default_rng(ng)
    n, q = (12, 12, 12), np.array([0.1, 0.2, 0.3])
    mill = gs.sphere(n, count=ng, q=q)
    a = gs.cell_side(12)
    sv = orc.coulomb_sqrt(n, a, q, mill)
    x = rng.standard_normal((ng, rank or 2 * ng)) + 1j * rng.standard_normal((ng, rank or 2 * ng))
    d = 1.0 / (0.2 + np.arange(ng)) ** 1.5                         # a spectrum that falls as the screening's does
    s = -(x * d[:, None]) @ (x * d[:, None]).conj().T / (2 * ng)
    eps_inv = np.eye(ng) + s / (sv[:, None] * sv[None, :])
    psi = rng.standard_normal((3, 12 ** 3)) + 1j * rng.standard_normal((3, 12 ** 3))
    psi = (psi / np.sqrt((np.abs(psi) ** 2).sum(1))[:, None]).astype(np.complex64)
    print(f"[case] ng={ng} nm={nm} rank={rank}", flush=True)
    dev = lambda v: torch.from_numpy(np.ascontiguousarray(v)).to("cuda:0")
    sig, om, modes, its, res = gw.plasmon_pole(dev(eps_inv), n, a, q, mill, dev(psi), n_modes=nm)
    w, v = np.linalg.eigh(sv[:, None] * (eps_inv - np.eye(ng)) * sv[None, :])
    sig, modes = sig.cpu().numpy(), modes.cpu().numpy()
    assert np.max(np.abs(sig - w[:nm])) < 1e-12 * abs(w[0])
    for j in range(nm):
        gap = np.min(np.abs(np.delete(w, j) - w[j])) if ng > 1 else 1.0
        assert abs(abs(np.vdot(v[:, j], modes[:, j])) - 1.0) < max(1e-9, (1e-9 * abs(w[0]) / gap) ** 2)
    assert np.all(om.cpu().numpy() > 0) and res <= 1e-10


# More rows than one pass of the Gram kernel's workgroups holds (96 each, 32 workgroups): a matrix of known
# eigenvectors and values, tolerances as above.
@pytest.mark.parametrize("ng", [3071, 3100])
def test_long_blocks(gw, ng):
    rng = np.random.default_rng(ng)
    n, q, nm, rank = (20, 20, 20), np.array([0.1, 0.2, 0.3]), 8, 40
    mill = gs.sphere(n, count=ng, q=q)
    a = gs.cell_side(20)
    sv = orc.coulomb_sqrt(n, a, q, mill)
    u = np.linalg.qr(rng.standard_normal((ng, rank)) + 1j * rng.standard_normal((ng, rank)))[0]
    w = -1.0 / (0.2 + np.arange(rank)) ** 1.5
    eps_inv = np.eye(ng) + (u * w) @ u.conj().T / (sv[:, None] * sv[None, :])
    psi = rng.standard_normal((3, 20 ** 3)) + 1j * rng.standard_normal((3, 20 ** 3))
    psi = (psi / np.sqrt((np.abs(psi) ** 2).sum(1))[:, None]).astype(np.complex64)
    print(f"[case] ng={ng}", flush=True)
    dev = lambda v: torch.from_numpy(np.ascontiguousarray(v)).to("cuda:0")
    sig, _, modes, _, res = gw.plasmon_pole(dev(eps_inv), n, a, q, mill, dev(psi), n_modes=nm)
    modes = modes.cpu().numpy()
    assert np.max(np.abs(sig.cpu().numpy() - w[:nm])) < 1e-12 * abs(w[0]) and res <= 1e-10
    for j in range(nm):
        gap = np.min(np.abs(np.delete(w, j) - w[j]))
        assert abs(abs(np.vdot(u[:, j], modes[:, j])) - 1.0) < max(1e-9, (1e-9 * abs(w[0]) / gap) ** 2)


def test_a_value_that_is_not_finite_is_passed_on(gw):
    """A NaN in eps^-1 gives NaN strengths, in one iteration, and no error."""
    rng = np.random.default_rng(0)
    n, q, ng = (8, 8, 8), np.array([0.1, 0.2, 0.3]), 60
    eps_inv = np.eye(ng, dtype=np.complex128) * 0.5
    eps_inv[3, 4] = np.nan
    psi = (rng.standard_normal((2, 512)) + 1j * rng.standard_normal((2, 512))).astype(np.complex64)
    sig, _, _, its, _ = gw.plasmon_pole(dev(eps_inv), n, gs.cell_side(8), q, gs.sphere(n, count=ng, q=q), dev(psi),
                                        n_modes=4)
    assert its == 1 and np.all(np.isnan(sig.cpu().numpy()))


# The one-pass pole form (up to 32 modes) and the three-pass one, at the edges of the 64 x 64 tiles, with the row and
# column of q + G = 0 from the static matrix.  All weights of one frequency have the same sign, so the moduli of an
# entry's terms add up to at most the largest diagonal entry, and their rounding to 50 x 4 x 1.1e-16 = 2e-14 of it.
@pytest.mark.parametrize("ng,nm", [(1, 1), (63, 32), (64, 1), (65, 33), (130, 32), (130, 50)])
def test_pole_form_of_given_modes(gw, ng, nm):
    print(f"[case] ng={ng} nm={nm}", flush=True)
    rng = np.random.default_rng(ng + nm)
    for q in (np.zeros(3), np.array([0.1, 0.2, 0.3])):
        n, a = (12, 12, 12), gs.cell_side(12)
        mill = gs.sphere(n, count=ng, q=q)
        sv = orc.coulomb_sqrt(n, a, q, mill)
        ei = rng.standard_normal((ng, ng)) + 1j * rng.standard_normal((ng, ng))
        modes = rng.standard_normal((ng, nm)) + 1j * rng.standard_normal((ng, nm))
        sig, om, freqs = -rng.uniform(0.1, 1.0, nm), rng.uniform(1.0, 2.0, nm), np.array([0.0, 0.5, 3.0])
        got = gw.pp_eps_inverse(dev(ei), n, a, q, mill, dev(modes), dev(sig), dev(om), freqs).cpu().numpy()
        ref = pp.pp_eps_inverse(ei, sig, om, modes, sv, freqs)
        assert np.max(np.abs(got - ref)) <= 1e-13 * np.max(np.abs(ref))
        if not q.any():
            assert np.array_equal(got[:, 0], ref[:, 0]) and np.array_equal(got[:, :, 0], ref[:, :, 0])


def test_pole_forms_round_alike(gw):
    """One mode by the one-pass form and, with 32 modes of zeros beside it, by the three-pass one: with powers of two
    for its values the sums are exact, and the division by sqrt(V) sqrt(V') leaves the same bits."""
    rng = np.random.default_rng(0)
    n, q, ng = (12, 12, 12), np.array([0.1, 0.2, 0.3]), 200
    mill = gs.sphere(n, count=ng, q=q)
    one = dev(2.0 ** rng.integers(-2, 3, (ng, 1)) + 0j)
    many = torch.cat([one, torch.zeros((ng, 32), dtype=one.dtype, device=one.device)], 1)
    ei = dev(np.eye(ng, dtype=np.complex128))
    out = [gw.pp_eps_inverse(ei, n, gs.cell_side(12), q, mill, m.contiguous(), dev(np.full(m.shape[1], -1.0)),
                             dev(np.ones(m.shape[1])), [0.0]) for m in (one, many)]
    assert torch.equal(out[0], out[1])
