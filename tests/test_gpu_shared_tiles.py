"""Update tiles cut along K (the default tile where the last round of tiles leaves CUs idle) against the FP64 sum:
FP32 1e-5, split precisions 1e-4 as everywhere; and the workspace rules of the parts' buffer."""
import numpy as np
import pytest

import oracle as orc

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def gw():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1810_07772_amd as gw
    gw.load()
    return gw


def bands(nr, nv, nc, seed=0):
    rng = np.random.default_rng(seed)
    a = (rng.standard_normal((nv + nc, nr)) + 1j * rng.standard_normal((nv + nc, nr))).astype(np.complex64)
    a /= np.float32(np.sqrt(2 * nr))
    return a[:nv].copy(), a[nv:].copy(), np.sort(rng.uniform(-0.6, 0.0, nv)), np.sort(rng.uniform(0.05, 1.2, nc))


def reference(pv, pc, ev, ec):
    p = np.zeros((pv.shape[1],) * 2, np.complex128)
    for v in range(len(pv)):
        f = pv[v].astype(np.complex128).conj()[None, :] * pc * np.sqrt(1.0 / (ec - ev[v]))[:, None]
        p -= f.conj().T @ f
    return p


def dev(x):
    return torch.from_numpy(np.ascontiguousarray(x)).to("cuda:0")


# One tile and many parts; parts that begin inside an unoccupied chunk (nv = 7), with ragged points and bands;
# one occupied band; whole rounds before the cut tiles (2900 points: 276 FP32 tiles, of which 20 are cut; 4200
# points: 289 blocks, of which 33); parts longer than 32768 pairs, whose sums are folded on the way (27 points,
# 512 x 4096 bands).
@pytest.mark.parametrize("prec", ["fp32", "bf16", "fp16"])
@pytest.mark.parametrize("nr,nv,nc", [(64, 3, 100), (1000, 7, 101), (129, 1, 600), (2900, 5, 50), (4200, 3, 60),
                                      (27, 512, 4096)])
def test_cut_tiles_match_the_sum(gw, prec, nr, nv, nc):
    print(f"[case] {prec} nr={nr} nv={nv} nc={nc}", flush=True)
    pv, pc, ev, ec = bands(nr, nv, nc)
    got = gw.polarizability_r(dev(pv), dev(pc), ev, ec, precision=prec).cpu().numpy()
    e = orc.rel_f(got, reference(pv, pc, ev, ec))
    assert e < (1e-5 if prec == "fp32" else 1e-4)
    assert np.max(np.abs(got - got.conj().T)) <= (1e-6 if prec == "fp32" else 1e-4) * np.max(np.abs(got))


@pytest.mark.parametrize("prec", ["fp32", "bf16"])
def test_cut_tiles_accumulate(gw, prec):
    pv, pc, ev, ec = bands(700, 9, 64, seed=1)
    p = torch.full((700, 700), 0.25 - 0.5j, dtype=torch.complex64, device="cuda:0")
    p0 = torch.triu(p, 1) + torch.triu(p, 1).conj().T                     # a Hermitian start
    out = gw.polarizability_r(dev(pv), dev(pc), ev, ec, precision=prec, accumulate=True, out=p0.clone())
    ref = p0.cpu().numpy().astype(np.complex128) + reference(pv, pc, ev, ec)
    assert orc.rel_f(out.cpu().numpy(), ref) < (1e-5 if prec == "fp32" else 1e-4)


def test_cut_tiles_give_way_under_a_workspace_cap(gw):
    """A cap that the call without parts just meets: the update runs uncut or its parts' buffer is freed for the
    transforms; a call with a chosen tile needs no parts."""
    import gwsynth as gs
    s = gs.make_system(16, 4, 64, r2_psi=20.0, seed=2)
    c64 = lambda x: dev(x.astype(np.complex64))
    pv, pc = c64(s.psi_v), c64(s.psi_c)
    tile = gw.tile_names().index(gw.default_tile_name("fp32"))
    args = (s.e_v, s.e_c, s.n, s.a_bohr, s.q, s.miller)
    plain = gw.Context(0)
    ref = gw.polarizability(pv, pc, *args, tile=tile, ctx=plain)
    need = plain.workspace_bytes
    capped = gw.Context(0, workspace_cap=need)
    for _ in range(2):
        out = gw.polarizability(pv, pc, *args, ctx=capped)
        assert orc.rel_f(out.cpu().numpy(), ref.cpu().numpy()) < 1e-6
        assert capped.workspace_bytes <= need
    tight = gw.Context(0, workspace_cap=(4 + 64) * 8 + 2 * 4 * 64 * 4 + 1024)
    p = gw.polarizability_r(pv, pc, s.e_v, s.e_c, ctx=tight)
    assert torch.equal(p, gw.polarizability_r(pv, pc, s.e_v, s.e_c, tile=tile, ctx=plain))


# Whole rounds before the cut tiles in every precision: FP32 256 tiles and 20 in seven parts each, the others 256 blocks
# and 16 in eight parts each (of the sizes above, the split precisions cut none at 2900 and 4200 points).  That the
# tiles are cut shows in the workspace, which holds their parts.
@pytest.mark.parametrize("accumulate", [False, True])
@pytest.mark.parametrize("prec", ["fp32", "bf16", "fp16"])
def test_cut_after_whole_rounds(gw, prec, accumulate):
    nr, nv, nc = (2900, 5, 50) if prec == "fp32" else (4096, 4, 250)
    print(f"[case] {prec} accumulate={accumulate}", flush=True)
    pv, pc, ev, ec = bands(nr, nv, nc, seed=3)
    whole, cut = gw.Context(0), gw.Context(0)
    tile = gw.tile_names().index(gw.default_tile_name(prec))
    p0 = torch.full((nr, nr), 0.25 - 0.5j, dtype=torch.complex64, device="cuda:0")
    p0 = torch.triu(p0, 1) + torch.triu(p0, 1).conj().T
    run = lambda ctx, tile: gw.polarizability_r(dev(pv), dev(pc), ev, ec, precision=prec, accumulate=accumulate,
                                                out=p0.clone(), tile=tile, ctx=ctx).cpu().numpy()
    got, plain = run(cut, -1), run(whole, tile)
    parts = 20 * 7 * 4 if prec == "fp32" else 16 * 8 * 8
    assert cut.workspace_bytes - whole.workspace_bytes >= parts * 32768
    ref = reference(pv, pc, ev, ec) + (p0.cpu().numpy() if accumulate else 0.0)
    tol = 1e-5 if prec == "fp32" else 1e-4
    assert orc.rel_f(got, ref) < tol and orc.rel_f(plain, ref) < tol
    assert not np.array_equal(got, plain)


def test_cut_fp16_accumulate(gw):
    pv, pc, ev, ec = bands(1000, 7, 101, seed=4)
    p0 = torch.eye(1000, dtype=torch.complex64, device="cuda:0")
    got = gw.polarizability_r(dev(pv), dev(pc), ev, ec, precision="fp16", accumulate=True, out=p0.clone())
    assert orc.rel_f(got.cpu().numpy(), np.eye(1000) + reference(pv, pc, ev, ec)) < 1e-4


def test_tuning_keeps_the_cut(gw):
    """A tuned shape is no slower than an untuned one, and a batch of it equals the calls of their own bit for bit."""
    import gwsynth as gs
    b = gs.make_batched_q(n=10, nv=8, nc=100, r2_psi=9.0, nq=2, sizes=(100, 120))
    pv = dev(b["psi_v"].astype(np.complex64))
    ctx = gw.Context(0)
    jobs = [dict(psi_c=dev(j["psi_c"].astype(np.complex64)), e_c=j["e_c"], q=j["q"], miller=j["miller"],
                 p_gg=torch.empty((len(j["miller"]),) * 2, dtype=torch.complex64, device="cuda:0"), eps_inv=None)
            for j in b["jobs"]]
    gw.polarizability_batched(pv, b["e_v"], b["n"], b["a_bohr"], jobs, precision="fp32", ctx=ctx)
    for j in jobs:
        out = gw.polarizability(pv, j["psi_c"], b["e_v"], j["e_c"], b["n"], b["a_bohr"], j["q"], j["miller"],
                                precision="fp32", ctx=ctx)
        assert torch.equal(out, j["p_gg"])
    # 36 tiles on 256 CUs: cut seven-fold they take a quarter of their time in one piece (the best of three tunings)
    default = gw.default_tile_name("fp32")
    runs = [gw.autotune(pv, jobs[0]["psi_c"], b["e_v"], jobs[0]["e_c"], precision="fp32", ctx=gw.Context(0))[1]
            for _ in range(3)]
    best = {k: min(r[k] for r in runs) for k in runs[0]}
    assert best[default] < 0.5 * min(v for k, v in best.items() if k != default)
