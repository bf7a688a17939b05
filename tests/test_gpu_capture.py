"""Calls captured into a HIP graph: replays read the caller's energies and Miller lists as they are then, whatever eager
calls with other ones came between, and equal the eager result bit for bit."""
import numpy as np
import pytest

import gwsynth as gs

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


def captured(call):
    call()                                             # sizes the workspace
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        call()
    return g


@pytest.mark.parametrize("entry", ["noalloc", "update", "pairs"])
def test_replays_read_the_energies(gw, entry):
    print(f"[case] {entry}", flush=True)
    s = gs.make_system(12, 8, 64, r2_psi=10.0, seed=3)
    pv, pc = dev(s.psi_v.astype(np.complex64)), dev(s.psi_c.astype(np.complex64))
    ev, ec = np.array(s.e_v, np.float64), np.array(s.e_c, np.float64)
    ctx, tile = gw.Context(0), gw.tile_names().index(gw.default_tile_name("fp32"))
    shape = (8 * 64, s.nr) if entry == "pairs" else (s.nr, s.nr)
    out, eager = (torch.empty(shape, dtype=torch.complex64, device="cuda:0") for _ in range(2))
    call = {"noalloc": lambda o, **k: gw.polarizability_r_noalloc(pv, pc, ev, ec, o, ctx=ctx, **k),
            "update": lambda o, **k: gw.polarizability_r(pv, pc, ev, ec, out=o, ctx=ctx, **k),
            "pairs": lambda o, **k: gw.pair_products(pv, pc, ev, ec, out=o, ctx=ctx)}[entry]
    g = captured(lambda: call(out))                    # the update runs uncut
    seen = []
    for scale in (1.0, 1.3, 0.7):
        ec *= scale
        g.replay()
        torch.cuda.synchronize()
        seen.append(out.clone())
        call(eager, tile=tile)
        torch.cuda.synchronize()
        assert torch.equal(out, eager), scale
    assert not torch.equal(seen[0], seen[1])


def test_replays_read_the_miller_list(gw):
    n, a, q, ctx = (12, 12, 12), 10.0, np.array([0.1, 0.2, 0.3]), gw.Context(0)
    first = np.ascontiguousarray(gs.sphere(n, count=200), np.int32)
    other = first[::-1].copy()
    g0 = torch.Generator().manual_seed(0)
    p = torch.randn(200, 200, generator=g0, dtype=torch.complex64).to("cuda:0")
    modes = torch.randn(200, 5, generator=g0, dtype=torch.complex128).to("cuda:0")
    ei = torch.randn(200, 200, generator=g0, dtype=torch.complex128).to("cuda:0")
    sig, om = dev(-np.arange(5.0, 0.0, -1.0)), dev(np.linspace(1.0, 2.0, 5))
    eps, ew = (torch.empty(s, dtype=torch.complex128, device="cuda:0") for s in ((200, 200), (1, 200, 200)))
    calls = [lambda m: gw.epsilon(p, n, a, q, m, out=eps, ctx=ctx),
             lambda m: gw.pp_eps_inverse(ei, n, a, q, m, modes, sig, om, [0.3], out=ew, ctx=ctx)]
    for call, out in zip(calls, (eps, ew)):
        call(first)
        torch.cuda.synchronize()
        want = out.clone()
        g = captured(lambda: call(first))
        for _ in range(3):
            call(other)
            torch.cuda.synchronize()
            assert not torch.equal(out, want)
            g.replay()
            torch.cuda.synchronize()
            assert torch.equal(out, want)
            call(first)
            torch.cuda.synchronize()
            assert torch.equal(out, want)
