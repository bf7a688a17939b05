"""Pair products whose rows start anywhere in a 128-byte line, against NumPy in FP64 (tolerance as in
test_gpu_parity: 2e-7 of the largest value, FP32 rounding of a three-factor product)."""
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


# One point to several segments of 512, one point either side of a segment, every remainder of a line; output that
# starts in the middle of a line (offset, in values); more energies than a launch's arguments hold (500 bands),
# and than the launches that carry them (2100).
@pytest.mark.parametrize("nr,nv,nc,offset", [(1, 1, 1, 0), (15, 3, 5, 0), (16, 9, 4, 0), (511, 8, 4, 0), (512, 2, 9, 0),
                                             (513, 1, 7, 0), (1025, 3, 3, 0), (527, 9, 13, 0), (1536, 2, 5, 3),
                                             (700, 5, 6, 1), (529, 3, 4, 15), (40, 3, 500, 0), (17, 2, 2100, 0)])
def test_rows_at_every_line_offset(gw, nr, nv, nc, offset):
    rng = np.random.default_rng(nr)
    a = (rng.standard_normal((nv + nc, nr)) + 1j * rng.standard_normal((nv + nc, nr))).astype(np.complex64)
    ev, ec = np.sort(rng.uniform(-0.6, 0.0, nv)), np.sort(rng.uniform(0.05, 1.2, nc))
    pv, pc = torch.from_numpy(a[:nv].copy()).cuda(), torch.from_numpy(a[nv:].copy()).cuda()
    print(f"[case] nr={nr} nv={nv} nc={nc} offset={offset}", flush=True)
    buf = torch.full((nv * nc * nr + 2 * offset + 32,), 7.0, dtype=torch.complex64, device="cuda:0")
    out = buf[offset:offset + nv * nc * nr].view(nv * nc, nr)
    gw.pair_products(pv, pc, ev, ec, prefactor=2.0, out=out)
    ref = (a[:nv].astype(np.complex128).conj()[:, None, :] * a[nv:]
           * np.sqrt(2.0 / (ec[None, :] - ev[:, None]))[:, :, None]).reshape(nv * nc, nr)
    assert np.max(np.abs(out.cpu().numpy() - ref)) < 2e-7 * np.max(np.abs(ref))
    rest = torch.cat([buf[:offset], buf[offset + nv * nc * nr:]])
    assert bool((rest == 7.0).all())                       # nothing written outside the output


# Each split of the occupied bands over workgroups (one band, up to four, five to eight, two blocks of five to eight of
# which the last is short or full), at the edges of its segments and with the scales from the table (490 bands) and
# from the launch's arguments.
@pytest.mark.parametrize("nv", [1, 2, 3, 4, 5, 6, 7, 8, 9, 11, 12, 13, 17])
@pytest.mark.parametrize("nr,nc,offset", [(1, 3, 1), (255, 5, 0), (257, 490, 7), (513, 6, 15), (1040, 4, 0)])
def test_splits_of_the_occupied_bands(gw, nr, nv, nc, offset):
    test_rows_at_every_line_offset(gw, nr, nv, nc, offset)
