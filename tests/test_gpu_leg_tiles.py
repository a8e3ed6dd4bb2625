"""The Legendre kernels at forced numbers of tiles per wave, on a grid with
several tile groups of each form: five and more polar and belt tiles (700 ring
pairs), so that groups of four and of two are followed by ragged ones."""
import numpy as np
import pytest

from oracle import geometry, sht

pytestmark = pytest.mark.gpu

SPEC, LMAX = ("healpix", 350), 61
NMAPS = 9
_ref = {}


def _reference():
    """Oracle transforms of nine maps, formed once."""
    if not _ref:
        og = geometry.make_grid(SPEC)
        rng = np.random.default_rng(103)
        _ref["alm"] = rng.standard_normal((NMAPS, sht.nalm(LMAX)))
        # a ring in three carries data: the oracle's sums are naive
        m = np.zeros((NMAPS, og.npix))
        keep = np.arange(0, og.nring, 3)
        for r in keep:
            m[:, og.offset[r]:og.offset[r] + og.nphi[r]] = rng.standard_normal((NMAPS, og.nphi[r]))
        _ref["maps"] = m
        sub = geometry.Grid("rings", og.z[keep], og.sint[keep], og.nphi[keep], og.phi0[keep],
                            og.ring_weight[keep], {})
        pick = np.concatenate([np.arange(og.offset[r], og.offset[r] + og.nphi[r]) for r in keep])
        _ref["pick"] = pick
        _ref["synth"] = sht.synth(sub, LMAX, _ref["alm"])
        _ref["adjoint"] = sht.adjoint(sub, LMAX, m[:, pick])
    return _ref


@pytest.mark.parametrize("tiles", [1, 2, 4])
@pytest.mark.parametrize("nmaps", [1, 2, 3, 4, 5, 6, 8, 9])
def test_forced_tiles_match_oracle(nmaps, tiles, monkeypatch):
    """1e-12 of the largest value: 61 steps and 1399 rings of rounding (1e-14)
    with the oracle's own phases (m phi up to 400, rounded: 5e-14) beside it."""
    import torch
    from paper_1710_00621_amd import crsolve
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    monkeypatch.setenv("CRS_LEG_TS", str(tiles))
    monkeypatch.setenv("CRS_LEG_TA", str(tiles))
    print(f"case forced tiles {tiles} nmaps={nmaps}", flush=True)
    ref = _reference()
    g = crsolve.Grid.from_spec(SPEC)
    c = crsolve.legendre_choice(g, LMAX, nmaps)
    assert c["adjoint_tiles_per_wave"] == tiles
    assert c["synth_pairs_per_lane"] == min(tiles, 4 if nmaps == 1 else 2 if nmaps <= 4 else 1)
    dev = torch.device("cuda")
    got = crsolve.sht_synth(g, LMAX, torch.tensor(ref["alm"][:nmaps], device=dev)).cpu().numpy()[:, ref["pick"]]
    back = crsolve.sht_adjoint(g, LMAX, torch.tensor(ref["maps"][:nmaps], device=dev)).cpu().numpy()
    for a, b in ((got, ref["synth"][:nmaps]), (back, ref["adjoint"][:nmaps])):
        assert np.abs(a - b).max() < 1e-12 * np.abs(b).max()
