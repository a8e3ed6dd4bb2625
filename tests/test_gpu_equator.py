"""Accuracy of the transforms on the rings next to the equator and in the belt,
where lambda_lm(z) is small against lambda_lm(z) / z or the recurrence turns
fastest: against 80-bit Legendre functions, normalised by those rings alone.

Bound: each of L / 2 steps of a two-step recurrence rounds a handful of times by
at most 2^-53 of its function, errors that add up like the square root of their
number: 2 sqrt(L) 2^-53 (rms over the compared values).  In the belt the phase
error of a step acts on a neighbour that is 1 / z away: twice that."""
import math

import numpy as np
import pytest

from oracle import geometry, sht

pytestmark = pytest.mark.gpu

LD = np.longdouble


def _lambda_ld(z, sint, lmax, m):
    """lambda_lm, l = m .. lmax, in 80 bits ([l - m, ring])."""
    z = np.asarray(z, dtype=LD)
    lam = np.zeros((lmax - m + 1, len(z)), dtype=LD)
    cur = 1 / np.sqrt(4 * LD(math.pi) + 4 * LD(1.2246467991473531772e-16)) * np.ones_like(z)
    for k in range(1, m + 1):
        cur = cur * np.sqrt((2 * LD(k) + 1) / (2 * LD(k))) * np.asarray(sint, dtype=LD)
    prev = np.zeros_like(z)
    l = np.arange(m, lmax + 2).astype(LD)
    eps = np.sqrt((l * l - m * m) / (4 * l * l - 1))
    for j in range(lmax - m + 1):
        lam[j] = cur
        prev, cur = cur, (z * cur - eps[j] * prev) / eps[j + 1]
    return lam


def _angles(og, r, m):
    """m phi of the pixels of ring r, reduced to one turn before rounding."""
    n = int(og.nphi[r])
    num = int(round(float(og.phi0[r]) * n / math.pi))  # phi0 = num pi / n, num 0 or 1
    return ((m * (num + 2 * np.arange(n, dtype=np.int64))) % (2 * n)) * (math.pi / n)


def _rings(og, lmax, where):
    eq = (og.nring - 1) // 2
    if where == "equator":
        k = [eq, eq + 1, eq - 2, eq + 5, eq - 9]
    else:  # |z| about 0.2, 0.45, 0.62, 0.7 north and south
        k = [int(np.argmin(np.abs(np.asarray(og.z) - z))) for z in (0.2, -0.45, 0.62, -0.7)]
    return np.array(sorted(set(k)))


CASES = [
    # every number of maps that has its own kernel, one and several tiles per wave, odd and even lmax
    (("healpix", 1024), 2000, 1), (("healpix", 512), 1023, 2), (("healpix", 256), 512, 3),
    (("healpix", 256), 513, 8), (("healpix", 128), 256, 4), (("healpix", 100), 201, 5),
    (("healpix", 64), 128, 6), (("healpix", 64), 128, 1), (("gl", 513, 1026), 512, 7),
]


@pytest.mark.parametrize("where", ["equator", "belt"])
@pytest.mark.parametrize("spec,lmax,nmaps", CASES)
def test_rings_near_the_equator_keep_their_accuracy(spec, lmax, nmaps, where):
    import torch
    from paper_1710_00621_amd import crsolve
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    print(f"case {where} {spec} lmax={lmax} nmaps={nmaps}", flush=True)
    og = geometry.make_grid(spec)
    g = crsolve.Grid.from_spec(spec)
    rings = _rings(og, lmax, where)
    # the functions of a ring pair are those of its northern ring
    north = np.minimum(rings, og.nring - 1 - rings)
    z = g.pixel_centres()[0][og.offset[north]] * np.where(rings == north, 1.0, -1.0)
    st = np.asarray(og.sint)[north]
    # (Gauss-Legendre nodes of two programs differ by an ulp of sin theta, m of them in lambda_mm)
    top = lmax if spec[0] == "healpix" else 16
    ms = [m for m in (0, 1, 2, 3, 7, 16, 63, 100, 250, 511, 900, 1500, 1999) if m <= top]
    rng = np.random.default_rng(83)
    tol = (2.0 if where == "equator" else 4.0) * math.sqrt(lmax) * 2.0 ** -53
    # synthesis of those m alone
    alm = np.zeros((nmaps, sht.nalm(lmax)))
    # adjoint of maps that are zero on every other ring
    maps = np.zeros((nmaps, og.npix))
    for r in rings:
        maps[:, og.offset[r]:og.offset[r] + og.nphi[r]] = rng.standard_normal((nmaps, og.nphi[r]))
    ref = [np.zeros((nmaps, int(og.nphi[r])), dtype=LD) for r in rings]
    cols, want = [], []
    for m in ms:
        lam = _lambda_ld(z, st, lmax, m)
        cm = LD(1) if m == 0 else np.sqrt(LD(2))
        n, o = lmax - m + 1, sht.m_offset(lmax, m)
        for part in range(1 if m == 0 else 2):
            s = slice(o + part * n, o + (part + 1) * n)
            alm[:, s] = rng.standard_normal((nmaps, n)) / np.sqrt(1.0 + np.arange(m, lmax + 1))
            F = cm * (alm[:, s].astype(LD) @ lam)
            v = np.zeros((nmaps, n), dtype=LD)
            for i, r in enumerate(rings):
                ang = _angles(og, r, m)
                e = (np.cos(ang) if part == 0 else np.sin(ang)).astype(LD)
                ref[i] += F[:, i:i + 1] * e
                px = maps[:, og.offset[r]:og.offset[r] + og.nphi[r]].astype(LD)
                v += cm * (px @ e)[:, None] * lam[:, i]
            cols.append(np.arange(s.start, s.stop))
            want.append(v)
    dev = torch.device("cuda")
    got = crsolve.sht_synth(g, lmax, torch.tensor(alm, device=dev)).cpu().numpy()
    got = np.concatenate([got[:, og.offset[r]:og.offset[r] + og.nphi[r]] for r in rings], axis=1)
    ref = np.concatenate(ref, axis=1)
    err_s = float(np.sqrt(np.mean((got - ref) ** 2) / np.mean(ref ** 2)))
    back = crsolve.sht_adjoint(g, lmax, torch.tensor(maps, device=dev)).cpu().numpy()
    want = np.concatenate(want, axis=1)
    err_a = float(np.sqrt(np.mean((back[:, np.concatenate(cols)] - want) ** 2) / np.mean(want ** 2)))
    print(f"rms synthesis {err_s:.2e} adjoint {err_a:.2e} bound {tol:.2e}", flush=True)
    assert err_s < tol and err_a < tol
