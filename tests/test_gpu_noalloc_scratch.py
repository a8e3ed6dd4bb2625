"""What sht_adjoint_noalloc accepts: requests whose phase rows and one partial
vector per 128 ring pairs fit 64 MiB, also on grids whose ring pairs are padded
to more tiles than that; the result is sht_adjoint's, bit for bit."""
import ctypes

import pytest

from tests.test_zz_no_alloc import _call

pytestmark = pytest.mark.gpu

CASES = [
    (("healpix", 90), 180, 33),    # 180 pairs in four tile groups, three of them taking turns in two vectors
    (("healpix", 64), 230, 24),    # 128 pairs in three tile groups, two taking turns in one
    (("healpix", 31), 600, 16),    # padded polar slots, a partial vector where 64-pair tiles have one
    (("gl", 4, 9), 2500, 1),       # two ring pairs in two forms of the recurrence
    (("gl", 70, 141), 1000, 7),
    (("healpix", 151), 56, 107),   # two tiles per wave where the waves allow four: four tile groups after the first
    (("healpix", 256), 512, 2),    # as many partial vectors as fit
]


@pytest.mark.parametrize("spec,lmax,nmaps", CASES)
def test_noalloc_takes_what_fits_its_scratch(spec, lmax, nmaps):
    import torch
    from paper_1710_00621_amd import _lib, crsolve
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    lib = _lib.lib()
    print(f"case noalloc scratch {spec} lmax={lmax} nmaps={nmaps}", flush=True)
    g = crsolve.Grid.from_spec(spec)
    gen = torch.Generator(device="cpu").manual_seed(89)
    maps = torch.randn(nmaps, g.npix, generator=gen, dtype=torch.float64).to("cuda")
    st, ref = _call(lib, "sht_adjoint", g, lmax, maps, torch, crsolve)
    assert st == 0
    st, got = _call(lib, "sht_adjoint_noalloc", g, lmax, maps, torch, crsolve)
    buf = ctypes.create_string_buffer(512)
    lib.crs_last_error(buf, 512)
    assert st == 0, buf.value
    assert torch.equal(got, ref)
    # strided results, the gaps untouched
    pad = torch.full((nmaps, (lmax + 1) ** 2 + 3), 7.0, dtype=torch.float64, device="cuda")
    st = lib.sht_adjoint_noalloc(g._h, lmax, nmaps, maps.data_ptr(), g.npix, pad.data_ptr(), pad.shape[1],
                                 torch.cuda.current_stream().cuda_stream)
    assert st == 0
    torch.cuda.synchronize()
    assert torch.equal(pad[:, :-3], ref) and bool((pad[:, -3:] == 7.0).all())
