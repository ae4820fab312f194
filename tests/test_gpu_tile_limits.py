"""Work-item sizes above the interpolating loop's tile (2560 bins FP64, 4608
mixed) that a plan got from tuning the exact loop are refused by that loop, on
plans with and without block spectra; and a caller's item size stays one tile
per item on the mixed path when only FP64 is tuned."""
import os

import numpy as np
import pytest

from paper_2407_10797_amd import synth as S

pytestmark = pytest.mark.gpu
T = 4.0e7


@pytest.fixture
def cache(tmp_path):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    old = os.environ.get("FSTAT_TUNE_CACHE")
    path = tmp_path / "tune.txt"
    os.environ["FSTAT_TUNE_CACHE"] = str(path)
    yield path
    del os.environ["FSTAT_TUNE_CACHE"]
    if old is not None:
        os.environ["FSTAT_TUNE_CACHE"] = old


def _plan(nbins, chunk=0):
    from paper_2407_10797_amd import fstat
    g = S.Grid(T_obs=T, df=1.0 / T, k_lo=int(0.04 * T), nbins=nbins)
    psd = S.psd_tdix(g.freqs())
    return fstat.Plan(S.noise(psd, g.df, 9800), psd, g.T_obs, g.df, g.k_lo, chunk=chunk)


def _points(n=24):
    import torch
    box = np.array([[1.02 * T, 1.3 * T], [25.0, 40.0], [0.0, 0.9], [0.0, np.pi], [0.0, 2 * np.pi],
                    [0.0, 0.1]])
    return torch.from_numpy(S.uniform_box(box, n, 9801)).cuda()


@pytest.mark.parametrize("nbins", [20_001, 800_001])      # without, with spectra
@pytest.mark.parametrize("mixed", [False, True])
def test_exact_loop_sizes_are_refused_by_the_interpolating_loop(cache, nbins, mixed):
    from paper_2407_10797_amd import fstat
    prm = _points()
    plan = _plan(nbins)
    try:
        print(f"[limits] {nbins} bins, mixed={mixed}", flush=True)
        ref = plan.eval(prm, 4, mixed=mixed, exact=True)
        plan.autotune(prm, 2000, mixed=mixed, exact=True, force=True)
        key = cache.read_text().splitlines()[-1].split("|")[0]
        with open(cache, "a") as f:
            f.write(key.replace(" np2048 ", " np4096 ") + "|8192 1 0\n")
        assert plan.autotune(prm, 4000, mixed=mixed, exact=True) == (8192, 1, -1.0)
        for noalloc in (False, True):
            with pytest.raises(fstat.FstatError) as err:
                plan.eval(prm, 4, mixed=mixed, noalloc=noalloc)
            assert err.value.code == fstat.FSTAT_EINVAL
        F = plan.eval(prm, 4, mixed=mixed, exact=True)
        np.testing.assert_allclose(F.cpu().numpy(), ref.cpu().numpy(), rtol=1e-5 if mixed else 1e-9)
    finally:
        plan.close()


def test_callers_tile_on_the_mixed_path_after_fp64_tuning(cache):
    prm = _points()
    plan, own = _plan(800_001, chunk=1024), None
    try:
        c = plan.autotune(prm, 4, force=True)[0]
        plan.eval(prm, 4, mixed=True)
        items = plan.interp_stats()[0]
        own = _plan(800_001, chunk=c)
        own.eval(prm, 4, mixed=True)
        print(f"[limits] FP64 tuned to {c} bins: {items} mixed items", flush=True)
        assert items == own.interp_stats()[0]
        plan.autotune(prm, 4, mixed=True, force=True)     # the mixed path's own choice
        plan.eval(prm, 4, mixed=True)
        assert plan.interp_stats()[0] != items or c >= 5120
    finally:
        plan.close()
        if own is not None:
            own.close()
