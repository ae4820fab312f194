"""The autotuner's cache over plans of one band class: a choice made on a plan
with block spectra is not taken for one without (and the reverse), and an entry
whose item size the plan's own search would not try is measured again."""
import os

import numpy as np
import pytest

from paper_2407_10797_amd import synth as S

pytestmark = pytest.mark.gpu


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


def _plan(nbins):
    from paper_2407_10797_amd import fstat
    T = 4.0e6
    g = S.Grid(T_obs=T, df=1.0 / T, k_lo=int(0.02 * T), nbins=nbins)
    psd = S.psd_tdix(g.freqs())
    return fstat.Plan(S.noise(psd, g.df, 9700), psd, g.T_obs, g.df, g.k_lo)


def _points(n=32):
    import torch
    T = 4.0e6
    box = np.array([[1.6 * T, 3.0 * T], [25.0, 40.0], [0.0, 0.9], [0.0, np.pi], [0.0, 2 * np.pi],
                    [0.0, 0.1]])
    return torch.from_numpy(S.uniform_box(box, n, 9701)).cuda()


# sizes of one class (2^17, 2^15 bins) without and with spectra of the precision
@pytest.mark.parametrize("mixed, sizes", [(False, (70_001, 120_001)), (True, (20_001, 30_001))])
@pytest.mark.parametrize("first", [0, 1])
def test_plans_with_and_without_spectra_keep_their_own_choice(cache, mixed, sizes, first):
    npart = 600 + 600 * first         # keys of its own: choices last as long as the process
    prm = _points()
    a, b = _plan(sizes[first]), _plan(sizes[1 - first])
    try:
        print(f"[tune] mixed={mixed}, {sizes[first]} bins before {sizes[1 - first]}", flush=True)
        ca = a.autotune(prm, npart, mixed=mixed, force=True)
        cb = b.autotune(prm, npart, mixed=mixed)
        assert ca[2] > 0 and cb[2] > 0                        # both measured
        assert a.autotune(prm, npart, mixed=mixed) == (ca[0], ca[1], -1.0)
        assert b.autotune(prm, npart, mixed=mixed) == (cb[0], cb[1], -1.0)
        assert (cb if first == 0 else ca)[0] >= 2048          # the plan with spectra
    finally:
        a.close()
        b.close()


def test_entries_outside_the_plans_search_are_measured_again(cache):
    prm = _points()
    plan = _plan(20_001)
    try:
        plan.autotune(prm, 4096, mixed=True, force=True)
        key = cache.read_text().splitlines()[-1].split("|")[0]
        with open(cache, "a") as f:
            f.write(key.replace(" np4096 ", " np8192 ") + "|5120 1 0\n")      # above the per-bin loop's tile
            f.write(key.replace(" np4096 ", " np16384 ") + "|512 2 0\n")
        c, m, ms = plan.autotune(prm, 8192, mixed=True)
        assert ms > 0 and c <= 4608
        assert plan.autotune(prm, 16384, mixed=True) == (512, 2, -1.0)
        plan.eval(prm, 8192, mixed=True)
    finally:
        plan.close()
