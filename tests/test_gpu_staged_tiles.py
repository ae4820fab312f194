"""The per-bin loop on items longer than its LDS stage (2560 bins FP64, 4608
mixed): a wave takes such an item in parts and adds to its sums.  FP64: items of
two 2560-bin tiles above the frequency where the block loop ends; mixed: 5120-bin
tiles of chirps too slow for the block loop.  Against the exact template at every
bin, with the interpolating loops' bars (5e-10 relative FP64, 1e-4 mixed): a part
left out or taken twice is an error of order one."""
import os

import numpy as np
import pytest

from paper_2407_10797_amd import synth as S

pytestmark = pytest.mark.gpu
MSUN_S = 4.925490947641267e-6


@pytest.fixture(scope="module")
def torch_cuda():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    return torch


def _compare(plan, prm, npart, mixed, bar):
    P = plan.eval(prm, npart, mixed=mixed, want_parts=True)[1].cpu().numpy()
    items, rej, _, mix = plan.interp_stats(bin_mix=True)
    runs = sum(mix[7:13]) / (items - rej)
    Pe = plan.eval(prm, npart, exact=True, want_parts=True)[1].cpu().numpy()
    r = np.abs(P - Pe) / np.maximum(np.abs(Pe), 1.0)
    print(f"[stages] mixed={mixed} Np={npart}: {items} items, {rej} exact, {runs:.1f} runs and "
          f"{sum(mix[:6]) / (items - rej):.0f} bins per item, largest error {r.max():.2e}", flush=True)
    assert np.all(r <= bar), float(r.max())
    return items, rej, runs, sum(mix[:6]) / (items - rej)


def test_items_of_two_tiles_fp64(torch_cuda):
    from paper_2407_10797_amd import fstat
    T = 7.89e7                                   # nearly all of the band is above 62.5 mHz
    g = S.Grid(T_obs=T, df=1.0 / T, k_lo=int(0.0624 * T), nbins=870_001)
    psd = S.psd_tdix(g.freqs())
    plan = fstat.Plan(S.noise(psd, g.df, 9960), psd, g.T_obs, g.df, g.k_lo)
    box = np.array([[0.2 * g.T_obs, 0.99 * g.T_obs], [10.0, 50.0], [0.0, 0.9], [0.0, np.pi],
                    [0.0, 2 * np.pi], [0.0, 0.1]])
    try:
        for npart in (1, 3):
            _, _, runs, bins = _compare(plan, torch_cuda.from_numpy(S.uniform_box(box, 12, 9961)), npart,
                                        False, 5e-10)
            assert runs > 55.0 and bins > 2560.0         # the per-bin loop, above its stage
    finally:
        plan.close()


def test_tiles_above_the_stage_mixed(torch_cuda, tmp_path):
    from paper_2407_10797_amd import fstat
    T = 2.2e6
    g = S.Grid(T_obs=T, df=1.0 / T, k_lo=22000, nbins=390_001)
    psd = S.psd_tdix(g.freqs())
    rng = np.random.default_rng(9971)
    n = 16
    prm = np.zeros((n, 6))
    prm[:, 0] = 3.0 * T * (1.0 + 0.1 * rng.random(n))
    # Newtonian chirps that start at 30 mHz: supports of some 10,000 bins
    prm[:, 1] = ((5.0 / (256.0 * prm[:, 0])) ** 0.375 / (np.pi * 0.03)) ** 1.6 / MSUN_S
    prm[:, 2] = 0.1
    prm[:, 3] = np.arccos(rng.uniform(-1.0, 1.0, n))
    prm[:, 4] = rng.uniform(0.0, 2.0 * np.pi, n)
    prm[:, 5] = 0.01 * rng.random(n)
    prm = torch_cuda.from_numpy(prm).cuda()
    old = os.environ.get("FSTAT_TUNE_CACHE")
    cache = tmp_path / "tune.txt"
    os.environ["FSTAT_TUNE_CACHE"] = str(cache)
    plan = fstat.Plan(S.noise(psd, g.df, 9970), psd, g.T_obs, g.df, g.k_lo)
    try:
        one = prm[:1].contiguous()
        plan.autotune(one, 20000, mixed=True, force=True)
        key = cache.read_text().splitlines()[-1].split("|")[0]
        with open(cache, "a") as f:
            f.write(key.replace(" np32768 ", " np65536 ") + "|5120 1 0\n")
        assert plan.autotune(one, 65536, mixed=True) == (5120, 1, -1.0)
        items, rej, runs, _ = _compare(plan, prm, 1, True, 1e-4)
        # three items per particle: the middle one is a whole tile
        assert items == 3 * n and rej < n and runs > 55.0
    finally:
        plan.close()
        del os.environ["FSTAT_TUNE_CACHE"]
        if old is not None:
            os.environ["FSTAT_TUNE_CACHE"] = old
