"""Which loop takes the items: plans of the block loop's grids have their block
spectra (an item is sixteen lanes' work there, up to 64 in the per-bin loop), item
sizes that are no multiple of a block rule them out, and a plan made while the
device is nearly full has none, says so, and gives the same statistic bin by bin
(5e-10 relative FP64, 1e-4 mixed, the block loop's bars)."""
import warnings

import numpy as np
import pytest

from paper_2407_10797_amd import synth as S
from tests.test_gpu_blocks import GRIDS, _case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("chunk", [0, 256, 1000])
@pytest.mark.parametrize("name", list(GRIDS))
def test_block_loop_takes_the_items(name, chunk):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2407_10797_amd import fstat
    g, pts = _case(name)
    psd = S.psd_tdix(g.freqs())
    plan = fstat.Plan(S.noise(psd, g.df, 9200), psd, g.T_obs, g.df, g.k_lo, chunk=chunk)
    try:
        for mixed in (False, True):
            plan.eval(torch.from_numpy(pts), 1, mixed=mixed)
            items, rej, _, mix = plan.interp_stats(bin_mix=True)
            runs = sum(mix[7:13]) / (items - rej)
            print(f"[loops] {name} chunk={chunk} mixed={mixed}: {runs:.1f} runs per item", flush=True)
            # the last particle's short items may be the per-bin loop's
            assert runs > 40.0 if chunk == 1000 else 15.9 < runs < 24.0
    finally:
        plan.close()


def test_plan_without_room_for_spectra():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2407_10797_amd import fstat
    g = S.grid_paper()
    f = g.freqs()
    psd = np.array([S.psd_channel(f, c) for c in "AET"])
    data = torch.from_numpy(np.array([S.noise(psd[i], g.df, 9900 + i) for i in range(3)])).cuda()
    psd = torch.from_numpy(psd).cuda()
    prm = torch.from_numpy(S.uniform_box(S.PAPER_BOX, 6, 9903)).cuda()

    def plan_and_values():
        plan = fstat.Plan(data, psd, g.T_obs, g.df, g.k_lo, channels="AET")
        out = []
        try:
            for mixed in (False, True):
                P = plan.eval(prm, 16, want_parts=True, mixed=mixed)[1].cpu().numpy()
                items, rej, _, mix = plan.interp_stats(bin_mix=True)
                out.append((P, sum(mix[7:13]) / (items - rej)))     # runs per item
        finally:
            plan.close()
        return out

    with warnings.catch_warnings():
        warnings.simplefilter("error")
        full = plan_and_values()
    torch.cuda.empty_cache()
    # 13.6 GB of spectra need 54 GB free
    hold = torch.empty(max(torch.cuda.mem_get_info()[0] - 40 * 10 ** 9, 1), dtype=torch.uint8,
                       device="cuda")
    try:
        print(f"[memory] {torch.cuda.mem_get_info()[0] / 1e9:.1f} GB free", flush=True)
        with pytest.warns(RuntimeWarning, match="no block spectra"):
            bare = plan_and_values()
    finally:
        del hold
        torch.cuda.empty_cache()
    for (P, runs), (Pb, runs_b), bar in zip(full, bare, (5e-10, 1e-4)):
        assert 15.9 < runs < 17.0           # sixteen lanes per item: the block loop
        assert runs_b > 40.0                # up to 64: the per-bin loop
        r = np.abs(P - Pb) / np.maximum(np.abs(Pb), 1.0)
        print(f"[memory] with and without: {r.max():.2e}", flush=True)
        assert np.all(r <= bar), float(r.max())
