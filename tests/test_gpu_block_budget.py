"""The refinement budget where the block loop's own error is largest: high
frequencies over a long observation in a narrow band, so that the block spectra
have few slopes (Q = 64 and 128) and a bin's grid rounding turns its phase most.
The refined statistic is within the plan's budget, plus 4 eps cond(M_l), of the
exact template at every bin, at a budget below that error and at the default."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2407_10797_amd import synth as S
from tests.bars import FP64_KCOND

pytestmark = pytest.mark.gpu


# band [Hz], particles, budget (0: the default, 5e-10), loops: 370,831 bins (Q = 64) and
# 789,001 (Q = 128); the last band crosses 62.5 mHz, where the default budget's block
# loop ends at Q = 128
@pytest.mark.parametrize("f0, f1, n, budget, loops",
                         [(0.09, 0.1, 32, 5e-12, "bins"), (0.0953, 0.1, 8, 0.0, "bins"),
                          (0.0575, 0.0675, 12, 0.0, "both")])
def test_block_loop_errors_are_in_the_estimate(f0, f1, n, budget, loops):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2407_10797_amd import fstat
    g = S.grid_custom(7.89e7, f0, f1)
    psd = S.psd_tdix(g.freqs())
    data = S.noise(psd, g.df, 9600)
    box = np.array([[0.2 * g.T_obs, 0.99 * g.T_obs], [10.0, 50.0], [0.0, 0.9], [0.0, np.pi],
                    [0.0, 2 * np.pi], [0.0, 0.1]])
    pts = S.uniform_box(box, n, 9601)
    prm = torch.from_numpy(pts)
    plan = fstat.Plan(data, psd, g.T_obs, g.df, g.k_lo, precision=fstat.FSTAT_FP64,
                      refine_budget=budget)
    try:
        for npart in (1, 2, 8):
            print(f"[budget] {g.nbins} bins, budget {budget or 5e-10}, Np={npart}", flush=True)
            P = plan.eval(prm, npart, want_parts=True)[1].cpu().numpy()
            items, rej, ref, mix = plan.interp_stats(bin_mix=True)
            Pe = plan.eval(prm, npart, want_parts=True, exact=True)[1].cpu().numpy()
            cond = O.fstat(data, psd, g.k_lo, g.df, g.T_obs, pts, [npart], want_cond=True)[2]
            c = np.where(np.isfinite(cond), cond, 0.0)
            r = np.abs(P - Pe) / np.maximum(np.abs(Pe), 1.0)
            tol = (budget or 5e-10) + FP64_KCOND * c
            # a block-loop item is sixteen lanes' work, one of the per-bin loop up to 64
            runs = sum(mix[7:13]) / (items - rej)
            print(f"  {items} items, {rej} exact, {ref} refined, {runs:.1f} runs per item; largest "
                  f"{r.max():.2e}, {(r / tol).max():.2f} of its bar, {(r > tol).sum()} above", flush=True)
            assert np.all(r <= tol), float((r / tol).max())
            assert 30.0 < runs if loops == "bins" else 17.0 < runs < 55.0
    finally:
        plan.close()
