"""Block spectra by transforms (blocks of 256 bins, 512 slopes): plans of 6.3 million
bins whose slopes end at half a cycle, one cycle and just above one cycle per bin
(rows 257, 513 and 514 of a 512-point transform), with and without the FP32 table,
against the exact template at every bin.  Bars of the block loop's parity test:
5e-10 relative FP64, 1e-4 mixed."""
import numpy as np
import pytest

from paper_2407_10797_amd import synth as S

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tdf, precision", [(1.0, "both"), (0.5, "both"), (1.001, "both"),
                                            (1.0, "fp64")])
def test_transform_spectra_match_exact(tdf, precision):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2407_10797_amd import fstat
    nbins, df = 6_300_077, 1.0e-8
    T = tdf / df
    g = S.Grid(T_obs=T, df=df, k_lo=int(np.ceil(0.018 / df)), nbins=nbins)
    psd = S.psd_tdix(g.freqs())
    kw = {} if precision == "both" else {"precision": fstat.FSTAT_FP64}
    plan = fstat.Plan(S.noise(psd, g.df, 9500), psd, g.T_obs, g.df, g.k_lo, **kw)
    box = np.array([[1.02 * T, 1.3 * T], [12.0, 45.0], [0.0, 0.9], [0.0, np.pi], [0.0, 2 * np.pi],
                    [0.0, 0.1]])
    prm = torch.from_numpy(S.uniform_box(box, 6, 9501))
    try:
        for npart in (1, 16):
            print(f"[fft] T df = {tdf}, {precision}, Np={npart}", flush=True)
            Pe = plan.eval(prm, npart, want_parts=True, exact=True)[1].cpu().numpy()
            for mixed in (False, True)[:1 if precision == "fp64" else 2]:
                P = plan.eval(prm, npart, want_parts=True, mixed=mixed)[1].cpu().numpy()
                mix = plan.interp_stats(bin_mix=True)[3]
                assert sum(mix[3:6]) > 0.5 * sum(mix[:7])
                r = np.abs(P - Pe) / np.maximum(np.abs(Pe), 1.0)
                assert np.all(r <= (1e-4 if mixed else 5e-10)), float(r.max())
    finally:
        plan.close()
