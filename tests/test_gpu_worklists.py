"""Work lists: the one-kernel list (up to 8,192 particles) and the scanned one
above it, the grouping in one block (the three-particle calls) and the counted
one.  A list decides where an item is evaluated, not its sums: the same particles
in a short call and in a long one agree to 1e-9 (rounding of sums in another
order times the partitions' conditioning on this grid)."""
import numpy as np
import pytest

from paper_2407_10797_amd import synth as S

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    return torch


@pytest.mark.parametrize("n, npart", [(8192, 4), (8193, 4), (8193, 1)])
def test_long_lists_match_short_ones(torch_cuda, n, npart):
    from paper_2407_10797_amd import fstat
    T = 6.0e6
    df = 1.0 / T
    k0 = int(np.ceil(0.02 / df))
    g = S.Grid(T_obs=T, df=df, k_lo=k0, nbins=int(np.floor(0.05 / df)) - k0 + 1)
    psd = S.psd_tdix(g.freqs())
    plan = fstat.Plan(S.noise(psd, g.df, 9400), psd, g.T_obs, g.df, g.k_lo)
    box = np.array([[1.6 * T, 3.0 * T], [25.0, 40.0], [0.0, 0.9], [0.0, np.pi], [0.0, 2 * np.pi],
                    [0.0, 0.1]])
    prm = torch_cuda.from_numpy(S.uniform_box(box, n, 9401))
    try:
        print(f"[lists] n={n} Np={npart}", flush=True)
        for mixed in (False, True):
            F = plan.eval(prm, npart, mixed=mixed)
            for i in (0, n // 2, n - 3):
                Fs = plan.eval(prm[i:i + 3].contiguous(), npart, mixed=mixed)
                np.testing.assert_allclose(F[i:i + 3].cpu().numpy(), Fs.cpu().numpy(), rtol=1e-9)
    finally:
        plan.close()
