"""The block loop (items evaluated from the plan's block spectra) against the
exact template at every bin, on grids that give each block length and slope
count: partitions with no, one and many whole blocks, edges inside blocks, a
last block cut by the band's end, a zero-padded grid (T_obs df = 1/2), several
channels, and the work-item sizes that rule the spectra out.  Same budget as
the interpolating loop's own parity test: 5e-10 relative plus 4 eps cond(M_l);
mixed: 1e-4 + 20 2^-24 sqrt(cond M_l)."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2407_10797_amd import synth as S
from tests.bars import FP64_KCOND

MIXED_SQRT_COND = 20.0 * 2.0 ** -24

pytestmark = pytest.mark.gpu

# name: T_obs, df T_obs, band [Hz]; block lengths (FP64, mixed)
GRIDS = {
    "short": (6.0e6, 1.0, 0.02, 0.05),       # 180,001 bins: 32 and 64
    "mid": (1.0e7, 1.0, 0.02, 0.0605),       # 405,001 bins: 64 and 128
    "padded": (1.0e7, 0.5, 0.02, 0.0413),    # 426,001 bins at half the spacing: 64 and 128
    "long": (4.0e7, 1.0, 0.018, 0.06),       # 1,680,001 bins: 128 and 256
}


@pytest.fixture(scope="module")
def torch_cuda():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    return torch


def _case(name, n=8):
    T, tdf, f0, f1 = GRIDS[name]
    df = tdf / T
    k0 = int(np.ceil(f0 / df))
    g = S.Grid(T_obs=T, df=df, k_lo=k0, nbins=int(np.floor(f1 / df)) - k0 + 1)
    box = np.array([[1.6 * T, 3.0 * T], [25.0, 40.0], [0.0, 0.9], [0.0, np.pi], [0.0, 2 * np.pi],
                    [0.0, 0.1]])
    if name == "long":
        box[0] = [1.2 * T, 2.0 * T]
    pts = S.uniform_box(box, n, 9100)
    # the last particle leaves through the band's upper end: its last bins lie
    # in the block that the band's end cuts
    pts[-1, 0] = 1.02 * T
    return g, pts


def _rel(a, b):
    return np.abs(a - b) / np.maximum(np.abs(b), 1.0)


@pytest.mark.parametrize("chunk", [0, 256, 1000])
@pytest.mark.parametrize("name", list(GRIDS))
def test_block_loop_matches_exact(torch_cuda, name, chunk):
    from paper_2407_10797_amd import fstat
    g, pts = _case(name)
    psd = S.psd_tdix(g.freqs())
    data = S.noise(psd, g.df, 9200)
    plan = fstat.Plan(data, psd, g.T_obs, g.df, g.k_lo, chunk=chunk)
    prm = torch_cuda.from_numpy(pts)
    try:
        for npart in (1, 37, 700) if chunk == 0 else (37,):
            print(f"[blocks] {name} chunk={chunk} Np={npart}, {g.nbins} bins", flush=True)
            F, P = plan.eval(prm, npart, want_parts=True)
            items, rej, ref, mix = plan.interp_stats(bin_mix=True)
            Fm, Pm = plan.eval(prm, npart, mixed=True, want_parts=True)
            Fe, Pe = plan.eval(prm, npart, want_parts=True, exact=True)
            P, Pm, Pe = (t.cpu().numpy() for t in (P, Pm, Pe))
            _, Po, cond = O.fstat(data, psd, g.k_lo, g.df, g.T_obs, pts, [npart], want_cond=True)
            c = np.where(np.isfinite(cond), cond, 0.0)
            r, rm = _rel(P, Pe), _rel(Pm, Pe)
            print(f"  {items} items, {rej} exact, {ref} refined, smooth bins {sum(mix[3:6])}, "
                  f"direct {sum(mix[:3])}; fp64 {r.max():.2e}, mixed {rm.max():.2e}, cond "
                  f"{c.max():.1e}", flush=True)
            if npart < 100:
                assert sum(mix[3:6]) > 0.5 * sum(mix[:7])
            assert np.all(r <= 5e-10 + FP64_KCOND * c), float(r.max())
            assert np.all(rm <= 1e-4 + MIXED_SQRT_COND * np.sqrt(c)), float(rm.max())
    finally:
        plan.close()


def test_block_loop_channels_and_orders(torch_cuda):
    """Three channels (each with its own spectra), particles in another order and
    a batch of one: the same values bit for bit as in the full batch."""
    from paper_2407_10797_amd import fstat
    g, pts = _case("mid", 12)
    psd = np.array([S.psd_channel(g.freqs(), c) for c in "AET"])
    data = np.array([S.noise(psd[i], g.df, 9300 + i) for i in range(3)])
    plan = fstat.Plan(data, psd, g.T_obs, g.df, g.k_lo, channels="AET")
    try:
        prm = torch_cuda.from_numpy(pts)
        for mixed in (False, True):
            print(f"[blocks] A, E, T, mixed={mixed}", flush=True)
            F, P = plan.eval(prm, 16, want_parts=True, mixed=mixed)
            Fe, Pe = plan.eval(prm, 16, want_parts=True, exact=True)
            P, Pe = P.cpu().numpy(), Pe.cpu().numpy()
            assert np.all(_rel(P, Pe) <= (1e-4 if mixed else 5e-10))
            perm = np.arange(len(pts))[::-1].copy()
            Pr = plan.eval(torch_cuda.from_numpy(pts[perm]), 16, want_parts=True, mixed=mixed)[1]
            np.testing.assert_array_equal(Pr.cpu().numpy(), P[perm])
            P1 = plan.eval(torch_cuda.from_numpy(pts[3:4]), 16, want_parts=True, mixed=mixed)[1]
            np.testing.assert_array_equal(P1.cpu().numpy(), P[3:4])
    finally:
        plan.close()
