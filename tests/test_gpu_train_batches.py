"""Gradients of one training step at the batch sizes where the kernels change:
a last panel of k shorter than the others (192: splits of 96), the largest
batch whose column sums the products form themselves (4096), the first whose
sums are passes of their own (4160, a split of K = 32 by 2) and one with longer
slices (8192).  Bars of the small-batch test: BF16 operands (unit roundoff 2^-9)
through three 256-term layers, outputs within 1e-2 and every parameter group's
gradient within 3e-2 of FP64 (norm-wise)."""
import numpy as np
import pytest

from oracle import mlp_oracle as MO

pytestmark = pytest.mark.gpu


def _rel(a, b):
    return float(np.linalg.norm(a - b) / max(np.linalg.norm(b), 1e-30))


@pytest.mark.parametrize("B", [192, 4096, 4160, 8192])
def test_gradients_match_fp64_reference(B):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    from paper_2407_10797_amd import fstat
    rng = np.random.default_rng(B)
    p = MO.init(7).astype(np.float32)
    x = rng.uniform(-1, 1, (B, 3)).astype(np.float32)
    t = (-(1.0 / (1.0 + 0.45 * (x[:, 0] + 1.0))) ** (19.0 / 9.0)).astype(np.float32)
    loss, g, y = fstat.fstat_mlp_grad(p, x, t)
    y_ref, _, _ = MO.forward(p.astype(np.float64), x.astype(np.float64))
    loss_ref, g_ref = MO.loss_and_grad(p.astype(np.float64), x.astype(np.float64),
                                       t.astype(np.float64))
    assert _rel(y, y_ref) < 1e-2
    assert abs(loss - loss_ref) <= 2e-2 * loss_ref
    o = 0
    for name, shape in MO.SIZES:
        n = int(np.prod(shape))
        r = _rel(g[o:o + n], g_ref[o:o + n])
        print(f"[mlp] B={B} grad {name:3s} rel {r:.2e}", flush=True)
        assert r < 3e-2, name
        o += n
