"""The score fit at bandwidths whose square or cube leaves the range of a
double: only coincident neighbours keep a weight, and nothing turns to NaN.
Tolerances as in test_gpu_fit.py (the same FP64 terms in another order)."""
import numpy as np
import pytest

from paper_2512_10386_amd import synth

pytestmark = pytest.mark.gpu

PRM = dict(k=16, leaf_cap=512)


@pytest.mark.parametrize("copies", [0, 3])
@pytest.mark.parametrize("sigma", [1e-60, 1e-104, 1e-120, 1e-155, 1e-160, 1e-300, 5e-324, 1e104, 1e160, 1e300])
def test_fit_at_extreme_bandwidths(oracle, copies, sigma):
    import torch
    from paper_2512_10386_amd.fit import ScoreFit
    xyz, lab = synth.torus_bumpy(31, 0.01, n_torus=1500, n_bumpy=1500, n_out=300)
    if copies:  # points with neighbours at distance 0
        xyz, lab = np.concatenate([xyz] + [xyz[:400]] * copies), np.concatenate([lab] + [lab[:400]] * copies)
    f = ScoreFit(torch.from_numpy(xyz).cuda(), torch.from_numpy(lab).cuda(), temperature=0.7, **PRM)
    try:
        got = f.loss_grad(1.0, sigma, 2.0, 3.0).cpu().numpy()
    finally:
        f.close()
    ref = oracle.denoise(xyz, **PRM)
    exp = oracle.fit_loss_grad(xyz, ref, lab, 1.0, sigma, 2.0, 3.0, 0.7)
    assert np.isfinite(exp).all()
    assert (exp[5] > 0) == (copies > 0 or sigma > 1)
    assert got[5] == exp[5]
    for c in range(5):
        assert abs(got[c] - exp[c]) <= 1e-9 * abs(exp[c]) + 1e-12, (c, got[c], exp[c])
