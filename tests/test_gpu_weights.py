"""smc_normalised_weights on an array that is not the one of the last decision."""
import numpy as np
import pytest

import oracle as O

pytestmark = pytest.mark.gpu


def test_weights_of_another_array(dev):
    """exp(l_i - m) / Z with m and Z of the last resample: 0 at the low end, +inf above the
    exponential's range, NaN for a NaN."""
    import torch
    from paper_1905_10252_amd import smc
    print("weights of another array", flush=True)
    n = 1000
    R = smc.Resampler(n)
    lw = torch.linspace(-3.0, 0.5, n, dtype=torch.float64, device=dev)
    R.resample(lw, 1, O.MODE_FORCE)
    info = R.info()
    ends = np.array([-np.inf, -1e300, -746.5, -745.0, -1.0, 0.0, 1.0, 700.0, 709.0, 709.5, 710.0,
                     800.0, 1e9, 1e300, np.inf, np.nan])
    v = np.resize(ends, n)
    got = R.normalised_weights(torch.from_numpy(v + info["m"]).to(dev)).cpu().numpy()
    l = O.lib()
    want = np.array([l.orc_det_exp(float(a)) for a in (v + info["m"]) - info["m"]]) / info["Z"]
    assert np.array_equal(np.isnan(got), np.isnan(want)) and np.isnan(got).any()
    ok = ~np.isnan(want)
    assert np.array_equal(got[ok], want[ok])
