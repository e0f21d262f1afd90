"""Gaussian targets of two coordinates above one workgroup's size, against the oracle:
every place the proposal goes to, whole and ragged wavefronts, and arrays that are
not 16-byte aligned."""
import numpy as np
import pytest

import oracle as O
from paper_1905_10252_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def smc(dev):
    from paper_1905_10252_amd import smc as S
    return S


def bits(a):
    return np.ascontiguousarray(a).view(np.uint64)


def pair(smc, dev, n, d, mode, seed=31, **kw):
    rng = np.random.default_rng(d)
    mean, var = rng.standard_normal(d).tolist(), rng.uniform(0.5, 2.0, d).tolist()
    args = dict(seed=seed, rw_sd=0.4, init_mean=0.3, init_sd=2.5, mean=mean, var=var, mode=mode,
                log_norm=I.gauss_log_norm(var), init_log_norm=I.iso_gauss_log_norm(d, 2.5))
    g = smc.Sampler(n, d, "gauss", device=dev, **args, **kw)
    o = O.Sampler(n, d, O.T_GAUSS, **args)
    o.init()
    return g, o


def run_against(g, o, steps):
    assert np.array_equal(bits(g.x.cpu().numpy()), bits(o.x))
    for t in range(1, steps + 1):
        g.step()
        out, info = o.step(), g.info()
        for k in ("S", "U", "Q2_hi", "Q2_lo", "K", "resampled", "err"):
            assert info[k] == out["info"][k], (t, k)
        g.sync_weights()
        assert np.array_equal(bits(g.x.cpu().numpy()), bits(o.x)), t
        assert np.array_equal(bits(g.logw.cpu().numpy()), bits(o.logw)), t
        e = g.estimates()
        # FP64 sums of positive weights in another order: n roundings at the very most
        tol = max(1e-12, g.n * 2.0 ** -53)
        for k in ("mean", "m2", "rec_mean", "rec_m2"):
            err = np.abs(np.asarray(e[k]) - np.asarray(out[k])) / np.maximum(1.0, np.abs(out[k]))
            assert err.max() <= 10 * tol, (t, k, err.max())
    assert g.sync_error() == 0


@pytest.mark.parametrize("n", [2049, 2111, 131072, 600001])
@pytest.mark.parametrize("mode", [O.MODE_AUTO, O.MODE_FORCE, O.MODE_NEVER])
@pytest.mark.parametrize("lazy", [False, True])
def test_two_coordinates(smc, dev, n, mode, lazy):
    print("two coordinates", n, mode, lazy, flush=True)
    run_against(*pair(smc, dev, n, 2, mode, lazy_reset=lazy), 3)


@pytest.mark.parametrize("mode", [O.MODE_AUTO, O.MODE_FORCE, O.MODE_NEVER])
def test_two_coordinates_unaligned_rows(smc, dev, mode):
    import torch
    n = 5003
    g, o = pair(smc, dev, n, 2, mode)
    buf = torch.empty(2 * n + 1, dtype=torch.float64, device=dev)
    buf[1:] = g.x.reshape(-1)
    g.x = buf[1:].view(n, 2)
    assert g.x.data_ptr() % 16 == 8
    run_against(g, o, 4)
