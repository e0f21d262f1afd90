"""Sizes at which the kernels change shape: tile and segment edges, the limits
of the one-workgroup kernels, row widths, chunk remainders, MFMA k-steps.

Particles, weights, copies and decisions are integer-exact or fixed IEEE
sequences and must match the oracle bit for bit; sums are FP64 in another order.
"""
import math

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


def same(a, b):
    """Bit-equal, NaN where NaN."""
    a, b = np.ascontiguousarray(a), np.ascontiguousarray(b)
    return np.array_equal(bits(np.where(np.isnan(a), 0.0, a)),
                          bits(np.where(np.isnan(b), 0.0, b))) and \
        np.array_equal(np.isnan(a), np.isnan(b))


def close(a, b, rtol):
    a, b = np.asarray(a, float), np.asarray(b, float)
    return np.max(np.abs(a - b) / np.maximum(np.abs(b), 1.0)) <= rtol


EXACT = ("S", "U", "Q2_hi", "Q2_lo", "K", "resampled", "err")


# ------------------------------------------------------------- resampling
def weights(kind, n, seed):
    if kind == "equal":
        return np.zeros(n)
    if kind == "one":
        lw = np.full(n, -np.inf)
        lw[n // 2] = 3.0
        return lw
    return I.logw_normal(n, float(kind), seed)


# one launch up to 6144 weights (four, then eight a thread), the separate passes above;
# tiles of 1024 weights below 2^20, of 4096 from there on
@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 2047, 4095, 4096, 4097, 6143, 6144, 6145,
                               8192,
                               (1 << 20) - 1, 1 << 20])
@pytest.mark.parametrize("kind", ["equal", "one", "0.7", "8"])
def test_resample_size_edges(smc, dev, n, kind):
    import torch
    print("resample", n, kind, flush=True)
    lw = weights(kind, n, 40 + n % 1000)
    tl = torch.from_numpy(lw).to(dev)
    for mode in (O.MODE_FORCE, O.MODE_AUTO):
        for r in (0, (1 << 64) - 1, I.offset_word(n)):  # r = 0, equal weights: whole quotients
            onc, oinfo = O.resample(lw, r, mode)
            R = smc.Resampler(n, device=dev)
            nc = R.resample(tl, r, mode, ncopies=torch.full((n,), -7, dtype=torch.int64,
                                                            device=dev))
            info = R.info()
            for k in EXACT:
                assert info[k] == oinfo[k], (k, mode, r)
            assert abs(info["logZ"] - oinfo["logZ"]) <= 1e-12 * max(1.0, abs(oinfo["logZ"]))
            assert np.array_equal(nc.cpu().numpy(), onc), (mode, r)
            x = torch.arange(n, dtype=torch.float64, device=dev).reshape(n, 1)
            assert np.array_equal(R.redistribute(x).cpu().numpy()[:, 0],
                                  np.repeat(np.arange(n), onc))
            if n <= 1 << 20:
                na = torch.full((n,), -7, dtype=torch.int64, device=dev)
                smc.resample_noalloc(tl, r, na, mode)
                assert np.array_equal(na.cpu().numpy(), onc), ("noalloc", mode, r)


# rows of 4 w bytes at an address `off` values past a 16-byte boundary; the
# populations take segments of 256, 512, 1024 and 2048 merge steps
@pytest.mark.parametrize("n", [1, 255, 262144, 262145, 524289, 1048577])
@pytest.mark.parametrize("w,off", [(1, 0), (2, 1), (4, 1), (5, 0), (7, 3), (8, 2), (9, 0), (11, 1),
                                   (16, 0), (33, 0)])
def test_redistribute_row_edges(smc, dev, n, w, off):
    import torch
    print("rows", n, w, off, flush=True)
    rng = np.random.default_rng(n + w)
    nc = np.bincount(rng.integers(0, n, n) ** 2 // n, minlength=n).astype(np.int64)
    buf = torch.from_numpy(rng.integers(0, 1 << 31, n * w + 4, dtype=np.int32)).to(dev)
    out = torch.full((n * w + 8,), -1, dtype=torch.int32, device=dev)
    x, xo = buf[off:off + n * w].view(n, w), out[off:off + n * w].view(n, w)
    R = smc.Resampler(n, device=dev)
    R.redistribute(x, xo, ncopies=torch.from_numpy(nc).to(dev))
    assert R.sync_error() == 0
    want = np.repeat(x.cpu().numpy(), nc, axis=0)
    assert np.array_equal(xo.cpu().numpy(), want)
    got = out.cpu().numpy()  # nothing outside the rows
    assert (got[:off] == -1).all() and (got[off + n * w:] == -1).all()


# --------------------------------------------------------------- samplers
def gauss_pair(smc, dev, n, d, mode, seed=23):
    rng = np.random.default_rng(1000 * d + n % 997)
    mean, var = rng.standard_normal(d), rng.uniform(0.5, 2.0, d)
    ln, iln = I.gauss_log_norm(var), I.iso_gauss_log_norm(d, 3.0)
    kw = dict(seed=seed, rw_sd=0.4, init_mean=0.0, init_sd=3.0, mean=mean, var=var, mode=mode,
              log_norm=ln, init_log_norm=iln)
    g = smc.Sampler(n, d, "gauss", device=dev, **kw)
    o = O.Sampler(n, d, O.T_GAUSS, **kw)
    o.init()
    return g, o


def run_against(g, o, steps):
    for t in range(1, steps + 1):
        g.step()
        out = o.step()
        info = g.info()
        for k in EXACT:
            assert info[k] == out["info"][k], (t, k)
        assert np.array_equal(bits(g.x.cpu().numpy()), bits(o.x)), t
        assert np.array_equal(bits(g.logw.cpu().numpy()), bits(o.logw)), t
        e = g.estimates()
        assert close(e["mean"], out["mean"], 1e-11) and close(e["m2"], out["m2"], 1e-11), t
        assert close(e["rec_mean"], out["rec_mean"], 1e-10), t


# one workgroup: wavefronts of 128 particles, then the lines of its rule by d
SMALL = [(1, 1), (127, 1), (128, 2), (129, 3), (1025, 1), (2048, 1), (2048, 2), (2047, 2),
         (1536, 3), (1537, 3), (1536, 4), (1537, 4), (2, 5), (1023, 5), (1024, 6), (1025, 6),
         (512, 7), (513, 7), (512, 8), (513, 8), (64, 9)]


@pytest.mark.parametrize("n,d", SMALL)
@pytest.mark.parametrize("mode", [O.MODE_AUTO, O.MODE_FORCE, O.MODE_NEVER])
def test_small_population_edges(smc, dev, n, d, mode):
    print("small", n, d, mode, flush=True)
    run_against(*gauss_pair(smc, dev, n, d, mode), 4)


# rows in LDS: 256, 128, 64 or 32 particles a workgroup by d and n
ROWS = [(2049, 2), (16385, 3), (131072, 2), (131073, 11), (70001, 12), (65537, 23), (40000, 24),
        (32769, 47), (20011, 63), (16385, 64)]


@pytest.mark.parametrize("n,d", ROWS)
@pytest.mark.parametrize("mode", [O.MODE_AUTO, O.MODE_FORCE, O.MODE_NEVER])
def test_row_update_edges(smc, dev, n, d, mode):
    print("rows", n, d, mode, flush=True)
    run_against(*gauss_pair(smc, dev, n, d, mode), 2)


# batched proposals: 64-row chunks, one coordinate (rows of two), odd and even rows
@pytest.mark.parametrize("mode", [O.MODE_AUTO, O.MODE_FORCE])
def test_batch_row_edges(smc, dev, mode):
    sizes = [(n, d) for d in (1, 2, 3, 7, 8, 63, 64) for n in (1, 2, 63, 65, 257)]
    B = smc.Batch(len(sizes), device=dev)
    orc = []
    for k, (n, d) in enumerate(sizes):
        mean, U, _ = I.wishart_target(d, np.random.default_rng(900 + k))
        B.attach(k, n, d, mean, U, seed=(9 << 32) + k, sampler_id=k, rw_sd=0.5 / math.sqrt(d),
                 mode=mode)
        desc = B.slots[k]["desc"]
        o = O.Sampler(n, d, O.T_GAUSS_CHOL, seed=(9 << 32) + k, sampler_id=k,
                      rw_sd=0.5 / math.sqrt(d), init_mean=0.0, init_sd=3.0, mean=mean, chol=U,
                      mode=mode, log_norm=desc.log_norm, init_log_norm=desc.init_log_norm)
        o.init()
        orc.append(o)
    for t in range(1, 4):
        B.step()
        for k, o in enumerate(orc):
            out = o.step()
            assert B.info(k)["S"] == out["info"]["S"], (t, sizes[k])
            assert np.array_equal(bits(B.x(k).cpu().numpy()), bits(o.x)), (t, sizes[k])
            assert np.array_equal(bits(B.logw(k).cpu().numpy()), bits(o.logw)), (t, sizes[k])


# ---------------------------------------------------- the filter's fused step
def filter_pair(smc, dev, n, mode, obs, lazy):
    B = I.BEARING
    kw = dict(seed=5, mean=B["x0"], init_sd=B["init_sd"], obs=obs, delta=B["delta"],
              obs_var=B["obs_var"], mode=mode, device=dev, lazy_reset=lazy)
    return [smc.Sampler(n, 4, "bearing", **kw) for _ in range(2)]


# segments of 256 to 2048 merge steps; an odd and an even number of iterations (the
# rows start in place or in the copy); a call after one that left uniform weights
@pytest.mark.parametrize("n", [1, 2, 257, 2049, 131075, 262144, 524287, 1048576, 2100000])
@pytest.mark.parametrize("mode,lazy", [(O.MODE_AUTO, False), (O.MODE_FORCE, True),
                                       (O.MODE_NEVER, False)])
def test_filter_steps_equal_single_steps(smc, dev, n, mode, lazy):
    print("filter", n, mode, lazy, flush=True)
    _, ys = I.bearing_track(9, 7)
    a, b = filter_pair(smc, dev, n, mode, ys, lazy)
    for k in (3, 2, 4):
        got = a.steps(k, info=True, est=True)
        for i in range(k):
            b.step()
            info = b.info()
            for f in EXACT:
                assert got["info"][i][f] == info[f], (k, i, f)
            assert got["info"][i]["log_c"] == info["log_c"], (k, i)
            assert np.array_equal(bits(got["est"][i].cpu().numpy()),
                                  bits(b.est.cpu().numpy())), (k, i)
        assert np.array_equal(bits(a.x.cpu().numpy()), bits(b.x.cpu().numpy())), k
        for s in (a, b):
            s.sync_weights()
        assert np.array_equal(bits(a.logw.cpu().numpy()), bits(b.logw.cpu().numpy())), k


@pytest.mark.parametrize("n", [300, 200001])
def test_filter_steps_with_a_failed_iteration(smc, dev, n):
    _, ys = I.bearing_track(5, 7)
    ys = ys.copy()
    ys[2] = np.nan
    a, b = filter_pair(smc, dev, n, O.MODE_AUTO, ys, False)
    got = a.steps(5, info=True)
    errs = []
    for i in range(5):
        b.step()
        errs.append(b.info()["err"])
        assert got["info"][i]["err"] == errs[-1], i
    assert errs[1] == 0 and errs[2] != 0
    assert same(a.x.cpu().numpy(), b.x.cpu().numpy())
    assert same(a.logw.cpu().numpy(), b.logw.cpu().numpy())
    assert a.sync_error() == b.sync_error() != 0


# ------------------------------------------------------ FP64 likelihood
def softplus_sum(X, y, th):
    """sum_m softplus((1 - 2 y_m) x_m . theta), in extended precision."""
    u = (X.astype(np.longdouble) * (1 - 2 * y.astype(np.longdouble))[:, None]) @ \
        th.astype(np.longdouble).T
    return (np.maximum(u, 0) + np.log1p(np.exp(-np.abs(u)))).sum(0)


# every operand width (1, 2, 4, ... 16 k-steps), tiles of 16 rows, the 512 factors
# of a logarithm, particles of 16 and 64
@pytest.mark.parametrize("d", [1, 4, 5, 8, 9, 16, 17, 24, 25, 33, 41, 49, 57, 64])
@pytest.mark.parametrize("m_rows", [1, 15, 16, 2049])
def test_logreg_f64_operand_widths(smc, dev, d, m_rows):
    import torch
    rng = np.random.default_rng(d + m_rows)
    X, y, _ = I.logreg_data(m_rows, d, 7 + d)
    ln = I.iso_gauss_log_norm(d, math.sqrt(10.0))
    g = smc.Sampler(70, d, "logreg", X=X.astype(np.float64), y=y, prior_var=10.0,
                    precision="f64", log_norm=ln, device=dev)
    for n in (1, 16, 65):
        th = rng.standard_normal((n, d))
        lp = g.log_target(torch.from_numpy(th).to(dev)).cpu().numpy()
        want = ln - 0.05 * (th.astype(np.longdouble) ** 2).sum(1) - softplus_sum(X, y, th)
        # d + 2 roundings a term, then M additions of sums of its size
        mag = 1.0 + np.abs(X.astype(np.float64) @ th.T).sum(0)
        bound = 2.0 ** -53 * (m_rows + 4 * d + 16) * (mag + np.abs(want).astype(np.float64))
        assert (np.abs(lp - want.astype(np.float64)) <= bound).all(), (d, m_rows, n)


def test_logreg_f64_single_terms(smc, dev):
    """One row, one feature: softplus over the range of its exponential, the table's
    grid points and its clamp included."""
    import torch
    u = np.concatenate([np.linspace(-60, 60, 4001), np.geomspace(1e-320, 1e308, 3000),
                        -np.geomspace(1e-320, 1e5, 3000), np.arange(4096) * math.log(2) / 2048,
                        (np.arange(4096) + 0.5) * math.log(2) / 2048, [0.0, -0.0, 699.999,
                                                                       700.0, 700.001, 745.2]])
    # a wide prior keeps the quadratic term small; its part is taken out exactly
    g = smc.Sampler(u.size, 1, "logreg", X=np.ones((1, 1)), y=np.zeros(1), prior_var=1e300,
                    precision="f64", log_norm=0.0, device=dev)
    lp = g.log_target(torch.from_numpy(u.reshape(-1, 1)).to(dev)).cpu().numpy()
    ul = u.astype(np.longdouble)
    prior = np.where(np.abs(u) < 1e100, 0.0, 0.5e-300 * ul * ul)
    want = -(np.maximum(ul, 0) + np.log1p(np.exp(-np.abs(ul)))) - prior
    small = np.abs(u) < 1e100
    err = np.abs(lp[small] - want[small].astype(np.float64))
    # (u + |u|) / 2 and the logarithm: a few roundings of values up to |u| + 1
    assert (err <= 2.0 ** -52 * 4 * (1.0 + np.abs(u[small]))).all()
    assert np.isfinite(lp[small]).all()
