"""Rows at the ends of the redistribution's segments, for the populations that are
written past the caches: the rows past a segment's last whole round of loads take
another route than the others, one of three by the population's size."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def smc():
    from paper_1905_10252_amd import smc
    return smc


@pytest.mark.parametrize("n,row_bytes", [
    ((1 << 20) + 37, 128),     # whole 16-byte chunks, a power of two a row
    (1398101 + 2, 96),         # six chunks a row
    ((1 << 22) + 1, 32),       # two chunks a row
    ((13 << 20) - 1, 32),      # last size of the cached ends, first of the next route
    (13 << 20, 32),
    ((13 << 20) + 7, 48),
    ((1 << 24) + 3, 8),        # 8-byte rows
    ((1 << 25) - 1, 16),       # last size of that route, first of the third
    (1 << 25, 16),
    ((1 << 25) + 5, 16),
])
@pytest.mark.parametrize("s", [0.5, 2.0, 8.0])
def test_streamed_rows(smc, dev, n, row_bytes, s):
    check(smc, dev, n, row_bytes, s, False)


# counts and ancestors written too: three times the bytes, so the lines lie at a third of
# the populations
@pytest.mark.parametrize("n,row_bytes", [((1 << 22) + 3, 32), ((13 << 20) // 3, 48),
                                         ((13 << 20) // 3 + 1, 48), ((1 << 25) // 3, 16),
                                         ((1 << 25) // 3 + 1, 16)])
@pytest.mark.parametrize("s", [0.5, 8.0])
def test_streamed_rows_with_counts_and_ancestors(smc, dev, n, row_bytes, s):
    check(smc, dev, n, row_bytes, s, True)


def check(smc, dev, n, row_bytes, s, outputs):
    import torch
    print("streamed rows", n, row_bytes, s, outputs, flush=True)
    g = torch.Generator(device=dev).manual_seed(n + row_bytes)
    logw = s * torch.randn(n, generator=g, device=dev, dtype=torch.float64)
    x = torch.randint(-2**31, 2**31 - 1, (n, row_bytes // 4), generator=g, device=dev,
                      dtype=torch.int32)
    R = smc.Resampler(n)
    nc = torch.empty(n, dtype=torch.int64, device=dev)
    R.resample(logw, 0x9E3779B97F4A7C15, smc.L.MODE_FORCE, ncopies=nc)
    nco = torch.empty_like(nc) if outputs else None
    anc = torch.empty_like(nc) if outputs else None
    got = R.redistribute(x, ncopies_out=nco, anc=anc)
    assert R.sync_error() == 0
    if outputs:
        assert torch.equal(nco, nc)
        assert torch.equal(anc, torch.arange(n, device=dev).repeat_interleave(nc))
    assert int(nc.sum()) == n and int(nc.min()) >= 0
    assert torch.equal(got, x.repeat_interleave(nc, 0))
