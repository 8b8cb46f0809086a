"""Peakmap cleaning on the GPU against the cleaning oracle (Sec. "Removal of
time and frequency domain disturbances", appendix "Robust statistic"):
integer results and vetoed peakmaps bit-exact, robust statistics equal as
doubles."""
import numpy as np
import pytest

import oracle
from oracle import clean as oclean
from paper_1407_8333_amd import synth
from test_clean_oracle import _wandering_band

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_1407_8333_amd import api
    c = api.Context(0)
    yield c
    c.close()


def _download(dpm):
    import torch
    torch.cuda.synchronize()
    return dpm.download()


def test_gross_histogram_and_veto_match_the_oracle(ctx):
    from paper_1407_8333_amd import clean
    pm, _, _, _ = _wandering_band()
    dpm = ctx.upload(pm)
    for dt_h, df_h in [(6 * 3600.0, 0.01), (3 * 3600.0, 0.037), (1e9, 1.0)]:
        geo = clean.gross_geometry(pm.t, pm.k_lo, pm.k_hi, dt_h, df_h, pm.t_fft)
        assert geo == oclean.gross_geometry(pm.t, pm.k_lo, pm.k_hi, dt_h, df_h, pm.t_fft)
        h = clean.gross_histogram(ctx, dpm, geo).cpu().numpy()
        href = oclean.gross_histogram(pm, *geo)
        np.testing.assert_array_equal(h, href)
        thr = float(np.median(href)) + 12.5
        out, h2 = clean.clean_gross(ctx, dpm, geo, thr)
        off, bins = _download(out)
        roff, rbins = oclean.gross_veto(pm, *geo, thr)
        np.testing.assert_array_equal(h2.cpu().numpy(), href)
        np.testing.assert_array_equal(off, roff)
        np.testing.assert_array_equal(bins, rbins)
        out.release()
    # a histogram that covers only part of the peakmap: peaks outside are kept
    geo = (float(pm.t[10]), 4000.0, 5, 0.02, int(pm.k_lo / (0.02 * pm.t_fft)) + 3, 7)
    np.testing.assert_array_equal(clean.gross_histogram(ctx, dpm, geo).cpu().numpy(),
                                  oclean.gross_histogram(pm, *geo))
    out, _ = clean.clean_gross(ctx, dpm, geo, 2.0)
    off, bins = _download(out)
    roff, rbins = oclean.gross_veto(pm, *geo, 2.0)
    np.testing.assert_array_equal(off, roff)
    np.testing.assert_array_equal(bins, rbins)
    out.release()
    dpm.release()


def test_persistency_and_robust_statistic_match_the_oracle(ctx):
    from paper_1407_8333_amd import clean
    n, t_fft = 500, 1024.0
    pm = synth.make_noise_peakmap(n, t_fft, 10000, 12000, seed=5, velocity="none")
    segs = []
    for i in range(n):
        b = set(pm.bins[pm.offsets[i]:pm.offsets[i + 1]].tolist())
        if i % 5:
            b.update([10500, 11234])
        segs.append(sorted(b))
    off = np.zeros(n + 1, np.int64)
    off[1:] = np.cumsum([len(s) for s in segs])
    pm2 = synth.Peakmap(t_fft, pm.t, pm.v, off, np.array([b for s in segs for b in s], np.int32))
    dpm = ctx.upload(pm2)
    for k_lo, k_hi in [(10001, 11999), (9000, 10007), (11999, 12000)]:
        c = clean.bin_counts(ctx, dpm, k_lo, k_hi)
        np.testing.assert_array_equal(c.cpu().numpy(), oclean.bin_counts(pm2, k_lo, k_hi))
    out, c, m1, m2 = clean.persistency_veto(ctx, dpm, 10001, 11999, 6.0)
    rm1, rm2 = oclean.robust_stats(oclean.bin_counts(pm2, 10001, 11999))
    assert (m1, m2) == (rm1, rm2)
    o, b = _download(out)
    ro, rb = oclean.veto_bins(pm2, 10001, 11999, c.cpu().numpy(), 1, 0, rm1 + 6.0 * rm2)
    np.testing.assert_array_equal(o, ro)
    np.testing.assert_array_equal(b, rb)
    assert not np.isin(b, [10500, 11234]).any()
    out.release()
    dpm.release()


def test_robust_statistic_edge_cases(ctx):
    import torch
    from paper_1407_8333_amd import clean
    from paper_1407_8333_amd._lib import FHError
    rng = synth.rng_for(8)
    cases = [[1, 2, 3, 4, 100], [4, 1, 3, 2], [7], [5, 5, 5, 5], [0, 0, 1],
             rng.integers(0, 50, 1001).tolist(), rng.integers(0, 3000, 4096).tolist()]
    for xs in cases:
        x = torch.tensor(xs, dtype=torch.int32, device="cuda")
        assert clean.robust_stats(ctx, x, max(xs)) == oclean.robust_stats(xs)
        assert clean.robust_stats(ctx, x, max(xs) + 17) == oclean.robust_stats(xs)
    with pytest.raises(FHError):
        clean.robust_stats(ctx, torch.tensor([1, 9], dtype=torch.int32, device="cuda"), 8)
    with pytest.raises(FHError):
        clean.robust_stats(ctx, torch.tensor([1, -1], dtype=torch.int32, device="cuda"), 8)
    with pytest.raises(FHError):
        clean.robust_stats(ctx, torch.zeros(0, dtype=torch.int32, device="cuda"), 8)


def test_line_finder_without_doppler_matches_the_oracle(ctx):
    from paper_1407_8333_amd import clean
    n, t_fft = 300, 1024.0
    k_lo, k_hi = 20480, 20480 + 1024
    pm = synth.make_noise_peakmap(n, t_fft, k_lo, k_hi, seed=21)
    line = [20480 + 300, 20480 + 812]
    segs = []
    for i in range(n):
        b = set(pm.bins[pm.offsets[i]:pm.offsets[i + 1]].tolist())
        b.update(line)
        segs.append(sorted(b))
    off = np.zeros(n + 1, np.int64)
    off[1:] = np.cumsum([len(s) for s in segs])
    pm2 = synth.Peakmap(t_fft, pm.t, pm.v, off, np.array([b for s in segs for b in s], np.int32), k_lo, k_hi)
    dpm = ctx.upload(pm2)
    dfd = (1.0 / t_fft) / (n * t_fft * 0.5)
    grid = synth.Grid(kf=10, b0=10 * (k_lo + 20), nf=10 * 980, ns=3, fdot0=-dfd, dfdot=dfd,
                      t0=0.5 * (pm.t[0] + pm.t[-1]))
    lc = clean.line_counts(ctx, dpm, grid).cpu().numpy()
    ref = oclean.line_counts(oracle.hough_map(pm2, grid, np.zeros(3)))
    np.testing.assert_array_equal(lc, ref.astype(np.int32))
    assert lc[10 * line[0] - grid.b0] == n
    out, _ = clean.line_veto(ctx, dpm, grid, k_lo, k_hi, n / 2)
    o, b = _download(out)
    ro, rb = oclean.veto_bins(pm2, k_lo, k_hi, ref, 10, 10 * k_lo - grid.b0, n / 2)
    np.testing.assert_array_equal(o, ro)
    np.testing.assert_array_equal(b, rb)
    assert not np.isin(b, line).any()
    out.release()
    dpm.release()


def test_cleaning_an_empty_peakmap(ctx):
    from paper_1407_8333_amd import clean
    t = synth.fft_times(6, 1024.0)
    pm = synth.Peakmap(1024.0, t, np.zeros((6, 3)), np.zeros(7, np.int64), np.zeros(0, np.int32))
    dpm = ctx.upload(pm)
    geo = clean.gross_geometry(t, 1000, 2000, 3600.0, 0.1, 1024.0)
    assert not clean.gross_histogram(ctx, dpm, geo).cpu().numpy().any()
    out, _ = clean.clean_gross(ctx, dpm, geo, 0.0)
    off, bins = _download(out)
    assert not off.any() and bins.size == 0
    assert not clean.bin_counts(ctx, dpm, 1000, 2000).cpu().numpy().any()
    out.release()
    dpm.release()


@pytest.fixture(scope="module")
def wide_band():
    """37 FFTs over 140 000 natural bins, with a run of popular bins."""
    pm = synth.random_peakmap(37, 1024.0, 5000, 145000, 0.05, synth.rng_for(3), min_gap=2)
    return pm


@pytest.mark.parametrize("width", [1, 1023, 32768, 32769, 131072, 131073])
def test_bin_counts_at_the_edges_of_the_lds_segments(ctx, wide_band, width):
    from paper_1407_8333_amd import clean
    dpm = ctx.upload(wide_band)
    for k_lo in (5003, 0):
        c = clean.bin_counts(ctx, dpm, k_lo, k_lo + width)
        np.testing.assert_array_equal(c.cpu().numpy(), oclean.bin_counts(wide_band, k_lo, k_lo + width))
    dpm.release()


@pytest.mark.parametrize("n_f", [1, 8192, 8193])
def test_gross_histogram_at_the_edges_of_the_lds_row(ctx, wide_band, n_f):
    """Rows that fit the LDS and longer ones; time cells that change inside
    and at the ends of a workgroup's 16 FFTs, FFTs outside the histogram."""
    from paper_1407_8333_amd import clean
    dpm = ctx.upload(wide_band)
    step = 0.5 * wide_band.t_fft
    for dt_h, t0 in [(16 * step, 0.0), (5 * step, 3 * step), (1e9, 0.0)]:
        geo = (t0, dt_h, 5, 16.0 / wide_band.t_fft, 5000 // 16, n_f)
        np.testing.assert_array_equal(clean.gross_histogram(ctx, dpm, geo).cpu().numpy(),
                                      oclean.gross_histogram(wide_band, *geo))
    dpm.release()


@pytest.mark.parametrize("n,x_max", [(1, 0), (2, 1), (4599, 6286), (65536, 36863), (65537, 36863), (3000, 36864)])
def test_robust_statistic_of_every_route(ctx, n, x_max):
    import torch
    from paper_1407_8333_amd import clean
    rng = np.random.default_rng(n + x_max)
    for x in (rng.integers(0, x_max + 1, n), rng.binomial(x_max, 0.07, n), np.full(n, x_max)):
        x = x.astype(np.int32)
        assert clean.robust_stats(ctx, torch.as_tensor(x, device="cuda"), x_max) == oclean.robust_stats(x)
