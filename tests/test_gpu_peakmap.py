"""GPU peakmap construction against the oracle: bit-exact CSR."""
import numpy as np
import pytest

from oracle import peakmap
from paper_1407_8333_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_fft,n_bins,with_ar", [(1, 3, False), (7, 257, True), (300, 8500, True),
                                                   (3140, 1000, False)])
def test_peakmap_from_spectra_matches_oracle(n_fft, n_bins, with_ar):
    import torch
    from paper_1407_8333_amd import api
    rng = synth.rng_for(n_fft + n_bins)
    ar = rng.uniform(0.5, 2.0, (n_fft, n_bins)).astype(np.float32)
    sp = (rng.standard_exponential((n_fft, n_bins)).astype(np.float32) * ar).astype(np.float32)
    if not with_ar:
        sp = rng.standard_exponential((n_fft, n_bins)).astype(np.float32)
    t = synth.fft_times(n_fft, 1024.0)
    v = synth.detector_velocity(t, rng)
    with api.Context(0) as ctx:
        dsp = torch.as_tensor(sp, device="cuda")
        dar = torch.as_tensor(ar, device="cuda") if with_ar else None
        dpm = api.DevicePeakmap.from_spectra(ctx, dsp, 12345, 2.5, t, v, 1024.0, sar=dar)
        off, bins = dpm.download()
        ref_off, ref_bins = peakmap.peakmap_from_spectra(sp, ar if with_ar else None, 12345, 2.5)
        np.testing.assert_array_equal(off, ref_off)
        np.testing.assert_array_equal(bins, ref_bins)
        dpm.release()


def test_built_peakmap_feeds_the_hough_map():
    """The GPU-built peakmap gives the same Hough map as the uploaded one."""
    import torch
    from paper_1407_8333_amd import api
    rng = synth.rng_for(8)
    n_fft, t_fft = 400, 4096.0
    k_lo, n_bins = 300 * 4096 - 200, 1400
    sp = rng.standard_exponential((n_fft, n_bins)).astype(np.float32)
    t = synth.fft_times(n_fft, t_fft)
    v = synth.detector_velocity(t, rng)
    off, bins = peakmap.peakmap_from_spectra(sp, None, k_lo, 2.5)
    pm = synth.Peakmap(t_fft, t, v, off, bins)
    grid = synth.make_grid(pm, 300.0, 300.2, -1e-8, 1e-9)
    with api.Context(0) as ctx:
        built = api.DevicePeakmap.from_spectra(ctx, torch.as_tensor(sp, device="cuda"), k_lo, 2.5, t, v, t_fft)
        up = ctx.upload(pm)
        n = synth.sky_uniform(1, rng)[0]
        a = api.fh_hough_map_i32(ctx, built, n, grid)
        b = api.fh_hough_map_i32(ctx, up, n, grid)
        torch.cuda.synchronize()
        assert torch.equal(a, b)
        built.release()
        up.release()


@pytest.mark.parametrize("n_fft,n_bins", [(5, 4), (5, 66), (5, 513), (5, 514), (5, 515), (3, 2049), (3, 2050),
                                          (3, 2051), (3, 4099), (8191, 5), (8192, 5), (8200, 5), (16385, 4)])
@pytest.mark.parametrize("with_ar", [False, True])
def test_rows_at_the_edges_of_a_waves_run_and_of_the_scan(n_fft, n_bins, with_ar):
    """Rows that end around a wave's 512 bins and a workgroup's 2048, FFT
    counts around the scan's 8192, rows with a pitch, dense peaks, and
    infinities and NaN among the values."""
    import torch
    from paper_1407_8333_amd import api
    rng = synth.rng_for(n_fft * 7 + n_bins)
    ld = n_bins + 3
    sp = (4.0 * rng.standard_exponential((n_fft, ld))).astype(np.float32)
    sp[rng.random(sp.shape) < 0.02] = np.inf
    sp[rng.random(sp.shape) < 0.02] = np.nan
    ar = rng.uniform(0.5, 2.0, (n_fft, ld)).astype(np.float32)
    t = synth.fft_times(n_fft, 1024.0)
    with api.Context(0) as ctx:
        dsp = torch.as_tensor(sp, device="cuda")[:, :n_bins]
        dar = torch.as_tensor(ar, device="cuda")[:, :n_bins] if with_ar else None
        dpm = api.DevicePeakmap.from_spectra(ctx, dsp, 77, 2.5, t, np.zeros((n_fft, 3)), 1024.0, sar=dar)
        off, bins = dpm.download()
        with np.errstate(invalid="ignore"):
            ref_off, ref_bins = peakmap.peakmap_from_spectra(sp[:, :n_bins], ar[:, :n_bins] if with_ar else None,
                                                             77, 2.5)
        np.testing.assert_array_equal(off, ref_off)
        np.testing.assert_array_equal(bins, ref_bins)
        dpm.release()


def test_blocks_of_released_peakmaps_are_handed_on_safely():
    """Peakmaps built, filtered and released in turn, through two contexts:
    every live peakmap keeps its own peaks, and device memory goes back with
    the contexts."""
    import torch
    from paper_1407_8333_amd import api
    rng = synth.rng_for(99)
    t = synth.fft_times(50, 1024.0)
    v = synth.detector_velocity(t, rng)
    torch.cuda.synchronize()
    with api.Context(0) as a, api.Context(0) as b:
        live = []
        for turn in range(14):
            ctx = (a, b)[turn % 2]
            n_bins = int(rng.integers(40, 4000))
            sp = rng.standard_exponential((50, n_bins)).astype(np.float32)
            want = peakmap.peakmap_from_spectra(sp, None, 500, 2.5)
            pm = api.DevicePeakmap.from_spectra(ctx, torch.as_tensor(sp, device="cuda"), 500, 2.5, t, v, 1024.0)
            live.append((pm, want))
            if turn % 3 == 2:
                lo, hi = 500 + n_bins // 4, 500 + n_bins // 2 + 1
                sub = pm.slice(lo, hi)
                keep = (want[1] >= lo) & (want[1] < hi)
                off = np.concatenate([[0], np.cumsum(keep)])[want[0]]
                live.append((sub, (off, want[1][keep])))
            if len(live) > 5:
                live.pop(int(rng.integers(len(live))))[0].release()
            for p, (off, bins) in live:
                got = p.download()
                np.testing.assert_array_equal(got[0], off)
                np.testing.assert_array_equal(got[1], bins)
        for p, _ in live:
            p.release()


@pytest.mark.parametrize("what,value", [("t", np.nan), ("t", np.inf), ("v", np.nan), ("v", -np.inf), ("v", 1e-2),
                                        ("v", 1e200)])
@pytest.mark.parametrize("at", [0, 36])
def test_bad_times_and_velocities_are_refused(what, value, at):
    import torch
    from paper_1407_8333_amd import api
    from paper_1407_8333_amd._lib import FH_E_INVALID, FHError
    n = 37
    t, v = synth.fft_times(n, 1024.0), np.zeros((n, 3))
    if what == "t":
        t[at] = value
    else:
        v[at, 1] = value
    pm = synth.Peakmap(1024.0, t, v, np.arange(n + 1, dtype=np.int64), np.full(n, 5, np.int32))
    with api.Context(0) as ctx:
        for build in (lambda: ctx.upload(pm),
                      lambda: api.DevicePeakmap.from_spectra(ctx, torch.ones((n, 8), device="cuda"), 5, 2.5, t, v, 1024.0)):
            with pytest.raises(FHError) as e:
                build()
            assert e.value.status == FH_E_INVALID and "%s[%d]" % (what, at) in str(e.value)
