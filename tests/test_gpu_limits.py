"""Searches at the limits of the addresses and launches that they use."""
import numpy as np
import pytest

from paper_1407_8333_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture()
def ctx():
    from paper_1407_8333_amd import api
    c = api.Context(0)
    yield c
    c.close()


def test_stripe_edges_past_2_gib(ctx):
    """A direction whose stripe edges fill more than 2 GiB (541 M peaks, built
    on the GPU): the map and the candidates of 30 directions, in single launches
    and persistent ones, equal those of a slice that holds the peaks in reach."""
    import torch
    from paper_1407_8333_amd import api
    n_fft, n_bins, t_fft, k0 = 90_112, 17_970, 1024.0, 200_000
    if torch.cuda.mem_get_info()[0] < 120 << 30:
        pytest.skip("needs 120 GiB of device memory")
    print("case: stripe edges past 2 GiB", flush=True)
    rng = synth.rng_for(229)
    g = torch.Generator(device="cuda").manual_seed(8)
    sp = torch.rand((n_fft, n_bins), generator=g, device="cuda")  # a third of the bins are local maxima
    t = synth.fft_times(n_fft, t_fft)
    dpm = api.DevicePeakmap.from_spectra(ctx, sp, k0, 0.0, t, synth.detector_velocity(t, rng), t_fft)
    del sp
    torch.cuda.empty_cache()
    assert dpm.n_peaks + 16 * n_fft > (1 << 29) + 500 * n_bins // 3
    k_c = k0 + n_bins // 2
    part = dpm.slice(k_c - 1000, k_c + 1000)
    dfd = (1.0 / t_fft) / (n_fft * t_fft / 2)
    grid = synth.Grid(kf=10, b0=10 * (k_c - 32), nf=640, ns=17, fdot0=-8 * dfd, dfdot=dfd, t0=float(t[n_fft // 2]))
    sky = synth.sky_uniform(30, rng)
    sel = synth.Selection(width=64)
    maps = [api.fh_hough_map_i32(ctx, d, sky[0], grid).cpu().numpy() for d in (dpm, part)]
    assert maps[0].min() > 0.25 * n_fft
    np.testing.assert_array_equal(*maps)
    ref = api.fh_hough_candidates(ctx, part, sky, grid, sel)
    for n, tile_bins, chunk in ((2, 0, 0), (30, 64, 30)):  # windows searched for, and from rank tables
        got = api.fh_hough_candidates(ctx, dpm, sky[:n], grid, sel, tile_bins=tile_bins, sky_chunk=chunk)
        torch.cuda.synchronize()
        assert torch.equal(got, ref[:n]), n
    part.release()
    dpm.release()
