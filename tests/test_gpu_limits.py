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


def test_front_of_more_threads_than_a_launch_holds(ctx):
    """A long, sparse observation (too sparse for rank tables) in one chunk of
    so many directions that their fronts need more than one launch: the
    candidates, also weighted, equal those of small chunks."""
    import torch
    from paper_1407_8333_amd import api
    n_fft, n_sky, t_fft = 120_000, 2_300, 1024.0
    if torch.cuda.mem_get_info()[0] < 60 << 30:
        pytest.skip("needs 60 GiB of device memory")
    assert 1024 * 118 * n_sky // 16 > (1 << 32) // 256  # workgroups of 16 FFTs per direction
    print("case: front of %d directions, %d FFTs" % (n_sky, n_fft), flush=True)
    rng = synth.rng_for(232)
    t = synth.fft_times(n_fft, t_fft)
    bins = np.sort(rng.integers(100_000, 103_000, n_fft * 2).reshape(n_fft, 2), axis=1).astype(np.int32)
    bins[:, 1] += 1
    pm = synth.Peakmap(t_fft, t, synth.detector_velocity(t, rng), np.arange(0, 2 * n_fft + 1, 2, dtype=np.int64),
                       bins.reshape(-1), 100_000, 103_001)
    dfd = (1.0 / t_fft) / (n_fft * t_fft / 2)
    grid = synth.Grid(kf=10, b0=10 * 101_500, nf=640, ns=4, fdot0=-2 * dfd, dfdot=dfd, t0=float(t[n_fft // 2]))
    sky = synth.sky_uniform(n_sky, rng)
    sel = synth.Selection(width=64)
    dpm = ctx.upload(pm)
    for w in (None, torch.as_tensor(synth.fft_weights(n_fft, rng), device="cuda")):
        got = [api.fh_hough_candidates(ctx, dpm, sky, grid, sel, weights=w, tile_bins=640, sky_chunk=c)
               for c in (n_sky, 500)]
        torch.cuda.synchronize()
        assert torch.equal(*got)
        assert (api.decode_candidates(got[0])["value"][:, :, 0] > 0).all()
    dpm.release()
