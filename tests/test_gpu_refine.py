"""Refined grid around coarse candidates (Sec. "Refined Grid in the parameter
space") and peakmap slicing, against the oracle run on the full peakmap."""
import math

import numpy as np
import pytest

import oracle
from paper_1407_8333_amd import skygrid, synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    from paper_1407_8333_amd import api
    c = api.Context(0)
    yield c
    c.close()


def _signal_band():
    """400 FFTs of 8192 s at 100-100.2 Hz with Doppler and one signal of
    known direction, frequency and spin-down."""
    rng = synth.rng_for(4242)
    t_fft, n = 8192.0, 400
    nhat = synth.sky_uniform(1, rng)[0]
    t = synth.fft_times(n, t_fft)
    t0 = 0.5 * (t[0] + t[-1])
    inj = synth.Injection(100.0913, -3.3e-10, nhat, lam=2.5)
    pm = synth.make_noise_peakmap(n, t_fft, int(100.0 * t_fft) - 120, int(100.2 * t_fft) + 120, seed=11,
                                  injections=[inj], t0=t0)
    grid = synth.make_grid(pm, 100.0, 100.2, -1e-9, 1e-10, t0=t0)
    return pm, grid, inj


def _reference_directions(lam_c, beta_c, dlam, dbeta, k_sky):
    """The refined directions written out with the scalar functions the
    library uses, in the same order (so both sides get identical vectors)."""
    L = (k_sky - 1) // 2
    eps = math.radians(23.44)
    ce, se = math.cos(eps), math.sin(eps)
    out = []
    for j in range(-L, L + 1):
        for i in range(-L, L + 1):
            lam = lam_c + i * (dlam / k_sky)
            bet = beta_c + j * (dbeta / k_sky)
            if abs(bet) > 0.5 * math.pi:
                lam += math.pi
                bet = (math.pi if bet > 0 else -math.pi) - bet
            lam = math.fmod(lam, 2.0 * math.pi)
            if lam < 0:
                lam += 2.0 * math.pi
            x, ye, ze = math.cos(bet) * math.cos(lam), math.cos(bet) * math.sin(lam), math.sin(bet)
            n = [x, ye * ce - ze * se, ye * se + ze * ce]
            r = math.sqrt(n[0] * n[0] + n[1] * n[1] + n[2] * n[2])
            out.append((lam, bet, [n[0] / r, n[1] / r, n[2] / r]))
    return out


def _oracle_refined(pm, cand, kf, k_fdot, k_sky, dfdot, t0, w=None):
    """Best cell of the refined volume by the oracle on the full peakmap:
    larger value, then smaller direction index, smaller bin, smaller row."""
    f0c, fdc = cand[0], cand[1]
    rgrid = synth.Grid(kf=kf, b0=int(round(f0c * kf * pm.t_fft)) - kf, nf=2 * kf + 1, ns=4 * k_fdot,
                       fdot0=fdc - 2 * dfdot, dfdot=dfdot / k_fdot, t0=t0)
    dirs = _reference_directions(*cand[2:], k_sky)
    best = None
    for d, (lam, bet, n) in enumerate(dirs):
        m = oracle.hough_map(pm, rgrid, np.array(n), weights=None if w is None else w.astype(np.float64))
        vmax = m.max()
        rows, bins = np.nonzero(m == vmax)
        k = np.lexsort((rows, bins))[0]
        if best is None or vmax > best[0]:
            best = (vmax, d, int(bins[k]), int(rows[k]))
    return best, rgrid, dirs


def test_peakmap_slice_matches_a_host_selection(ctx):
    import torch
    from paper_1407_8333_amd import api
    pm, _, _ = _signal_band()
    dpm = ctx.upload(pm)
    k_lo, k_hi = int(100.05 * pm.t_fft), int(100.12 * pm.t_fft)
    sub = dpm.slice(k_lo, k_hi)
    torch.cuda.synchronize()
    off, bins = sub.download()
    want_off = [0]
    want = []
    for i in range(pm.n_fft):
        b = pm.bins[pm.offsets[i]:pm.offsets[i + 1]]
        sel = b[(b >= k_lo) & (b < k_hi)]
        want.extend(sel.tolist())
        want_off.append(len(want))
    np.testing.assert_array_equal(off, np.array(want_off))
    np.testing.assert_array_equal(bins, np.array(want, dtype=np.int32))
    sub.release()
    dpm.release()


@pytest.mark.parametrize("weighted", [False, True])
def test_refined_candidate_is_the_best_cell_of_the_refined_volume(ctx, weighted):
    import torch
    from paper_1407_8333_amd import api
    pm, grid, inj = _signal_band()
    dpm = ctx.upload(pm)
    w = synth.fft_weights(pm.n_fft, synth.rng_for(5)) if weighted else None
    wt = None if w is None else torch.as_tensor(w, device="cuda")
    # coarse candidate: the coarse sky point nearest the signal, its best cell
    # in the sub-band of the signal
    g = skygrid.coarse_grid(100.2, pm.t_fft)
    nh = g.nhat()
    c = int(np.argmax(nh @ inj.nhat))
    sel = synth.Selection(width=int(round(0.01 * grid.kf * pm.t_fft)))
    raw = api.fh_hough_candidates(ctx, dpm, nh[c:c + 1], grid, sel, weights=wt)
    dec = api.decode_candidates(raw)
    sb = int(inj.f0 * grid.kf * pm.t_fft - grid.b0) // sel.width
    b, s = int(dec["bin"][0, sb, 0]), int(dec["row"][0, sb, 0])
    f0c = (grid.b0 + b) / (grid.kf * pm.t_fft)
    fdc = grid.fdot0 + s * grid.dfdot
    kf, k_fdot, k_sky = grid.kf, 3, 5
    cand = [f0c, fdc, g.lam[c], g.beta[c], g.dlam[c], g.dbeta[c]]
    out = api.decode_refined(api.refine(ctx, dpm, [cand], kf, k_fdot, k_sky, grid.dfdot, grid.t0,
                                        weights=wt))[0]
    torch.cuda.synchronize()
    best, rgrid, dirs = _oracle_refined(pm, cand, kf, k_fdot, k_sky, grid.dfdot, grid.t0, w)
    assert out["valid"] == 1
    if w is None:
        assert (float(out["value"]), int(out["sky"]), int(out["bin"]), int(out["row"])) == \
            (float(best[0]), best[1], best[2], best[3])
    else:
        tol = 1e-5 * max(best[0], float(np.mean(w)))
        assert float(out["value"]) == pytest.approx(best[0], abs=2 * tol)
    lam, bet, _ = dirs[int(out["sky"])]
    assert (out["lambda"], out["beta"]) == (lam, bet)
    assert out["f0"] == pytest.approx((rgrid.b0 + int(out["bin"])) / (kf * pm.t_fft), rel=0, abs=1e-12)
    assert out["fdot"] == pytest.approx(rgrid.fdot0 + int(out["row"]) * rgrid.dfdot, rel=1e-12)
    # the refined cell lies on the signal: within one natural bin in frequency
    # and one and a half coarse spin-down steps
    assert abs(out["f0"] - inj.f0) <= 1.0 / pm.t_fft
    assert abs(out["fdot"] - inj.fdot) <= 1.5 * grid.dfdot
    dpm.release()


def test_several_candidates_in_one_call(ctx):
    """Candidates in different sub-bands and one whose refined sky crosses
    the north pole; each result is the oracle's best cell of its own volume."""
    from paper_1407_8333_amd import api
    pm, grid, inj = _signal_band()
    dpm = ctx.upload(pm)
    g = skygrid.coarse_grid(100.2, pm.t_fft)
    rng = synth.rng_for(77)
    c_sig = int(np.argmax(g.nhat() @ inj.nhat))
    c_rand = int(rng.integers(len(g)))
    c_pole = 1  # first ring below the pole
    cands = [
        [inj.f0, inj.fdot + 0.4 * grid.dfdot, g.lam[c_sig], g.beta[c_sig], g.dlam[c_sig], g.dbeta[c_sig]],
        [100.031, -5.0e-10, g.lam[c_rand], g.beta[c_rand], g.dlam[c_rand], g.dbeta[c_rand]],
        [100.17, 0.0, g.lam[c_pole], g.beta[c_pole], g.dlam[c_pole], 3.0 * g.dbeta[c_pole]],
    ]
    kf, k_fdot, k_sky = grid.kf, 2, 7
    out = api.decode_refined(api.refine(ctx, dpm, cands, kf, k_fdot, k_sky, grid.dfdot, grid.t0))
    assert [int(x) for x in out["cand"]] == [0, 1, 2]
    for c, cand in enumerate(cands):
        best, rgrid, dirs = _oracle_refined(pm, cand, kf, k_fdot, k_sky, grid.dfdot, grid.t0)
        o = out[c]
        assert o["valid"] == 1
        assert (float(o["value"]), int(o["sky"]), int(o["bin"]), int(o["row"])) == \
            (float(best[0]), best[1], best[2], best[3])
        assert (o["lambda"], o["beta"]) == dirs[int(o["sky"])][:2]
    # the third volume reaches past the pole (its latitudes fold back)
    assert cands[2][3] + (k_sky - 1) // 2 * cands[2][5] / k_sky > 0.5 * math.pi
    dpm.release()


def test_refine_edge_cases(ctx):
    """No candidates is a no-op; an even k_sky, a zero spin-down step and a
    candidate below bin 0 are rejected before any launch."""
    from paper_1407_8333_amd import api
    from paper_1407_8333_amd._lib import FHError
    pm, grid, _ = _signal_band()
    dpm = ctx.upload(pm)
    assert api.refine(ctx, dpm, np.zeros((0, 6)), grid.kf, 2, 5, grid.dfdot, grid.t0).numel() == 0
    good = [100.1, 0.0, 1.0, 0.2, 0.05, 0.05]
    for kw, cand in [(dict(k_sky=4), good), (dict(dfdot=0.0), good),
                     (dict(), [1e-9, 0.0, 1.0, 0.2, 0.05, 0.05])]:
        args = dict(kf=grid.kf, k_fdot=2, k_sky=5, dfdot=grid.dfdot, t0=grid.t0)
        args.update(kw)
        with pytest.raises(FHError):
            api.refine(ctx, dpm, [cand], **args)
    dpm.release()


@pytest.mark.parametrize("kf,k_fdot,k_sky,n_fft,t_fft,density,mode,weighted", [
    (10, 1, 1, 130, 2048.0, 0.07, "exact", False),   # smallest volume, one direction, a partial round of FFTs
    (10, 5, 3, 1037, 2048.0, 0.07, "exact", True),   # several rounds of FFTs, the last one partial
    (4, 3, 3, 512, 2048.0, 0.45, "shift", True),     # exactly one round; dense peaks, more than one list pass
    (64, 46, 1, 60, 1024.0, 0.07, "exact", False),   # the largest volume that fits the LDS ...
    (64, 47, 1, 60, 1024.0, 0.07, "exact", False),   # ... and one searched with the tiles
])
def test_refined_volumes_of_every_route(ctx, kf, k_fdot, k_sky, n_fft, t_fft, density, mode, weighted):
    """Volumes searched in one workgroup's LDS and those too large for it, at
    the edges of the rounds of FFTs, against the oracle's best cell."""
    import torch
    from paper_1407_8333_amd import api
    rng = synth.rng_for(91 + kf + k_fdot)
    pm = synth.random_peakmap(n_fft, t_fft, int(90.0 * t_fft), int(90.2 * t_fft), density, rng)
    dfdot = 1.0 / (t_fft * 0.5 * n_fft * t_fft)
    t0 = 0.5 * (pm.t[0] + pm.t[-1])
    cands = [[90.1, -1.5 * dfdot, 1.0, 0.3, 0.05, 0.04], [90.03, 2.0 * dfdot, 4.0, -1.1, 0.03, 0.02]]
    w = synth.fft_weights(n_fft, rng) if weighted else None
    dpm = ctx.upload(pm)
    ctx.set_doppler(mode)
    try:
        out = api.decode_refined(api.refine(ctx, dpm, cands, kf, k_fdot, k_sky, dfdot, t0,
                                            weights=None if w is None else torch.as_tensor(w, device="cuda")))
    finally:
        ctx.set_doppler("exact")
    for o, cand in zip(out, cands):
        rgrid = synth.Grid(kf=kf, b0=int(round(cand[0] * kf * t_fft)) - kf, nf=2 * kf + 1, ns=4 * k_fdot,
                           fdot0=cand[1] - 2 * dfdot, dfdot=dfdot / k_fdot, t0=t0)
        best = None
        for d, (_, _, n) in enumerate(_reference_directions(*cand[2:], k_sky)):
            m = oracle.hough_map(pm, rgrid, np.array(n), weights=None if w is None else w.astype(np.float64),
                                 doppler=mode)
            rows, bins = np.nonzero(m == m.max())
            k = np.lexsort((rows, bins))[0]
            if best is None or m.max() > best[0]:
                best = (float(m.max()), d, int(bins[k]), int(rows[k]))
        if w is None:
            assert (float(o["value"]), int(o["sky"]), int(o["bin"]), int(o["row"])) == best
        else:
            # every cell is within 1e-5 of its exact sum, so the chosen one is
            # within twice that of the best
            assert float(o["value"]) == pytest.approx(best[0], abs=2e-5 * max(best[0], float(np.mean(w))))
    dpm.release()


def test_refinement_in_a_peakmap_of_more_peaks_than_32_bits_count(ctx):
    """A peakmap of more than 2^31 peaks, built on the GPU: the volumes, which
    need a few bins of it, equal those refined in a slice around them (the last
    32 FFTs and more lie past 2^31)."""
    import torch
    from paper_1407_8333_amd import api
    n_fft, n_bins, t_fft, k0 = 16_416, 400_000, 1024.0, 50_000
    if torch.cuda.mem_get_info()[0] < 80 << 30:
        pytest.skip("needs 80 GiB of device memory")
    print("case: refinement past 2^31 peaks", flush=True)
    rng = synth.rng_for(2031)
    g = torch.Generator(device="cuda").manual_seed(7)
    sp = torch.rand((n_fft, n_bins), generator=g, device="cuda")  # a third of the bins are local maxima
    t = synth.fft_times(n_fft, t_fft)
    dpm = api.DevicePeakmap.from_spectra(ctx, sp, k0, 0.0, t, synth.detector_velocity(t, rng), t_fft)
    del sp
    torch.cuda.empty_cache()
    assert dpm.n_peaks > (1 << 31) + 40 * n_bins // 3
    k_c = k0 + n_bins // 2
    part = dpm.slice(k_c - 2000, k_c + 2000)
    dfdot = 1.0 / (t_fft * 0.5 * n_fft * t_fft)
    t0 = 0.5 * (t[0] + t[-1])
    f_c = k_c / t_fft
    cands = [[f_c, -1.5 * dfdot, 1.0, 0.3, 0.05, 0.04], [f_c + 0.3, 2.0 * dfdot, 4.0, -1.1, 0.03, 0.02]]
    for mode in ("exact", "shift"):
        ctx.set_doppler(mode)
        try:
            got, ref = (api.decode_refined(api.refine(ctx, d, cands, 10, 5, 3, dfdot, t0)) for d in (dpm, part))
        finally:
            ctx.set_doppler("exact")
        assert got["valid"].all() and (got["value"] > 0.25 * n_fft).all()
        np.testing.assert_array_equal(got, ref)
    part.release()
    dpm.release()
