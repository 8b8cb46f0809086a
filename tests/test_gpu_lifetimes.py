"""What a context keeps past a call (captured searches, blocks of released
peakmaps, workspaces) against peakmaps that come and go."""
import numpy as np
import pytest

import oracle
from paper_1407_8333_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture()
def ctx():
    from paper_1407_8333_amd import api
    c = api.Context(0)
    yield c
    c.close()


def _band(seed, density, n_fft=300):
    """n_fft FFTs of random peaks, and a grid that does not depend on seed."""
    rng = synth.rng_for(seed)
    t_fft = 2048.0
    pm = synth.random_peakmap(n_fft, t_fft, 60_000, 60_400, density, rng)
    dfd = (1.0 / t_fft) / (n_fft * t_fft / 2)
    grid = synth.Grid(kf=10, b0=10 * 60_020, nf=10 * 360, ns=17, fdot0=-8 * dfd, dfdot=dfd, t0=0.0)
    return pm, grid


def test_captured_searches_of_successive_peakmaps(ctx):
    """One peakmap after the other, each released before the next is made, so
    that handles and blocks are used again: a captured search with the same
    grid, output and stream runs on its own peakmap every time."""
    import torch
    from paper_1407_8333_amd import api
    st = torch.cuda.Stream()
    sky = synth.sky_uniform(5, synth.rng_for(3))
    sel = synth.Selection(width=600)
    out = None
    for rep, density in enumerate((0.05, 0.08, 0.02, 0.08)):
        print("case: peakmap %d of density %g" % (rep, density), flush=True)
        pm, grid = _band(500 + rep, density)
        dpm = ctx.upload(pm)
        if out is None:
            out = torch.empty((5, api.n_subbands(grid, sel), 2, 8), dtype=torch.int32, device="cuda")
        with torch.cuda.stream(st):
            for _ in range(2):  # captured, then replayed
                out.zero_()
                api.fh_hough_candidates(ctx, dpm, sky, grid, sel, use_graph=1, out=out, stream=st)
                ref = api.fh_hough_candidates(ctx, dpm, sky, grid, sel, stream=st)
                st.synchronize()
                assert torch.equal(out, ref), rep
        idx, _ = oracle.candidates(oracle.hough_map(pm, grid, sky[2]), sel.width, sel.excl, sel.sep)
        np.testing.assert_array_equal(api.decode_candidates(out)["bin"][2][idx[..., 0] == 1],
                                      idx[..., 1][idx[..., 0] == 1])
        dpm.release()


def test_map_after_a_refused_allocation(ctx):
    """An allocation that the device has no room for fails its own call only:
    HIP keeps the error of a failed call, and launches report it."""
    import torch
    from paper_1407_8333_amd import api
    from paper_1407_8333_amd._lib import FHError
    pm, grid = _band(510, 0.08)
    dpm = ctx.upload(pm)
    nhat = synth.sky_uniform(1, synth.rng_for(4))[0]
    with pytest.raises(FHError) as e:
        api.Server(ctx, 1 << 46)
    assert e.value.status == -2  # FH_E_NOMEM
    got = api.fh_hough_map_i32(ctx, dpm, nhat, grid)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(got.cpu().numpy(), oracle.hough_map(pm, grid, nhat).astype(np.int32))
    dpm.release()


def test_release_beside_a_capture(ctx):
    """A peakmap released on one thread while another thread captures the
    static map of another peakmap: the capture stands, and its replays are
    right, also with another peakmap built in between."""
    import threading

    import torch
    from paper_1407_8333_amd import _lib, api
    pm, grid = _band(520, 0.08)
    nhat = synth.sky_uniform(1, synth.rng_for(5))[0]
    ref = oracle.hough_map(pm, grid, nhat).astype(np.int32)
    dpm, other = ctx.upload(pm), ctx.upload(_band(521, 0.05)[0])
    out = torch.empty((grid.ns, grid.nf), dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, capture_error_mode="thread_local"):
        t = threading.Thread(target=_lib.fh_peakmap_release, args=(ctx.handle, other.handle))
        t.start()
        t.join()
        other.handle = None
        api.fh_hough_map_i32_static(ctx, dpm, nhat, grid, out)
    for rep in range(3):
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        np.testing.assert_array_equal(out.cpu().numpy(), ref)
        ctx.upload(_band(522 + rep, 0.05)[0]).release()
    dpm.release()
