"""gs_bin_sort with the key count returned: the count is the call's own on every
thread and stream, and a call that overflows places nothing (needs an MI355X)."""
import threading

import pytest
import torch

from paper_2409_09295_amd import scenes

pytestmark = pytest.mark.gpu


def _setup(gs, n, seed, capacity):
    cam = scenes.pinhole(160, 120, 128.0)
    sp = scenes.random_splats(n, [cam], seed, sigma_px=(0.6, 3.0), cull_frac=0.3)
    views = gs.Views([cam])
    bins = gs.Bins.empty(capacity, views.n_tiles)
    ws = gs.workspace(gs.gs_bin_sort_workspace_size(n, views, capacity))
    return gs.Projected.from_splats(sp), n, views, bins, ws


@pytest.mark.parametrize("n", [200, (1 << 18) + 1])   # short path, general path
def test_count_and_overflow(gs, n):
    proj, n, views, bins, ws = _setup(gs, n, 1, 1 << 23)
    want = gs.gs_bin_sort(proj, n, views, bins, ws, sync=True)
    torch.cuda.synchronize()
    assert want == int(bins.n_keys) == int((bins.ranges[:, 1] - bins.ranges[:, 0]).sum()) > 0
    few = gs.Bins.empty(want - 1, views.n_tiles)
    few.values.fill_(-1)
    few.ranges.fill_(-1)
    with pytest.raises(gs.GsError) as e:
        gs.gs_bin_sort(proj, n, views, few, ws, sync=True)
    assert e.value.status == gs.GS_ERR_CAPACITY and e.value.required == want
    assert int((few.values + 1).abs().sum()) == 0 and int(few.ranges.abs().sum()) == 0
    assert torch.equal(few.order.cpu(), torch.arange(views.n_tiles, dtype=torch.int32))


def test_threads_and_streams_get_their_own_counts(gs):
    sizes = [1, 300, 5000, (1 << 18) + 1]
    calls = [_setup(gs, n, 7 + n, 1 << 23) for n in sizes]
    want = [gs.gs_bin_sort(*c, sync=True) for c in calls]
    torch.cuda.synchronize()
    got = [[] for _ in sizes]

    def work(i):
        stream = torch.cuda.Stream()
        for _ in range(25):
            got[i].append(gs.gs_bin_sort(*calls[i], sync=True, stream=stream))
        stream.synchronize()

    threads = [threading.Thread(target=work, args=(i,)) for i in range(len(sizes))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert got == [[w] * 25 for w in want]
