"""gs_bin_sort with the key count returned: the count is the call's own on every
thread and stream, and a call that overflows places nothing (needs an MI355X)."""
import ctypes
import threading
import time

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


def test_count_after_a_call_that_failed_behind_its_launches(gs):
    """A call that reports an error after its kernels were launched (here one that an
    earlier call of the thread left behind) returns with them done: its count, written
    late, would be taken for the next call's."""
    path = next(line.split()[-1] for line in open("/proc/self/maps") if "libamdhip64" in line)
    hip = ctypes.CDLL(path)
    small, large = _setup(gs, 300, 3, 1 << 16), _setup(gs, 5000, 4, 1 << 20)
    want = [gs.gs_bin_sort(*c, sync=True) for c in (small, large)]
    assert want[0] != want[1]
    a = torch.randn(4096, 4096, device="cuda")
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    torch.cuda.synchronize()
    with torch.cuda.stream(streams[0]):
        for _ in range(40):   # some ms in front of the failing call's kernels
            a @ a
    assert not streams[0].query()
    assert hip.hipSetDevice(1 << 20) != 0   # leaves its error for the thread's next check
    with pytest.raises(gs.GsError) as e:
        gs.gs_bin_sort(*small, sync=True, stream=streams[0])
    assert e.value.status == gs.GS_ERR_HIP
    assert streams[0].query()
    assert gs.gs_bin_sort(*large, sync=True, stream=streams[1]) == want[1]
    assert gs.gs_bin_sort(*small, sync=True, stream=streams[0]) == want[0]
    torch.cuda.synchronize()


def test_thread_that_binned_ends_while_another_records(gs):
    """What a thread's calls leave is given back without a call that recording forbids."""
    call = _setup(gs, 300, 5, 1 << 16)
    want = gs.gs_bin_sort(*call, sync=True)
    x = torch.zeros(64, device="cuda")
    done, go, got = threading.Event(), threading.Event(), []

    def work():
        stream = torch.cuda.Stream()
        got.append(gs.gs_bin_sort(*call, sync=True, stream=stream))
        stream.synchronize()
        done.set()
        go.wait()

    t = threading.Thread(target=work)
    t.start()
    done.wait()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        x.add_(1.0)
        go.set()
        t.join()
        time.sleep(0.2)   # join returns before the thread's own storage is taken down
        x.add_(1.0)
    for _ in range(3):
        graph.replay()
        torch.cuda.synchronize()
    assert got == [want] and bool((x == 6.0).all())


def test_more_calls_at_once_than_count_words(gs):
    """80 threads wait behind one stream's work: the calls past the 64 words copy theirs."""
    calls = [_setup(gs, 100 + k, 50 + k, 1 << 16) for k in range(80)]
    want = [gs.gs_bin_sort(*c, sync=True) for c in calls]
    a = torch.randn(8192, 8192, device="cuda")
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()
    got = [None] * len(calls)

    def work(k):
        got[k] = gs.gs_bin_sort(*calls[k], sync=True, stream=stream)

    threads = [threading.Thread(target=work, args=(k,)) for k in range(len(calls))]
    with torch.cuda.stream(stream):
        for _ in range(10):   # a tenth of a second in float32
            a @ a
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert got == want


def test_refused_wait_leaves_nothing_under_way(gs):
    """While another thread records in the global mode, waiting for a count is refused, as
    synchronising is: the call reports it, and returns with its stream done."""
    path = next(line.split()[-1] for line in open("/proc/self/maps") if "libamdhip64" in line)
    hip = ctypes.CDLL(path)
    call = _setup(gs, 300, 6, 1 << 16)
    want = gs.gs_bin_sort(*call, sync=True)
    a = torch.randn(8192, 8192, device="cuda")
    stream = torch.cuda.Stream()
    # a stream of its own: a spoilt recording leaves it unfit for the next one
    recorded, graph = ctypes.c_void_p(), ctypes.c_void_p()
    assert hip.hipStreamCreateWithFlags(ctypes.byref(recorded), 1) == 0   # non-blocking
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        for _ in range(10):   # a tenth of a second in front of the call's kernels
            a @ a
    seen = []

    def work():
        try:
            seen.append(gs.gs_bin_sort(*call, sync=True, stream=stream))
        except gs.GsError as e:
            seen.append(e.status)
        mode = ctypes.c_int(2)   # relaxed: the query is allowed
        hip.hipThreadExchangeStreamCaptureMode(ctypes.byref(mode))
        seen.append(stream.query())

    assert hip.hipStreamBeginCapture(recorded, 0) == 0   # global
    t = threading.Thread(target=work)
    t.start()
    t.join()
    hip.hipStreamEndCapture(recorded, ctypes.byref(graph))   # the refused wait has spoilt it
    hip.hipStreamDestroy(recorded)
    hip.hipGetLastError()
    assert seen == [gs.GS_ERR_HIP, True]
    assert gs.gs_bin_sort(*call, sync=True) == want
    torch.cuda.synchronize()
