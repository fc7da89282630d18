"""What a call does when the small-image engine cannot finish its images or
finds no room: the path taken, by the launches it takes, how long others keep it
waiting, and the result against the oracle."""
import threading
import time

import numpy as np
import pytest

import oracle
from paper_1603_09180_amd import synth, thin

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def ridges():
    return synth.ridges_512().image()[:230, :301].copy()


def launches(F, lam, adj, ref=None, **kw):
    """Round and engine launches of one call, its result checked."""
    t = torch.from_numpy(F.copy()).cuda()
    with thin.Context(profile=True, **kw) as ctx:
        st = ctx.run(t, lam, adj)
        n = int(ctx.profile().launches)
    ref = ref or oracle.sweep_dirty(F, lam, adj)
    assert np.array_equal(t.cpu().numpy(), ref.image)
    assert (st.passes, st.lowerings, st.converged) == (ref.passes, ref.lowerings, True)
    return n


def test_an_image_given_up_is_not_handed_back(monkeypatch):
    """One launch that gives up, then the rounds to the end."""
    F = ridges()
    print("case give-up launches", flush=True)
    monkeypatch.setenv("THIN_FLOW", "0")
    rounds = launches(F, 20, "8,4")
    assert rounds > 20
    monkeypatch.setenv("THIN_FLOW", "1")
    assert launches(F, 20, "8,4") == 1
    monkeypatch.setenv("THIN_FLOW", "1,0")
    assert launches(F, 20, "8,4") == rounds + 1


def test_a_give_up_is_remembered_for_a_while(monkeypatch):
    """The calls of a context go straight to rounds for a second after a give-up,
    then try the engine again; a context that did not give up uses it."""
    F = ridges()
    ref = oracle.sweep_dirty(F, 20, "8,4")
    monkeypatch.setenv("THIN_FLOW", "0")
    rounds = launches(F, 20, "8,4", ref)
    monkeypatch.setenv("THIN_FLOW", "1,0")
    print("case give-up remembered", flush=True)
    seen = []
    with thin.Context(profile=True) as ctx:
        for pause in (0, 0, 0, 1.2, 0):
            time.sleep(pause)
            t = torch.from_numpy(F.copy()).cuda()
            st = ctx.run(t, 20, "8,4")
            assert np.array_equal(t.cpu().numpy(), ref.image) and st.passes == ref.passes
            seen.append(int(ctx.profile(reset=True).launches))
    assert seen == [rounds + 1, rounds, rounds, rounds + 1, rounds]
    monkeypatch.setenv("THIN_FLOW", "1")
    assert launches(F, 20, "8,4", ref) == 1


@pytest.mark.parametrize("env", ["", "1", "1,0"])
def test_rounds_by_the_flag(env, monkeypatch):
    """The flag keeps small images to rounds, whatever shape is asked for."""
    F = ridges()
    ref = oracle.sweep_dirty(F, 20, "8,4")
    if env:
        monkeypatch.setenv("THIN_FLOW", env)
    print("case rounds flag", env, flush=True)
    n = launches(F, 20, "8,4", ref, rounds=True)
    monkeypatch.setenv("THIN_FLOW", "0")
    assert n == launches(F, 20, "8,4", ref)


def test_a_stream_of_few_compute_units(monkeypatch):
    """A stream with a compute-unit mask keeps to rounds: it cannot hold the blocks
    that the device holds."""
    import ctypes

    hip = ctypes.CDLL("libamdhip64.so")
    handle = ctypes.c_void_p()
    mask = (ctypes.c_uint32 * 8)(*[0x0000FFFF] * 8)
    torch.zeros(1, device="cuda")
    assert hip.hipExtStreamCreateWithCUMask(ctypes.byref(handle), 8, mask) == 0
    F = ridges()
    ref = oracle.sweep_dirty(F, 20, "8,4")
    print("case masked stream", flush=True)
    n = launches(F, 20, "8,4", ref, stream=torch.cuda.ExternalStream(handle.value))
    assert hip.hipStreamDestroy(handle) == 0
    monkeypatch.setenv("THIN_FLOW", "0")
    assert n == launches(F, 20, "8,4", ref)


def test_a_run_of_more_than_100000_passes():
    """A spiral corridor, consumed from its ends a pixel or two a pass: the
    engine stays with it to the end."""
    n, r, c, d, turns = 741, 2, 2, 0, 0
    F = np.full((n, n), 255, np.uint8)
    F[r, c] = 55
    step = [(0, 1), (1, 0), (0, -1), (-1, 0)]
    while turns < 2:
        y, x = r + step[d][0], c + step[d][1]
        yy, xx = y + step[d][0], x + step[d][1]
        if not (2 <= y < n - 2 and 2 <= x < n - 2) or (2 <= yy < n - 2 and 2 <= xx < n - 2
                                                       and F[yy, xx] == 55):
            d, turns = (d + 1) % 4, turns + 1
            continue
        r, c, turns = y, x, 0
        F[r, c] = 55
    ref = oracle.sweep_dirty(F, 0, "4,8")
    assert ref.passes > 131072
    print("case long spiral", ref.passes, flush=True)
    assert launches(F, 0, "4,8", ref) == 1


def sleep_cycles(ms):
    """The argument of torch.cuda._sleep for about `ms`."""
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    torch.cuda._sleep(100_000)
    a.record()
    torch.cuda._sleep(1_000_000)
    b.record()
    b.synchronize()
    return int(1_000_000 * ms / a.elapsed_time(b))


def independent_streams(cycles):
    """Two streams of which the second does not wait for the first's work (the
    device has few hardware queues, and streams may share one)."""
    first = torch.cuda.Stream()
    for _ in range(16):
        other = torch.cuda.Stream()
        with torch.cuda.stream(first):
            torch.cuda._sleep(cycles)
        t0 = time.perf_counter()
        with torch.cuda.stream(other):
            torch.zeros(8, device="cuda")
        other.synchronize()
        quick = time.perf_counter() - t0 < 0.05
        first.synchronize()
        if quick:
            return first, other
    pytest.skip("every stream shares the first one's queue")


def test_calls_do_not_wait_for_a_stream_that_is_not_there_yet():
    """One thread's stream has 150 ms of other work before its 512x512 image; the
    128x128 images of another thread, which do not fit beside that one, take
    their usual time: in one launch, but for those that come before the first
    thread knows that room is sought."""
    cycles = sleep_cycles(150)
    streams = independent_streams(cycles)
    F, G = synth.gen_blobs(512, 512, 1), synth.gen_blobs(128, 128, 2)
    refF, refG = oracle.sweep_dirty(F, 5, "8,4"), oracle.sweep_dirty(G, 5, "8,4")
    wrong, times, stop, launches = [], [], threading.Event(), []

    def slow():
        stream = streams[0]
        with torch.cuda.stream(stream), thin.Context(stream=stream) as ctx:
            src = torch.from_numpy(F).cuda()
            while not stop.is_set():
                t = src.clone()
                torch.cuda._sleep(cycles)
                ctx.run(t, 5, "8,4")
                if not np.array_equal(t.cpu().numpy(), refF.image):
                    wrong.append("slow")

    def quick():
        stream = streams[1]
        with torch.cuda.stream(stream), thin.Context(stream=stream, profile=True) as ctx:
            src = torch.from_numpy(G).cuda()
            for rep in range(50):
                t = src.clone()
                t0 = time.perf_counter()
                st = ctx.run(t, 5, "8,4")
                times.append(time.perf_counter() - t0)
                launches.append(int(ctx.profile(reset=True).launches))
                if not (np.array_equal(t.cpu().numpy(), refG.image) and st.passes == refG.passes):
                    wrong.append(rep)
                time.sleep(0.01)
        stop.set()

    print("case other work in a stream", flush=True)
    threads = [threading.Thread(target=f) for f in (slow, quick)]
    for th in threads:
        th.start()
    for th in threads:
        th.join()
    print("ms:", [round(1e3 * x, 2) for x in sorted(times)], flush=True)
    assert wrong == []
    assert sorted(times[4:])[-2] < 0.03
    assert sum(n == 1 for n in launches[20:]) >= 26, launches
