"""GPU parity of the small-image engine (all steps of an image in one launch,
tiles exchanging their halos), bit for bit against the oracle: every compiled
tile shape at image sides around its tile and halo, both pixel types, pairings
and operators, several images at once, a bound of its waits so tight that it
gives up and the rounds of launches take over, and the no-allocation call."""
import numpy as np
import pytest

import oracle
from paper_1603_09180_amd import synth, thin

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def image(h, w, seed, dt):
    return synth.gen_blobs(h, w, seed, dt, nblobs=8, sigma=(2.0, 12.0))


def assert_image(t, st, ref):
    bad = np.argwhere(t.cpu().numpy() != ref.image)
    assert bad.size == 0, f"{len(bad)} pixels differ, first at {bad[:5].tolist()}"
    assert (st.passes, st.lowerings, st.converged) == (ref.passes, ref.lowerings, True)


# (shape, its tile's rows, columns)
SHAPES = [(1, 16, 16), (2, 24, 48), (3, 48, 48), (4, 128, 48), (5, 176, 48)]


@pytest.mark.parametrize("shape,th,tw", SHAPES)
def test_sides_around_the_tile(shape, th, tw, monkeypatch):
    monkeypatch.setenv("THIN_FLOW", str(shape))
    for k, (h, w) in enumerate([(3, 3), (th, tw), (th + 1, tw + 1), (th - 1, 2 * tw + 7),
                                (th + 8, tw - 5), (2 * th + 3, 3 * tw + 1)]):
        dt, lam, adj = (np.uint8, 5, "8,4") if k % 2 else (np.uint16, 900, "4,8")
        for op in ("leveling", "skeleton"):
            print("case flow shape", shape, h, w, np.dtype(dt).name, op, flush=True)
            F = image(h, w, 31 * k + shape, dt)
            t = torch.from_numpy(F.copy()).cuda()
            with thin.Context() as ctx:
                st = ctx.run(t, lam, adj, op=op)
            assert_image(t, st, oracle.sweep_dirty(F, lam, adj, op=op))


@pytest.mark.parametrize("shape", [1, 2, 3])
def test_long_runs(shape, monkeypatch):
    """Hundreds of rounds, through a pitched view."""
    monkeypatch.setenv("THIN_FLOW", str(shape))
    print("case flow long run shape", shape, flush=True)
    F = synth.ridges_512().image()[:230, :301].copy()
    frame = torch.full((230, 333), 7, dtype=torch.uint8, device="cuda")
    t = frame[:, :301]
    t.copy_(torch.from_numpy(F))
    with thin.Context() as ctx:
        st = ctx.run(t, 20, "8,4")
    assert_image(t, st, oracle.sweep_dirty(F, 20, "8,4"))
    assert bool((frame[:, 301:] == 7).all())


def test_several_images_at_once():
    """A batch whose tiles fit the device together runs as one launch; the
    same context runs it twice, then a single image, then the batch again."""
    rng = np.random.default_rng(3)
    imgs, lams, adjs, ops = [], [], [], []
    for i in range(24):
        h, w = int(rng.integers(1, 90)), int(rng.integers(1, 90))
        imgs.append(image(h, w, 500 + i, np.uint8 if i % 2 else np.uint16))
        lams.append(int(rng.integers(0, 30)))
        adjs.append(["8,4", "4,8"][i % 2])
        ops.append(["leveling", "skeleton"][(i // 2) % 2])
    refs = [oracle.sweep_dirty(F, l, a, op=o) for F, l, a, o in zip(imgs, lams, adjs, ops)]
    with thin.Context() as ctx:
        for rep in range(3):
            print("case flow batch", rep, flush=True)
            ts = [torch.from_numpy(F.copy()).cuda() for F in imgs]
            for t, st, ref in zip(ts, ctx.run_batch(ts, lams, adjs, ops=ops), refs):
                assert_image(t, st, ref)
            one = torch.from_numpy(imgs[rep].copy()).cuda()
            assert_image(one, ctx.run(one, lams[rep], adjs[rep], op=ops[rep]), refs[rep])


@pytest.mark.parametrize("shape", [1, 2])
def test_giving_up_falls_back_to_launches(shape, monkeypatch):
    """With no second look at a neighbour's words allowed, images of several
    tiles are given up (every block leaves) and come out right all the same."""
    monkeypatch.setenv("THIN_FLOW", f"{shape},0")
    Fs = [image(150, 201, 77, np.uint8), image(60, 90, 78, np.uint16)]
    ts = [torch.from_numpy(F.copy()).cuda() for F in Fs]
    print("case flow gives up", shape, flush=True)
    with thin.Context() as ctx:
        sts = ctx.run_batch(ts, [5, 300], ["8,4", "4,8"])
        one = torch.from_numpy(Fs[0].copy()).cuda()
        st = ctx.run(one, 5, "8,4")
    refs = [oracle.sweep_dirty(Fs[0], 5, "8,4"), oracle.sweep_dirty(Fs[1], 300, "4,8")]
    for t, s, r in zip(ts + [one], sts + [st], refs + refs[:1]):
        assert_image(t, s, r)


def test_scratch_cap_and_noalloc():
    """Under a cap too small for the exchange words the call still runs; the
    no-allocation call gives the same bytes and counts."""
    F = image(200, 333, 12, np.uint16)
    ref = oracle.sweep_dirty(F, 300, 1)
    t = torch.from_numpy(F.copy()).cuda()
    print("case flow scratch cap", flush=True)
    with thin.Context(max_device_bytes=400_000) as ctx:
        assert_image(t, ctx.run(t, 300, 1), ref)
    t = torch.from_numpy(F.copy()).cuda()
    raw = thin.thin_stats()
    with thin.Context() as ctx:
        assert thin.thin_run_noalloc(ctx.handle, t.data_ptr(), 200, 333, thin.THIN_U16, 300, 1,
                                     raw) == thin.THIN_OK
    torch.cuda.synchronize()
    assert_image(t, thin.Stats.of(raw), ref)


@pytest.mark.parametrize("polls", ["", ",0"], ids=["taken", "given_up"])
def test_last_images_handed_over(polls, monkeypatch):
    """A batch too large for the engine starts on the rounds of launches and
    leaves its last images to it (here 1092 tiles, 512 of them resident at
    most), or goes on in rounds when the engine gives up."""
    monkeypatch.setenv("THIN_FLOW", "2" + polls)
    imgs, lams, adjs, ops = [], [], [], []
    for i in range(12):
        dt = np.uint8 if i % 3 else np.uint16
        if i < 3:  # the long runs
            imgs.append(synth.gen_ridges(300, 300, 40 + i, dt))
        else:
            imgs.append(image(300, 300 - i, 600 + i, dt))
        lams.append((0, 12, 40)[i % 3] * (1 if i % 3 else 257))
        adjs.append(["8,4", "4,8"][i % 2])
        ops.append(["leveling", "skeleton"][(i // 2) % 2])
    refs = [oracle.sweep_dirty(F, l, a, op=o) for F, l, a, o in zip(imgs, lams, adjs, ops)]
    assert max(r.passes for r in refs) > 2 * min(r.passes for r in refs)
    ts = [torch.from_numpy(F.copy()).cuda() for F in imgs]
    print("case hand-over", polls, [r.passes for r in refs], flush=True)
    with thin.Context() as ctx:
        for t, st, ref in zip(ts, ctx.run_batch(ts, lams, adjs, ops=ops), refs):
            assert_image(t, st, ref)


def test_several_threads_and_streams():
    """Each thread runs images of its own on a stream of its own: launches that
    fit the device together (16x16 tiles), one that fills it (512x512 by 16x16
    tiles, alone) and a cooperative run."""
    import threading

    jobs = []
    for i in range(6):
        h, w = [(33, 60), (300, 290), (129, 120), (70, 33), (512, 512), (100, 90)][i]
        F = image(h, w, 900 + i, np.uint8 if i % 2 else np.uint16)
        lam = 5 if i % 2 else 700
        jobs.append((F, lam, ["8,4", "4,8"][i % 2], oracle.sweep_dirty(F, lam, ["8,4", "4,8"][i % 2])))
    wrong = []

    def work(i):
        F, lam, adj, ref = jobs[i]
        stream = torch.cuda.Stream()
        engine = thin.THIN_ENGINE_COOP if i == 5 else thin.THIN_ENGINE_AUTO
        with torch.cuda.stream(stream), thin.Context(stream=stream, engine=engine) as ctx:
            src = torch.from_numpy(F).cuda()
            for rep in range(8):
                t = src.clone()
                st = ctx.run(t, lam, adj)
                if not (np.array_equal(t.cpu().numpy(), ref.image) and
                        (st.passes, st.lowerings) == (ref.passes, ref.lowerings)):
                    wrong.append((i, rep))

    print("case flow threads", flush=True)
    threads = [threading.Thread(target=work, args=(i,)) for i in range(len(jobs))]
    for th in threads:
        th.start()
    for th in threads:
        th.join()
    assert wrong == []


def test_tune_cache_keeps_the_engine(tmp_path):
    """A recorded class whose second line says that the small-image engine beat
    its shape runs in one launch; without that line it runs the shape's rounds.
    Tuning leaves one line of the class's shape either way."""
    arch = torch.cuda.get_device_properties(0).gcnArchName.split(":")[0]
    F = image(300, 200, 4321, np.uint8)
    ref = oracle.sweep_dirty(F, 5, "8,4")
    path = tmp_path / "tune.txt"

    def launches():
        t = torch.from_numpy(F.copy()).cuda()
        with thin.Context(tune_cache=str(path), profile=True) as ctx:
            assert_image(t, ctx.run(t, 5, "8,4"), ref)
            return int(ctx.profile().launches)

    print("case flow tune cache", flush=True)
    shape = " 15 15 64 64 16 256 3 1.0\n"
    path.write_text(arch + shape)
    assert launches() > 1
    path.write_text(arch + shape + arch + "+flow" + shape)
    assert launches() == 1
    with thin.Context(tune_cache=str(path)) as ctx:
        ctx.autotune([torch.from_numpy(F.copy()).cuda()], [5], [0], reps=1)
    lines = path.read_text().splitlines()
    assert [l.startswith(arch + " 15 15 ") for l in lines].count(True) == 1
    assert (launches() == 1) == any(l.startswith(arch + "+flow 15 15 ") for l in lines)
