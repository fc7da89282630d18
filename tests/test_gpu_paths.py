"""Paths that image sizes alone no longer lead every test to: the rounds of
launches out of the static array, the default shape's rounds on mixed batches,
the last images of a batch handed over, engine launches larger than one
block to a compute unit from several threads, and what tuning records.  Results against the oracle, and
the path by the launches taken."""
import threading

import numpy as np
import pytest

import oracle
from paper_1603_09180_amd import synth, thin

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def image(h, w, seed, dt):
    return synth.gen_blobs(h, w, seed, dt, nblobs=8, sigma=(2.0, 12.0))


def assert_image(t, st, ref):
    assert np.array_equal(t.cpu().numpy(), ref.image)
    assert (st.passes, st.lowerings, st.converged) == (ref.passes, ref.lowerings, True)


@pytest.mark.parametrize("rounds", [True, False], ids=["flag", "size"])
def test_noalloc_in_rounds(rounds):
    """Two calls in a row on one context, the second on a smaller image: by the
    flag in both tile shapes of the rounds, and by size (more tiles than the
    device holds at once)."""
    sizes = ([(1500, 1300), (200, 333), (97, 131)] if rounds else [(2100, 1500), (1700, 1611)])
    with thin.Context(rounds=rounds) as ctx:
        for k, (h, w) in enumerate(sizes):
            dt, lam, adj = (np.uint8, 20, 0) if k % 2 == 0 else (np.uint16, 300, 1)
            F = image(h, w, 40 + k, dt)
            t = torch.from_numpy(F.copy()).cuda()
            raw = thin.thin_stats()
            print("case noalloc in rounds", h, w, np.dtype(dt).name, flush=True)
            rc = thin.thin_run_noalloc(ctx.handle, t.data_ptr(), h, w,
                                       thin.THIN_U8 if dt == np.uint8 else thin.THIN_U16, lam, adj, raw)
            torch.cuda.synchronize()
            assert rc == thin.THIN_OK
            assert_image(t, thin.Stats.of(raw), oracle.sweep_dirty(F, lam, adj))


@pytest.mark.parametrize("seed", [91, 92])
def test_mixed_batch_in_rounds(seed):
    """The default shape of a few megapixels (128x128 bit-flag tiles, one launch
    a pixel type and round): tiny and partial tiles next to full ones, both
    pixel types, operators and pairings, pitched views."""
    rng = np.random.default_rng(seed)
    Fs, ts, lams, adjs, ops = [], [], [], [], []
    for i in range(60):
        h, w = (int(round(np.exp(x))) for x in rng.uniform(np.log(3), np.log(1100), size=2))
        dt = np.uint16 if rng.random() < 0.4 else np.uint8
        Fs.append(image(h, w, seed * 1000 + i, dt))
        lams.append(int(rng.choice([0, 3, 20, 60])) * (257 if dt == np.uint16 else 1))
        adjs.append(int(rng.integers(0, 2)))
        ops.append("skeleton" if rng.random() < 0.3 else "leveling")
        pad = int(rng.integers(1, 9)) if rng.random() < 0.3 else 0
        big = torch.zeros((h, w + pad), dtype=torch.uint8 if dt == np.uint8 else torch.uint16,
                          device="cuda")
        big[:, :w] = torch.from_numpy(Fs[-1].copy()).cuda()
        ts.append(big[:, :w])
    assert sum(F.size for F in Fs) > 1 << 20
    print("case mixed batch in rounds", seed, flush=True)
    with thin.Context(rounds=True, profile=True) as ctx:
        sts = ctx.run_batch(ts, lams, adjs, ops=ops)
        assert ctx.profile().launches > 2
    for F, t, st, lam, adj, op in zip(Fs, ts, sts, lams, adjs, ops):
        assert_image(t, st, oracle.sweep_dirty(F, lam, adj, op=op))


def test_last_images_take_fewer_launches(monkeypatch):
    """A batch of 2730 tiles of the engine's 24x48 shape, more than its bound for
    a whole call, with one long image: it starts in rounds and ends in the engine."""
    Fs = [image(300, 300, 700 + i, np.uint8) for i in range(29)]
    Fs.append(synth.gen_ridges(300, 300, 41, np.uint8))
    refs = [oracle.sweep_dirty(F, 12, "8,4") for F in Fs]
    assert refs[-1].passes > 2 * max(r.passes for r in refs[:-1])
    monkeypatch.setenv("THIN_FLOW", "2")
    n = {}
    for rounds in (True, False):
        print("case hand-over launches", rounds, flush=True)
        ts = [torch.from_numpy(F.copy()).cuda() for F in Fs]
        with thin.Context(rounds=rounds, profile=True) as ctx:
            for t, st, ref in zip(ts, ctx.run_batch(ts, [12] * 30, ["8,4"] * 30), refs):
                assert_image(t, st, ref)
            n[rounds] = int(ctx.profile().launches)
    assert 1 < n[False] < n[True]


def test_large_launches_from_several_threads(monkeypatch):
    """16x16 tiles: 640x500 pixels are 1280 blocks, more than half of what the
    device holds, so two such launches never run together; smaller ones and a
    cooperative run come between."""
    monkeypatch.setenv("THIN_FLOW", "1")
    jobs = []
    for i, (h, w) in enumerate([(640, 500), (640, 500), (300, 290), (129, 120), (100, 90)]):
        F = image(h, w, 900 + i, np.uint8 if i % 2 else np.uint16)
        lam, adj = (5, "8,4") if i % 2 else (700, "4,8")
        jobs.append((F, lam, adj, oracle.sweep_dirty(F, lam, adj)))
    wrong, launches = [], [[] for _ in jobs]

    def work(i):
        F, lam, adj, ref = jobs[i]
        stream = torch.cuda.Stream()
        engine = thin.THIN_ENGINE_COOP if i == 4 else thin.THIN_ENGINE_AUTO
        with torch.cuda.stream(stream), thin.Context(stream=stream, engine=engine,
                                                     profile=True) as ctx:
            src = torch.from_numpy(F).cuda()
            for rep in range(5):
                t = src.clone()
                st = ctx.run(t, lam, adj)
                launches[i].append(int(ctx.profile(reset=True).launches))
                if not (np.array_equal(t.cpu().numpy(), ref.image) and
                        (st.passes, st.lowerings) == (ref.passes, ref.lowerings)):
                    wrong.append((i, rep))

    print("case large launches from threads", flush=True)
    threads = [threading.Thread(target=work, args=(i,)) for i in range(len(jobs))]
    for th in threads:
        th.start()
    for th in threads:
        th.join()
    print(launches, flush=True)
    assert wrong == []
    assert 1 in launches[0] + launches[1]      # the engine took some of them


@pytest.mark.parametrize("kw", [dict(rounds=True), dict(graph=True), dict(max_passes=500)],
                         ids=["rounds", "graph", "cap"])
def test_tuning_without_the_engine_keeps_its_record(kw, tmp_path):
    """A context that may not use the small-image engine tunes the class's shape
    and leaves the record that the engine beat it; a file without the record
    gets none."""
    arch = torch.cuda.get_device_properties(0).gcnArchName.split(":")[0]
    F = image(300, 200, 4321, np.uint8)
    path = tmp_path / "tune.txt"
    line = " 15 15 64 64 16 256 3 1.0"
    for record in (True, False):
        path.write_text(arch + line + "\n" + (arch + "+flow" + line + "\n" if record else ""))
        print("case tuning without the engine", kw, record, flush=True)
        with thin.Context(tune_cache=str(path), **kw) as ctx:
            ctx.autotune([torch.from_numpy(F.copy()).cuda()], [5], [0], reps=1)
        names = [l.split()[0] for l in path.read_text().splitlines()]
        assert sorted(names) == [arch] + [arch + "+flow"] * record
        t = torch.from_numpy(F.copy()).cuda()
        with thin.Context(tune_cache=str(path), profile=True) as ctx:
            assert_image(t, ctx.run(t, 5, "8,4"), oracle.sweep_dirty(F, 5, "8,4"))
            assert (ctx.profile().launches == 1) == record


def test_tuning_times_the_untuned_call():
    """default_ms is a call of the context without tuning: for small crests one
    launch of the engine (1.37 ms), and with the engine kept out a run in rounds
    (2.2, as the best shape)."""
    t = torch.from_numpy(synth.ridges_512().image()).cuda()
    print("case tuning, untuned call", flush=True)
    with thin.Context() as ctx:
        res = ctx.autotune([t], [20], [0], reps=2)
    with thin.Context(rounds=True) as ctx:
        kept_out = ctx.autotune([t], [20], [0], reps=2)
    print(res, kept_out, flush=True)
    assert res["default_ms"] < 0.85 * res["ms"]
    assert kept_out["default_ms"] > 0.85 * kept_out["ms"]


def test_tuning_times_shapes_as_they_run(monkeypatch):
    """Shapes are timed with the last images handed over, as the calls that will
    use the choice run them: far fewer launches than without the engine, though
    the call as a whole does not qualify for it."""
    Fs = [image(300, 300, 700 + i, np.uint8) for i in range(29)]
    Fs.append(synth.gen_ridges(300, 300, 41, np.uint8))
    ts = [torch.from_numpy(F).cuda() for F in Fs]
    monkeypatch.setenv("THIN_FLOW", "2")
    n = {}
    for rounds in (True, False):
        print("case tuning with hand-over", rounds, flush=True)
        with thin.Context(rounds=rounds, profile=True) as ctx:
            ctx.autotune(ts, [12] * 30, [0] * 30, reps=1)
            n[rounds] = int(ctx.profile().launches)
    print(n, flush=True)
    assert n[False] < 0.7 * n[True]


@pytest.mark.parametrize("engine", [thin.THIN_ENGINE_STEP, thin.THIN_ENGINE_WORKLIST,
                                    thin.THIN_ENGINE_COOP], ids=["step", "worklist", "coop"])
def test_tuning_in_contexts_of_other_engines(engine):
    """Tuning is the tiled engine's whatever engine the context runs: also on an
    image longer than the work-list engine takes."""
    t = torch.from_numpy(image(3, 131080, 8, np.uint8)).cuda()
    print("case tuning in another engine's context", engine, flush=True)
    with thin.Context(engine=engine) as ctx:
        assert ctx.autotune([t], [5], [0], reps=1)["candidates"] > 40
