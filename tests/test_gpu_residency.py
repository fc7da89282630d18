"""GPU parity of the packed decision and of the seeded register-window
residency, bit for bit against the oracle, where they can go wrong: values at
both ends of the pixel type, lambda at and past the type's range, plateaus
(few levels, so every connectivity case and every tie occurs), and image sides
around the 32x32 tile and its 16-pixel halo."""
import numpy as np
import pytest

import oracle
from paper_1603_09180_amd import thin

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def check(F, lam, adj, op, **kw):
    ref = oracle.sweep_dirty(F, lam, adj, op=op)
    t = torch.from_numpy(F.copy()).cuda()
    with thin.Context(**kw) as ctx:
        st = ctx.run(t, lam, adj, op=op)
    torch.cuda.synchronize()
    bad = np.argwhere(t.cpu().numpy() != ref.image)
    assert bad.size == 0, f"{len(bad)} pixels differ, first at {bad[:5].tolist()}"
    assert (st.passes, st.lowerings, st.converged) == (ref.passes, ref.lowerings, True)


def plateaus(h, w, seed, levels):
    """Random image over the given gray levels, smoothed a little by repeating
    rows and columns so that plateaus of several pixels occur."""
    rng = np.random.default_rng(seed)
    small = rng.integers(0, len(levels), size=((h + 1) // 2, (w + 1) // 2))
    big = np.kron(small, np.ones((2, 2), np.int64))[:h, :w]
    noise = rng.integers(0, len(levels), size=(h, w))
    return levels[np.where(rng.random((h, w)) < 0.5, big, noise)]


SHAPES = [dict(tile=32, steps_per_round=16, threads=1024, variant=5),
          dict(tile=32, steps_per_round=16, threads=512, variant=5),
          dict(tile=32, steps_per_round=16, threads=1024, variant=2),
          dict(tile=64, steps_per_round=16, threads=512, variant=4),
          dict(tile=64, steps_per_round=16, threads=512, variant=0)]


@pytest.mark.parametrize("op", ["leveling", "skeleton"])
@pytest.mark.parametrize("adj", ["8,4", "4,8"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "t%d_n%d_v%d" % (s["tile"], s["threads"], s["variant"]))
def test_decision_at_the_ends_of_the_types(shape, adj, op):
    u8 = np.array([0, 1, 2, 127, 254, 255], np.uint8)
    u16 = np.array([0, 1, 255, 256, 32767, 32768, 65534, 65535], np.uint16)
    for i, lam in enumerate([0, 1, 254, 255, 65534, 65535, 65536, 2 ** 32 - 1]):
        print("case", shape, adj, op, "lambda", lam, flush=True)
        check(plateaus(70, 67, 100 + i, u8), lam, adj, op, **shape)
        check(plateaus(67, 70, 200 + i, u16), lam, adj, op, **shape)


@pytest.mark.parametrize("threads", [1024, 512])
@pytest.mark.parametrize("h,w", [(3, 3), (3, 64), (31, 33), (32, 32), (33, 31), (48, 49), (64, 65),
                                 (95, 97), (129, 17)])
def test_seeded_windows_around_the_tile(h, w, threads):
    levels = np.arange(0, 250, 7).astype(np.uint8)
    for op in ("leveling", "skeleton"):
        print("case seeded windows", h, w, threads, op, flush=True)
        check(plateaus(h, w, h * 1000 + w, levels), 9, "8,4", op, tile=32, steps_per_round=16,
              threads=threads, variant=5)
