"""Register-window tiles stage in groups of 4 pixels where base and pitch allow
it and pixel by pixel where not (and in one launch, which stages once): the last
group of a row cut at each of its pixels, a base off by one pixel, and pitches of
both kinds, in rounds, in one launch and in serving, against the oracle."""
import numpy as np
import pytest

import oracle
from paper_1603_09180_amd import synth, thin

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("how", ["rounds", "one_launch", "serving"])
@pytest.mark.parametrize("dt", [np.uint8, np.uint16], ids=["u8", "u16"])
def test_groups_and_single_pixels(how, dt):
    kw = dict(tile=32, steps_per_round=16, threads=1024, variant=2) if how == "rounds" else {}
    lam = 5 if dt == np.uint8 else 900
    for w in (61, 62, 63, 64, 65):
        F = synth.gen_blobs(70, w, 300 + w, dt, nblobs=8, sigma=(2.0, 12.0))
        ref = oracle.sweep_dirty(F, lam, "4,8")
        for pitch, off in ((68, 0), (68, 1), (68, 4), (67, 0)):
            print("case staging", how, np.dtype(dt).name, w, pitch, off, flush=True)
            flat = torch.full((70 * pitch + 8,), 7, dtype=torch.uint8 if dt == np.uint8 else torch.uint16,
                              device="cuda")
            t = flat[off:off + 70 * pitch].view(70, pitch)[:, :w]
            t.copy_(torch.from_numpy(F))
            with thin.Context(**kw) as ctx:
                if how == "serving":
                    assert ctx.serve_admit(t, lam, "4,8", tag=9)
                    done = []
                    while not done:
                        done, _ = ctx.serve_step(4)
                    st = done[0][1]
                else:
                    st = ctx.run(t, lam, "4,8")
            assert np.array_equal(t.cpu().numpy(), ref.image)
            assert (st.passes, st.lowerings) == (ref.passes, ref.lowerings)
            rest = flat.cpu().numpy().copy()
            keep = np.ones(rest.size, bool)
            for y in range(70):
                keep[off + y * pitch:off + y * pitch + w] = False
            assert (rest[keep] == 7).all()
