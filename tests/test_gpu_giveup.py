"""What a call does when the small-image engine cannot finish its images: the
path taken, by the launches it takes, and the result against the oracle."""
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
