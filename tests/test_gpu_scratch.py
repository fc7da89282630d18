"""The scratch cap (thin_config.max_device_bytes): what the small-image engine
and change bitmaps hold for speed never makes a call fail that fits the cap
without them, whatever ran on the context before."""
import numpy as np
import pytest

import oracle
from paper_1603_09180_amd import synth, thin

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def image(h, w, seed, dt=np.uint8):
    return synth.gen_blobs(h, w, seed, dt, nblobs=8, sigma=(2.0, 12.0))


def check(ctx, F, lam, adj):
    t = torch.from_numpy(F.copy()).cuda()
    print("case cap", F.shape, F.dtype, flush=True)
    st = ctx.run(t, lam, adj)
    ref = oracle.sweep_dirty(F, lam, adj)
    assert np.array_equal(t.cpu().numpy(), ref.image)
    assert (st.passes, st.lowerings, st.converged) == (ref.passes, ref.lowerings, True)


def test_a_large_image_after_a_small_one():
    """6 MB hold the 2.56 MB twin and the tile state of the 1601x1600 image,
    not beside the 4 MB of exchange words of the 1000x1000 image before it."""
    with thin.Context(max_device_bytes=6_000_000) as ctx:
        for h, w in [(1000, 1000), (1601, 1600), (1000, 1000)]:
            check(ctx, image(h, w, h), 5, "8,4")


def test_many_small_images():
    """1000 images of 30x30: 1 MB of twins and 0.2 MB of tile state fit 4.6 MB,
    not beside the engine's 4 MB of vote words."""
    Fs = [image(30, 30, 7000 + i) for i in range(1000)]
    with thin.Context(max_device_bytes=4_600_000) as ctx:
        for rep in range(2):
            print("case cap batch", rep, flush=True)
            ts = [torch.from_numpy(F.copy()).cuda() for F in Fs]
            sts = ctx.run_batch(ts, [5] * 1000, ["8,4"] * 1000)
            for F, t, st in zip(Fs, ts, sts):
                ref = oracle.sweep_dirty(F, 5, "8,4")
                assert np.array_equal(t.cpu().numpy(), ref.image)
                assert (st.passes, st.lowerings) == (ref.passes, ref.lowerings)


@pytest.mark.parametrize("kw", [dict(), dict(max_passes=1000), dict(engine=thin.THIN_ENGINE_COOP)],
                         ids=["auto", "rounds", "coop"])
def test_rounds_without_change_bitmaps(kw):
    """A 512x512 image takes 273408 bytes of twin, tile state and queues; change
    bitmaps (64 KB in seeded tiles) would not fit beside them."""
    with thin.Context(max_device_bytes=274_000, **kw) as ctx:
        check(ctx, image(512, 512, 5), 5, "8,4")


def test_change_bitmaps_give_way():
    """Under 400 kB the second image's larger twin takes the place of the first
    one's; change bitmaps kept from the first would leave no room for it."""
    with thin.Context(max_device_bytes=400_000, max_passes=1000) as ctx:
        for h, w in [(512, 512), (600, 560), (512, 512)]:
            check(ctx, image(h, w, h), 5, "8,4")


def test_gradient_after_a_small_image():
    """The gradient's 32 bytes a pixel of 400x500 under a cap that holds them and
    the image's twin, not the exchange words of the image before."""
    F = image(400, 500, 3)
    with thin.Context(max_device_bytes=6_800_000) as ctx:
        check(ctx, F, 5, "8,4")
        src = torch.from_numpy(F.copy()).cuda()
        dst = torch.empty_like(src)
        print("case cap gradient", flush=True)
        ctx.gradient(src, dst, 1.0, 12.0)
        with thin.Context() as free:
            want = torch.empty_like(src)
            free.gradient(src, want, 1.0, 12.0)
        assert torch.equal(dst, want)
        check(ctx, F, 5, "8,4")
