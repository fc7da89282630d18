"""Workloads of the thinning library and how to run one pass of each.

A case is a dict of plain values; its "path" says which public entry point a
pass goes through:

  run       Context.run on one image (the plain call)
  noalloc   thin_run_noalloc on one image (callers that must not allocate)
  gradient  Context.gradient on one image (magnitude and stored values)
  pipeline  Context.gradient into a u8 image, then Context.run on it (the
            paper's illustrated pipeline)
  batch     Context.run_batch on many images of uneven sizes
  serving   serve.replay of host requests that are all present at once:
            pinned inputs copied in, admitted, thinned, results copied back

The library thins in place, so a pass first copies the kept input over the
working buffer, as a program that thins a stream of images fills its buffer.
Gray levels and lambda are whole numbers: images, pass counts and lowering
counts have one right value.
"""
import math

import numpy as np
import torch

from paper_1603_09180_amd import serve, synth, thin

U8_TOP, U16_TOP = 255, 65535


def listed():
    return [
        # The smallest image the batch and serving workloads hold: what a call
        # costs when there is next to nothing to do.
        dict(name="run_blobs_67x64", path="run", kind="blobs", h=67, w=64, bits=8, lam=5,
             adj="8,4", op="leveling"),
        # The small parity image: plain destructible points only (lambda 0).
        dict(name="run_blobs_128", path="run", kind="blobs", h=128, w=128, bits=8, lam=0,
             adj="8,4", op="leveling"),
        # A serving loop under graph capture or without an allocator: ragged
        # 16-bit image, the other adjacency pair.
        dict(name="noalloc_blobs_301x451_u16", path="noalloc", kind="blobs", h=301, w=451, bits=16,
             lam=500, adj="4,8", op="leveling"),
        # The paper-shaped image (512 x 512, thin bright crests): leveling,
        # then the paper's own operator on it.
        dict(name="run_ridges_512", path="run", kind="ridges", h=512, w=512, bits=8, lam=20,
             adj="8,4", op="leveling"),
        dict(name="run_skeleton_512", path="run", kind="ridges", h=512, w=512, bits=8, lam=10,
             adj="8,4", op="skeleton"),
        # The paper's Fig. 1 from a gray image to its skeleton.
        dict(name="pipeline_512", path="pipeline", kind="blobs", h=512, w=512, bits=8, lam=10,
             adj="8,4", op="skeleton", alpha=1.0, gain=12.0),
        # The gradient front-end by itself on a larger ragged image, 16-bit
        # result and float magnitude.
        dict(name="gradient_1601x1283", path="gradient", kind="blobs", h=1601, w=1283, bits=8,
             out_bits=16, alpha=0.8, gain=257.0),
        # A larger ragged crest image in 16 bits under the skeleton.
        dict(name="run_skeleton_1283x1025_u16", path="run", kind="ridges", h=1283, w=1025, bits=16,
             lam=2570, adj="4,8", op="skeleton"),
        # The large plain call.
        dict(name="run_blobs_8192_u16", path="run", kind="blobs", h=8192, w=8192, bits=16, lam=500,
             adj="4,8", op="leveling", sigma=16.0),
        # The benchmark's batch: 512 uneven u8 images, 162 Mpixel.
        dict(name="batch_512", path="batch", n=512, lo=64, hi=2048, u16=False, mixed=False,
             pitched=False, plan=4),
        # A batch that mixes pixel types, operators, adjacency pairs and
        # pitched views of larger frames.
        dict(name="batch_mixed_96", path="batch", n=96, lo=64, hi=640, u16=True, mixed=True,
             pitched=True, plan=11),
        # Continuous batching from host memory, every request present.
        dict(name="serving_160", path="serving", n=160, lo=64, hi=2048, plan=5),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the listed ones' ranges: sides from 64 to 8192 (crest
    images to 1283 x 1025 pixels), both pixel types, pairings and operators,
    batches of 2 to 512 images."""
    path = rng.choice(["run", "run", "run", "noalloc", "gradient", "pipeline", "batch", "batch",
                       "serving"])
    adj = rng.choice(["8,4", "4,8"])
    op = rng.choice(["leveling", "skeleton"])
    bits = rng.choice([8, 16])
    lam = rng.choice([0, rng.randint(1, 60)]) * (1 if bits == 8 else rng.choice([1, 25, 257]))
    if path in ("batch", "serving"):
        mixed = rng.random() < 0.5
        hi = _log_int(rng, 256, 2048)
        # as many images as keep the expected pixels below the listed batch's
        mean = ((hi - 64) / math.log(hi / 64)) ** 2
        most = 512 if path == "batch" else 160
        n = _log_int(rng, 2, max(3, min(most, int(1.2e8 / mean))))
        if path == "serving":
            return dict(path=path, n=n, lo=64, hi=hi, plan=rng.randint(0, 10 ** 6))
        return dict(path=path, n=n, lo=64, hi=hi, u16=mixed or rng.random() < 0.3, mixed=mixed,
                    pitched=rng.random() < 0.3, plan=rng.randint(0, 10 ** 6))
    kind = rng.choice(["blobs", "ridges"])
    if path in ("run", "noalloc") and kind == "blobs" and op == "leveling":
        h, w = _log_int(rng, 64, 8192), _log_int(rng, 64, 8192)
        if path == "noalloc":
            h, w = min(h, 4096), min(w, 4096)
    elif path == "gradient":
        h, w = _log_int(rng, 64, 2048), _log_int(rng, 64, 2048)
    else:
        h, w = _log_int(rng, 64, 1283), _log_int(rng, 64, 1025)
    if path == "noalloc":
        op = "leveling"
    if path == "gradient":
        return dict(path=path, kind="blobs", h=h, w=w, bits=bits, out_bits=rng.choice([8, 16]),
                    alpha=round(rng.uniform(0.5, 2.0), 3), gain=round(rng.uniform(1.0, 16.0), 2))
    if path == "pipeline":
        return dict(path=path, kind="blobs", h=h, w=w, bits=8, lam=rng.randint(1, 40), adj=adj,
                    op=op, alpha=round(rng.uniform(0.5, 2.0), 3),
                    gain=round(rng.uniform(4.0, 16.0), 2))
    return dict(path=path, kind=kind, h=h, w=w, bits=bits, lam=lam, adj=adj, op=op)


# ------------------------------------------------------------------- inputs


def _np_dtype(bits):
    return np.uint8 if bits == 8 else np.uint16


def _image(case, seed):
    """The case's input image on the GPU: drawn on the host as the repository's
    workloads are, the large blob images on the GPU."""
    h, w, dt = case["h"], case["w"], _np_dtype(case["bits"])
    if case["kind"] == "ridges":
        return torch.from_numpy(synth.gen_ridges(h, w, seed, dt)).cuda()
    sigma = case.get("sigma", (4.0, 16.0))
    if h * w > 1 << 18:
        return synth.gen_blobs_device(h, w, seed, dt, sigma=sigma)
    return torch.from_numpy(synth.gen_blobs(h, w, seed, dt, sigma=sigma)).cuda()


def _plan(case):
    """Sizes and options of a batch's images: (h, w, bits, lam, adj, op, pitch)."""
    rng = np.random.default_rng(case["plan"])
    lo, hi = math.log(case["lo"]), math.log(case["hi"])
    rows = []
    for _ in range(case["n"]):
        h = int(np.rint(math.exp(rng.uniform(lo, hi))))
        w = int(np.rint(math.exp(rng.uniform(lo, hi))))
        if case["path"] == "serving":
            bits = 8 if rng.random() < 0.5 else 16
            rows.append((h, w, bits, int(rng.integers(0, 51)), "8,4", "leveling", w))
            continue
        lam = int(rng.choice([0, 5, 20, 50]))
        bits, adj, op = 8, "8,4", "leveling"
        if case["u16"] and rng.random() < 0.5:
            bits, lam = 16, lam * 10
        if case["mixed"]:
            adj = "8,4" if rng.random() < 0.5 else "4,8"
            op = "leveling" if rng.random() < 0.5 else "skeleton"
        pitch = w + int(rng.integers(1, 64)) if case["pitched"] and rng.random() < 0.5 else w
        rows.append((h, w, bits, lam, adj, op, pitch))
    return rows


def _flat_views(plan, flat):
    """Views of the plan's images inside one flat byte buffer, each image at a
    256-byte boundary."""
    out, off = [], 0
    for h, w, bits, _, _, _, pitch in plan:
        b = bits // 8
        part = flat[off:off + h * pitch * b]
        if bits == 16:
            part = part.view(torch.uint16)
        out.append(part.view(h, pitch)[:, :w])
        off += (h * pitch * b + 255) // 256 * 256
    return out


def _flat_bytes(plan):
    return sum((h * p * (b // 8) + 255) // 256 * 256 for h, _, b, _, _, _, p in plan)


def prepare(case, seed):
    state = {"case": case}
    path = case["path"]
    if path == "serving":
        plan = _plan(case)
        host_in = torch.zeros(_flat_bytes(plan), dtype=torch.uint8, pin_memory=True)
        host_out = torch.zeros(_flat_bytes(plan), dtype=torch.uint8, pin_memory=True)
        reqs = []
        for i, (row, src, out) in enumerate(zip(plan, _flat_views(plan, host_in),
                                                _flat_views(plan, host_out))):
            h, w, bits, lam, adj = row[:5]
            img = synth.gen_blobs_device(h, w, seed * 1000 + i, _np_dtype(bits))
            src.copy_(img)
            reqs.append(serve.Request(tag=i, image=img, lam=lam, adj=adj, host_in=src, host_out=out))
        state.update(reqs=reqs, out=host_out, copy_stream=torch.cuda.Stream(), ctx=thin.Context())
    elif path == "batch":
        plan = _plan(case)
        src = torch.zeros(_flat_bytes(plan), dtype=torch.uint8, device="cuda")
        for i, (view, row) in enumerate(zip(_flat_views(plan, src), plan)):
            view.copy_(synth.gen_blobs_device(row[0], row[1], seed * 1000 + i, _np_dtype(row[2])))
        work = torch.empty_like(src)
        state.update(src=src, work=work, views=_flat_views(plan, work), lams=[r[3] for r in plan],
                     adjs=[r[4] for r in plan], ops=[r[5] for r in plan], ctx=thin.Context())
    else:
        src = _image(case, seed)
        state.update(src=src, work=torch.empty_like(src), ctx=thin.Context())
        if path == "gradient":
            dt = torch.uint8 if case["out_bits"] == 8 else torch.uint16
            state["work"] = torch.empty(src.shape, dtype=dt, device="cuda")
            state["mag"] = torch.empty(src.shape, dtype=torch.float32, device="cuda")
    torch.cuda.synchronize()
    return state


# -------------------------------------------------------------------- passes


def _pixels(t):
    """The image's values; 16-bit ones as int16 (the same bytes), which more
    of torch's operators take."""
    return t.view(torch.int16) if t.dtype == torch.uint16 else t


def _counts(stats):
    return np.array([[s.passes, s.lowerings, int(s.converged)] for s in stats], dtype=np.int64)


def run(state):
    case, ctx = state["case"], state["ctx"]
    path = case["path"]
    if path == "serving":
        rep = serve.replay(ctx, state["reqs"], copy_stream=state["copy_stream"])
        return {"images": state["out"],
                "counts": _counts([rep.stats[r.tag] for r in state["reqs"]])}
    if path == "batch":
        state["work"].copy_(state["src"])
        st = ctx.run_batch(state["views"], state["lams"], state["adjs"], ops=state["ops"])
        return {"images": state["work"], "counts": _counts(st)}
    if path == "gradient":
        ctx.gradient(state["src"], state["work"], case["alpha"], case["gain"],
                     magnitude=state["mag"])
        return {"magnitude": state["mag"], "image": _pixels(state["work"])}
    work = state["work"]
    if path == "pipeline":
        ctx.gradient(state["src"], work, case["alpha"], case["gain"])
        st = ctx.run(work, case["lam"], case["adj"], op=case["op"])
        return {"image": work, "counts": _counts([st])}
    work.copy_(state["src"])
    if path == "noalloc":
        raw = thin.thin_stats()
        rc = thin.thin_run_noalloc(ctx.handle, work.data_ptr(), case["h"], case["w"],
                                   thin.THIN_U8 if case["bits"] == 8 else thin.THIN_U16,
                                   case["lam"],
                                   thin.THIN_ADJ_8_4 if case["adj"] == "8,4" else thin.THIN_ADJ_4_8,
                                   raw)
        if rc != thin.THIN_OK:
            raise thin.ThinError(rc, thin.thin_last_error(ctx.handle))
        st = thin.Stats.of(raw)
    else:
        st = ctx.run(work, case["lam"], case["adj"], op=case["op"])
    return {"image": _pixels(work), "counts": _counts([st])}


# ------------------------------------------------------------- what it takes


def work(case):
    """Each input pixel read once and each output written once; operations:
    one characterisation of every pixel (40 integer operations: 8 compares,
    a lookup, the lambda test, the maximum over the lower neighbours) and, for
    the gradient, its eight recursions (5 products and sums on average), the
    sums of their halves and the magnitude."""
    path = case["path"]
    if path in ("batch", "serving"):
        plan = _plan(case)
        return {"bytes": sum(2 * h * w * (b // 8) for h, w, b, *_ in plan),
                "flops": sum(40 * h * w for h, w, *_ in plan)}
    px, b = case["h"] * case["w"], case["bits"] // 8
    if path == "gradient":
        return {"bytes": px * (b + case["out_bits"] // 8 + 4), "flops": 50 * px}
    if path == "pipeline":
        return {"bytes": px * (b + 1), "flops": 90 * px}
    return {"bytes": 2 * px * b, "flops": 40 * px}


def _recursion(x, a0, a1, b1, b2, start):
    """y[n] = a0 x[n] + a1 x[n-1] + b1 y[n-1] + b2 y[n-2] down the rows, from
    the steady state of x extended by its first row."""
    y = np.empty_like(x)
    prev, y1 = x[0], x[0] * start
    y2 = y1
    for n in range(x.shape[0]):
        y[n] = a0 * x[n] + a1 * prev + b1 * y1 + b2 * y2
        prev, y2, y1 = x[n], y1, y[n]
    return y


def _smooth_and_derive(x, alpha):
    """Deriche's smoothing and derivative along the rows' direction in float64."""
    r = math.exp(-alpha)
    k = (1 - r) ** 2 / (1 + 2 * alpha * r - r * r)
    c = (1 - r) ** 3 / (2 * r * (1 + r))
    b1, b2 = 2 * r, -r * r
    den = 1 - b1 - b2
    late = np.concatenate([x[1:], x[-1:]])[::-1].copy()     # x[n + 1], last row first
    early = np.concatenate([x[:1], x[:-1]])                 # x[n - 1]
    a0, a1, a2, a3 = k, k * (alpha - 1) * r, k * (alpha + 1) * r, -k * r * r
    smooth = _recursion(x, a0, a1, b1, b2, (a0 + a1) / den)
    smooth += _recursion(late, a2, a3, b1, b2, (a2 + a3) / den)[::-1]
    derive = _recursion(early, -c * r, 0.0, b1, b2, -c * r / den)
    derive += _recursion(late, c * r, 0.0, b1, b2, c * r / den)[::-1]
    return smooth, derive


def exact(case, seed):
    """The gradient's magnitude in float64; the thinned images and stored
    values are whole numbers with nothing to be off by."""
    if case["path"] != "gradient":
        return None
    x = _image(case, seed).cpu().numpy().astype(np.float64)
    fi, gi = _smooth_and_derive(x, float(np.float32(case["alpha"])))
    _, gx = _smooth_and_derive(np.ascontiguousarray(fi.T), float(np.float32(case["alpha"])))
    gy, _ = _smooth_and_derive(np.ascontiguousarray(gi.T), float(np.float32(case["alpha"])))
    return {"magnitude": np.ascontiguousarray(np.hypot(gx, gy).T), "image": None}
