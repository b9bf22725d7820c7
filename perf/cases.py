"""The calls that users of the package make, as cases to time.

A case names an operation, the detector frames it works on and the coding options:

  op        one-compress    rsz.compress on one frame (buffers kept by the caller)
            one-decompress  rsz.decompress on one stream
            compress        rsz.Batch.run: a batch planned and compressed in one call
            graph           rsz.Batch.replay: a batch prepared once, replayed as a HIP graph
            decompress      rsz.rsz_decompress_batch: many streams in one call
            peaks           rsz.PeakBatch.run: peak finding over a batch
            verify          rsz.Verify.replay: compression and on-device verification, one graph
  kind      cspad     N(0, 2^2) noise + a smooth water ring
            jungfrau  40 ADU x Poisson(0.3) photons + N(0, 3^2) read noise
            mix       CSPAD, Jungfrau-4M and 1 x 2048 x 2048 frames in turn
  panels, height, width, frames; peaks: mean Bragg peaks per frame (a fifth of a batch's
  frames are non-hits); window, bin, mode, eb, dim, roi, run: the coding parameters.
"""
import math
import zlib

import numpy as np
import torch

from paper_2206_11297_amd import rsz

CSPAD = (32, 185, 388)
JUNGFRAU4M = (8, 512, 1024)
JUNGFRAU16M = (16, 512, 1024)
SQUARE4M = (1, 2048, 2048)
MIX = (("cspad", CSPAD), ("jungfrau", JUNGFRAU4M), ("jungfrau", SQUARE4M))
MIX_EB = (5.0, 10.0, 20.0)


def _case(op, kind, shape, frames, peaks, window=17, bin=2, eb=10.0, mode=0, dim=2, roi=0, run=0):
    P, H, W = shape
    return {"op": op, "kind": kind, "panels": P, "height": H, "width": W, "frames": frames,
            "peaks": peaks, "window": window, "bin": bin, "eb": eb, "mode": mode, "dim": dim,
            "roi": roi, "run": run}


def listed():
    return [
        # one frame as it leaves the detector: the smallest call, launches and latency
        dict(_case("one-compress", "cspad", CSPAD, 1, 60), name="one-compress"),
        # one stream read back by a viewer
        dict(_case("one-decompress", "cspad", CSPAD, 1, 60), name="one-decompress"),
        # what a serving slot holds: a few frames of several detectors and bounds
        dict(_case("compress", "mix", CSPAD, 24, 200), name="serve-mix"),
        # a run's frames at the published working point: the largest ordinary batch
        dict(_case("compress", "cspad", CSPAD, 1000, 60), name="cspad-batch"),
        # panels of odd size with a bin that divides neither side (vectors do not fit)
        dict(_case("compress", "cspad", (5, 187, 389), 200, 40, window=11, bin=3, eb=5.0),
             name="ragged-b3"),
        # a 16-Mpixel detector at a tight bound, prepared once and replayed
        dict(_case("graph", "jungfrau", JUNGFRAU16M, 64, 300, eb=1.0), name="jungfrau16m-graph"),
        # the 3D predictor with both lossless stages: the smallest streams
        dict(_case("compress", "cspad", CSPAD, 250, 60, dim=3, roi=1, run=1), name="coded-3d"),
        # an analysis reading a whole run back
        dict(_case("decompress", "cspad", CSPAD, 1000, 60), name="cspad-decode"),
        # the same for panels of half a megapixel
        dict(_case("decompress", "jungfrau", JUNGFRAU4M, 128, 120, window=11),
             name="jungfrau4m-decode"),
        # streams of the 3D predictor with both lossless stages read back
        dict(_case("decompress", "cspad", CSPAD, 250, 60, dim=3, roi=1, run=1),
             name="coded-3d-decode"),
        # Bragg peaks of a run found before it is compressed
        dict(_case("peaks", "cspad", CSPAD, 1000, 60), name="peaks"),
        # every stream decoded and checked on the device behind its compression
        dict(_case("verify", "jungfrau", JUNGFRAU4M, 48, 120), name="verify"),
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["one-compress", "one-decompress", "compress", "compress", "compress",
                     "graph", "decompress", "decompress", "decompress", "peaks", "verify"])
    kind = rng.choice(["cspad", "jungfrau"])
    shape = rng.choice([CSPAD, JUNGFRAU4M, JUNGFRAU16M, SQUARE4M, None, None, None, None])
    if shape is None:   # any detector, odd sizes among them
        shape = (_logint(rng, 1, 32), _logint(rng, 48, 1100), _logint(rng, 48, 1100))
    pix = shape[0] * shape[1] * shape[2]
    frames = 1
    if not op.startswith("one"):
        frames = max(1, min(1000, int(_logint(rng, 1 << 20, 300 << 20) / pix)))
        if op == "verify":
            frames = min(frames, 48)
    # at most a tenth of a frame's pixels in windows
    window = rng.choice([7, 11, 17, 25])
    most = max(1, int(0.1 * pix / window ** 2))
    peaks = min(most, _logint(rng, 4, 800))
    coded = op in ("one-compress", "one-decompress", "compress", "decompress")
    return _case(op, kind, shape, frames, peaks, window=window,
                 bin=rng.choice([1, 2, 2, 2, 3, 4, 4, 5, 8]),
                 eb=rng.choice([1.0, 2.0, 5.0, 10.0, 20.0]),
                 mode=rng.choice([0, 0, 0, 1]), dim=rng.choice([1, 2, 2, 3]),
                 roi=rng.choice([0, 1]) if coded else 0, run=rng.choice([0, 1]) if coded else 0)


# ----------------------------------------------------------------- inputs


def _groups(case):
    """(kind, shape, eb, frames) of the case's frames, in order of their groups."""
    if case["kind"] != "mix":
        shape = (case["panels"], case["height"], case["width"])
        return [(case["kind"], shape, case["eb"], case["frames"])]
    n = case["frames"]
    return [(kind, shape, MIX_EB[g], n // 3 + (g < n % 3)) for g, (kind, shape) in enumerate(MIX)]


def _peak_counts(case, group, n):
    """Peaks per frame: Poisson, a fifth of the frames non-hits.  They depend on the case
    alone, so that the sizes of its buffers do."""
    text = "%s %s" % (sorted((k, v) for k, v in case.items() if k != "name"), group)
    rng = np.random.default_rng(zlib.crc32(text.encode()))
    if n == 1:
        return np.full(1, case["peaks"])
    counts = rng.poisson(case["peaks"], n)
    counts[rng.permutation(n)[: n // 5]] = 0
    return counts


def _ring(shape, device):
    P, H, W = shape
    cols = 4 if P % 4 == 0 else (2 if P % 2 == 0 else 1)
    cy, cx = P // cols * H / 2.0, cols * W / 2.0
    p = torch.arange(P, device=device)
    y = (p // cols * H)[:, None] + torch.arange(H, device=device)[None, :] - cy
    x = (p % cols * W)[:, None] + torch.arange(W, device=device)[None, :] - cx
    rho = torch.sqrt(y.double()[:, :, None] ** 2 + x.double()[:, None, :] ** 2)
    return (40.0 * torch.exp(-(rho - 300.0) ** 2 / (2 * 30.0 ** 2))).float()


def _frames(kind, shape, counts, seed, group, device):
    """Frames float32 [n, stride] (stride: the frame's pixels up to whole 16 bytes), the
    peaks int32 [total, 3] and their starts."""
    P, H, W = shape
    n, pix = len(counts), P * H * W
    stride = (pix + 3) // 4 * 4
    rng = np.random.default_rng([int(seed), group])
    gen = torch.Generator(device=device)
    gen.manual_seed(int(rng.integers(1 << 62)))
    total = int(counts.sum())
    at = np.concatenate([[0], np.cumsum(counts)])
    pk = np.stack([rng.integers(0, P, total), rng.integers(0, H, total),
                   rng.integers(0, W, total)], axis=1).astype(np.int32)
    sig = rng.uniform(0.8, 1.5, total)
    amp = np.exp(rng.uniform(math.log(200.0), math.log(5000.0), total))
    sig, amp, peaks = (torch.from_numpy(v).to(device) for v in (sig, amp, pk))
    x = torch.randn((n, stride), generator=gen, device=device)
    x *= 2.0 if kind == "cspad" else 3.0
    ring = _ring(shape, device).reshape(1, pix) if kind == "cspad" else None
    d = torch.arange(-8, 9, device=device)
    step = max(1, (64 << 20) // pix)
    for f0 in range(0, n, step):
        f1 = min(f0 + step, n)
        body = x[f0:f1, :pix]
        if ring is not None:
            body += ring
        else:
            body += 40.0 * torch.poisson(torch.full_like(body, 0.3), generator=gen)
        k0, k1 = int(at[f0]), int(at[f1])
        if k1 > k0:   # Gaussian spots; where two meet, the higher one
            f = torch.from_numpy(np.repeat(np.arange(f1 - f0), counts[f0:f1])).to(device)
            p, i, j = (peaks[k0:k1, c].long() for c in range(3))
            u, v = i[:, None] + d, j[:, None] + d
            e = torch.exp(-d.double()[None, :] ** 2 / (2.0 * sig[k0:k1, None] ** 2))
            spot = (amp[k0:k1, None, None] * e[:, :, None] * e[:, None, :]).float()
            inside = ((u >= 0) & (u < H))[:, :, None] & ((v >= 0) & (v < W))[:, None, :]
            to = ((f * P + p)[:, None, None] * H + u[:, :, None]) * W + v[:, None, :]
            spots = torch.zeros((f1 - f0) * pix, device=device)
            spots.scatter_reduce_(0, to[inside], spot[inside], "amax")
            body += spots.view(f1 - f0, pix)
    x[:, pix:] = 0.0
    return x, peaks, at


def _inputs(case, seed, device="cuda"):
    """Per frame: its [P, H, W] view, its peaks and its eb; the group's whole tensors beside."""
    frames, peaks, ebs, whole = [], [], [], []
    for g, (kind, shape, eb, n) in enumerate(_groups(case)):
        counts = _peak_counts(case, g, n)
        x, pk, at = _frames(kind, shape, counts, seed, g, device)
        P, H, W = shape
        for f in range(n):
            frames.append(x[f, :P * H * W].view(P, H, W))
            peaks.append(pk[int(at[f]):int(at[f + 1])])
            ebs.append(eb)
        whole.append((shape, eb, x, pk, counts))
    return frames, peaks, ebs, whole


# ---------------------------------------------------------- prepare and run


def _tuple(case, eb):
    return (case["window"], case["bin"], eb, case["mode"], case["dim"], case["roi"], case["run"])


def _batch(case, seed):
    frames, peaks, ebs, _ = _inputs(case, seed)
    B = rsz.Batch(frames, peaks, [_tuple(case, eb) for eb in ebs])
    B.out.zero_()   # the bytes between the streams are nobody's
    return B


def _streams(case, seed):
    """The compressed streams of the case's frames, packed, and their places."""
    B = _batch(case, seed)
    B.run()
    sizes = B.sizes.cpu().tolist()
    if int(B.status.abs().max()):
        raise RuntimeError("a frame did not compress")
    at = [0]
    for s in sizes:
        at.append(at[-1] + (s + 255) // 256 * 256)
    packed = torch.zeros(at[-1], dtype=torch.uint8, device="cuda")
    for i, s in enumerate(sizes):
        packed[at[i]:at[i] + s] = B.stream(i, sizes)
    return packed, at, sizes


def prepare(case, seed):
    op = case["op"]
    if op == "one-compress":
        frames, peaks, ebs, _ = _inputs(case, seed)
        B = rsz.Batch(frames, peaks, _tuple(case, case["eb"]))   # sizes the caller's buffers
        ws = rsz.workspace(B.ws.numel() + 4096)
        return {"op": op, "frame": frames[0], "peaks": peaks[0], "out": torch.zeros_like(B.out),
                "ws": ws, "options": dict(window=case["window"], bin=case["bin"], eb=case["eb"],
                                          bin_mode=case["mode"], dim=case["dim"],
                                          roi_coding=case["roi"], run_coding=case["run"])}
    if op == "one-decompress":
        packed, at, sizes = _streams(case, seed)
        head = packed[:80].cpu().numpy().tobytes()
        st, need = rsz.rsz_decompress_workspace_bytes(head)
        return {"op": op, "stream": packed[:sizes[0]], "ws": rsz.workspace(need)}
    if op == "compress":
        return {"op": op, "batch": _batch(case, seed)}
    if op == "graph":
        B = _batch(case, seed)
        B.prepare()
        B.graph()
        return {"op": op, "batch": B}
    if op == "verify":
        B = _batch(case, seed)
        B.prepare()
        V = rsz.Verify(B)
        V.graph()
        return {"op": op, "batch": B, "verify": V}
    if op == "peaks":
        frames, _, _, _ = _inputs(case, seed)
        return {"op": op, "batch": rsz.PeakBatch(frames)}
    if op == "decompress":
        packed, at, sizes = _streams(case, seed)
        n, pix = len(sizes), case["panels"] * case["height"] * case["width"]
        out = torch.zeros((n, (pix + 3) // 4 * 4), dtype=torch.float32, device="cuda")
        heads = [packed[at[i]:at[i] + 80] for i in range(n)]
        heads = torch.stack(heads).cpu().numpy().copy()
        descs = (rsz.rsz_decode_desc * n)()
        for i in range(n):
            descs[i] = rsz.rsz_decode_desc(packed.data_ptr() + at[i], sizes[i],
                                           heads.ctypes.data + 80 * i, out[i].data_ptr(), pix)
        st, need = rsz.rsz_decompress_batch_workspace_bytes(descs)
        status = torch.zeros(n, dtype=torch.int32, device="cuda")
        return {"op": op, "descs": descs, "heads": heads, "packed": packed, "out": out,
                "status": status, "ws": rsz.workspace(need)}
    raise ValueError(op)


def run(state):
    op = state["op"]
    if op == "one-compress":
        stream = rsz.compress(state["frame"], state["peaks"], out=state["out"], ws=state["ws"],
                              **state["options"])
        return {"out": state["out"], "bytes": stream.numel()}
    if op == "one-decompress":
        return {"frame": rsz.decompress(state["stream"], ws=state["ws"])}
    if op == "decompress":
        s = state
        st = rsz.rsz_decompress_batch(s["descs"], s["status"].data_ptr(), s["ws"].data_ptr(),
                                      s["ws"].numel(), torch.cuda.current_stream().cuda_stream)
        if st:
            raise rsz.RszError(st, "rsz_decompress_batch")
        return {"frames": s["out"], "status": s["status"]}
    B = state["batch"]
    if op == "peaks":
        B.run()
        return {"peaks": B.out, "counts": B.counts, "status": B.status}
    if op == "verify":
        state["verify"].replay()
        return {"out": B.out, "sizes": B.sizes, "status": B.status,
                "bad": state["verify"].bad, "frames": state["verify"].frames}
    if op == "graph":
        B.replay()
    else:
        B.run()
    return {"out": B.out, "sizes": B.sizes, "status": B.status}


# ------------------------------------------------------------ exact and work


def _restored(shape, eb, x, pk, counts, window, b, mode, dtype=torch.float64):
    """What a stream restores, in float64: the window pixels as they are, elsewhere the
    bin mean of the pixels outside the windows (mode 1: of all) to the nearest 2 eb."""
    P, H, W = shape
    n, pix = len(counts), P * H * W
    Hb, Wb, h = -(-H // b), -(-W // b), window // 2
    dev = x.device
    out = torch.zeros(x.shape, dtype=dtype, device=dev)
    starts = np.concatenate([[0], np.cumsum(counts)])
    step = max(1, (16 << 20) // pix)
    for f0 in range(0, n, step):
        f1 = min(f0 + step, n)
        m = f1 - f0
        f = torch.from_numpy(np.repeat(np.arange(m), counts[f0:f1])).to(dev)
        p, i, j = (pk[int(starts[f0]):int(starts[f1]), c].long() for c in range(3))
        # windows by the corners of their rectangles, summed along both axes
        edge = torch.zeros((m * P, H + 1, W + 1), dtype=torch.int32, device=dev)
        r0, r1 = (i - h).clamp(min=0), (i - h + window).clamp(max=H)
        c0, c1 = (j - h).clamp(min=0), (j - h + window).clamp(max=W)
        for r, c, s in ((r0, c0, 1), (r0, c1, -1), (r1, c0, -1), (r1, c1, 1)):
            to = ((f * P + p) * (H + 1) + r) * (W + 1) + c
            edge.view(-1).index_add_(0, to, torch.full_like(to, s, dtype=torch.int32))
        roi = (edge.cumsum(1).cumsum(2) > 0)[:, :H, :W]
        y = x[f0:f1, :pix].reshape(m * P, H, W).double()
        pad = (0, Wb * b - W, 0, Hb * b - H)
        yp = torch.nn.functional.pad(y, pad)
        inc = torch.ones_like(roi) if mode else ~roi
        inc = torch.nn.functional.pad(inc, pad)
        S = torch.zeros((m * P, Hb, Wb), dtype=torch.float64, device=dev)
        k = torch.zeros_like(S)
        for di in range(b):
            for dj in range(b):
                on = inc[:, di::b, dj::b]
                S = torch.where(on, S + yp[:, di::b, dj::b], S)
                k += on
        q = torch.where(k > 0, torch.round(S / (k.clamp(min=1) * (2.0 * eb))), 0.0)
        v = (q * (2.0 * eb)).repeat_interleave(b, 1).repeat_interleave(b, 2)[:, :H, :W]
        out[f0:f1, :pix] = torch.where(roi, y, v).reshape(m, pix)
    return out


def exact(case, seed):
    op = case["op"]
    if op not in ("one-decompress", "decompress", "verify"):
        return None   # streams and peak lists: bytes and whole numbers
    _, _, _, whole = _inputs(case, seed)
    shape, eb, x, pk, counts = whole[0]
    y = _restored(shape, eb, x, pk, counts, case["window"], case["bin"], case["mode"])
    P, H, W = shape
    if op == "decompress":
        return {"frames": y, "status": None}
    frames = [y[f, :P * H * W].view(P, H, W) for f in range(len(counts))]
    if op == "one-decompress":
        return {"frame": frames[0]}
    return {"out": None, "sizes": None, "status": None, "bad": None, "frames": frames}


def work(case):
    """Bytes: the pixels once and the streams once (decoding: the other way round; verifying:
    the pixels read, the decoded frames written).  A stream holds its windows and at least
    the entropy of its bins' codes, a Gaussian's here."""
    pixels = windows = bins = stream = 0.0
    for g, (kind, shape, eb, n) in enumerate(_groups(case)):
        P, H, W = shape
        b = case["bin"]
        counts = _peak_counts(case, g, n)
        pixels += float(n) * P * H * W
        windows += float(counts.sum()) * case["window"] ** 2
        nb = float(n) * P * -(-H // b) * -(-W // b)
        noise = 2.0 if kind == "cspad" else math.sqrt(0.3 * 40.0 ** 2 + 9.0)
        sigma = 2.0 * noise / b / (2.0 * eb)   # of the difference of four bins' codes
        bits = max(0.1 if case["run"] else 1.0, math.log2(sigma * math.sqrt(2 * math.pi * math.e)))
        bins += nb
        stream += nb * bits / 8 + 1104.0 * n
    stream += 4.0 * windows * (0.9 if case["roi"] else 1.0)
    if case["op"] == "peaks":
        return {"bytes": 4.0 * pixels, "flops": pixels}
    if case["op"] == "verify":
        return {"bytes": 8.0 * pixels + stream, "flops": 4.0 * pixels}
    return {"bytes": 4.0 * pixels + stream, "flops": pixels + 4.0 * bins}
