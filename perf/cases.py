"""The workloads this repository's speed is measured on.

``listed()`` names twelve of them and ``draw()`` gives more of the same ranges.
Every case is a dict of plain values with a ``kind``:

  pair     one eager call of ``iqa_tiles``, ``lisi_tiles`` or ``auglisi_tiles``
           on one image pair, outputs allocated by the call
  stream   a program that follows a field: a fixed ring of image pairs and
           output buffers, its calls captured once into a HIP graph; a pass is
           one replay over the whole ring
  pyramid  ``pyramid`` and the whole-image value from its finest level's sums
  merge    ``merge_tiles`` on the sums of an earlier pass
  batch    a planned ``Batch`` of many pairs, run once
  serve    a resident-reference ``Server``: a burst of requests, submitted,
           drained and polled

Images are beam-convolved point sources on Gaussian noise, the second one
without the faintest sources and with noise of its own; ``blanks`` sets the
pixels outside the inscribed circle to NaN, as primary-beam-cut images have.
"""

from __future__ import annotations

import math
import random

import torch

from paper_2501_10653_amd import auglisi_tiles, iqa_tiles, lisi_tiles, merge_tiles, pyramid
from paper_2501_10653_amd.batch import Batch
from paper_2501_10653_amd.serve import Server

CONST = 1e-6            # C1, C2 and C of every call; D is the default C1/2
NOISE = 1e-4
SIGMA = 4.0 / 2.3548    # beam of 4 pixels FWHM


# ---------------------------------------------------------------------------
# The cases
# ---------------------------------------------------------------------------

def listed():
    return [
        # The smallest call of the benchmark: one 8 x 8 IQA matrix; latency.
        dict(name="pair_256_nt32", kind="pair", N=256, NT=32, which="both", sums=False,
             blanks=False),
        # Snapshot imaging at a low resolution: launches of a few microseconds.
        dict(name="stream_1024_nt32", kind="stream", N=1024, NT=32, pairs=16, which="both",
             blanks=False),
        # The paper's shape (2048^2 with 64^2 tiles), the headline of the benchmark.
        dict(name="stream_2048_nt64", kind="stream", N=2048, NT=64, pairs=12, which="both",
             blanks=False),
        # The same images with few large tiles (the sweep's coarsest column).
        dict(name="stream_2048_nt256", kind="stream", N=2048, NT=256, pairs=12, which="both",
             blanks=False),
        # A round decimal image size with decimal tiles, primary-beam cut.
        dict(name="stream_3000_nt100", kind="stream", N=3000, NT=100, pairs=6, which="both",
             blanks=True),
        # An odd image side (a central pixel) with odd tiles: no row is aligned.
        dict(name="stream_2025_nt45", kind="stream", N=2025, NT=45, pairs=12, which="both",
             blanks=False),
        # The paper's two separate kernels, at a tile side that is no multiple of 4.
        dict(name="separate_2000_nt50", kind="stream", N=2000, NT=50, pairs=8, which="separate",
             blanks=False),
        # The largest image of the sweep with its finest tiles, sums exported.
        dict(name="pair_8192_nt16_sums", kind="pair", N=8192, NT=16, which="both", sums=True,
             blanks=False),
        # A coarse look at a large image: 4 x 4 tiles.
        dict(name="stream_4096_nt1024", kind="stream", N=4096, NT=1024, pairs=4, which="both",
             blanks=False),
        # All scales of one pair (20, 40, ..., 1280 pixels) and the whole-image value.
        dict(name="pyramid_3840_nt20", kind="pyramid", N=3840, NT=20),
        # A night's snapshots of mixed fields in one launch (the ragged recipe).
        dict(name="batch_ragged_30", kind="batch", mix="ragged", count=30, pick=7),
        # A burst of requests against resident references (the serving recipe).
        dict(name="serve_24", kind="serve", refs=16, requests=24, pick=11),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


_ODD_NT = (9, 10, 15, 18, 21, 25, 27, 30, 33, 45, 50, 54, 63, 75, 90, 125, 150, 225)
_EVEN_NT = (8, 12, 16, 20, 24, 32, 40, 48, 60, 64, 80, 96, 100, 120, 128, 160, 192, 200, 256, 300)
_WIDE_NT = (320, 384, 400, 500, 512, 640, 750, 768, 1000, 1024, 1500, 2048)


def _shape(rng, lo, hi):
    """An image side of about lo..hi (spread over its logarithm) and a tile side that divides it."""
    N = _log_int(rng, lo, hi)
    kinds = rng.random()
    nts = _ODD_NT if kinds < 0.3 else _EVEN_NT if kinds < 0.85 or N < 1500 else _WIDE_NT
    NT = rng.choice([v for v in nts if v <= max(16, N // 2)])
    return NT * max(1, int(N / NT)), NT


def draw(rng):
    kind = rng.choice(["pair", "stream", "stream", "stream", "pyramid", "merge", "batch", "serve"])
    if kind == "pair":
        N, NT = _shape(rng, 96, 8192)
        which = rng.choice(["both", "both", "lisi", "auglisi"])
        return dict(kind=kind, N=N, NT=NT, which=which, sums=which == "both" and rng.random() < 0.5,
                    blanks=rng.random() < 0.3)
    if kind == "stream":
        N, NT = _shape(rng, 200, 6000)
        pairs = max(2, min(16, int(4.5e8 / (8 * N * N))))
        return dict(kind=kind, N=N, NT=NT, pairs=pairs,
                    which=rng.choice(["both", "both", "separate"]), blanks=rng.random() < 0.3)
    if kind == "pyramid":
        NT = rng.choice([8, 10, 16, 20, 24, 25, 32, 45, 48, 64])
        ns = rng.choice([1, 3, 5, 7]) << rng.randint(2, 7)
        while NT * ns > 5000:
            ns //= 2
        return dict(kind=kind, N=NT * ns, NT=NT)
    if kind == "merge":
        f = rng.choice([2, 3, 4, 5, 8, 10, 16, 25, 64, 100])
        np_ = max(1, int(_log_int(rng, 8, 512) / f))
        return dict(kind=kind, ns=f * np_, f=rng.choice([f, f * np_]))
    if kind == "batch":
        return dict(kind=kind, mix=rng.choice(["ragged", "small", "odd"]),
                    count=rng.randint(3, 30), pick=rng.randrange(10000))
    case = dict(kind=kind, refs=rng.randint(2, 16), requests=rng.randint(1, 24),
                pick=rng.randrange(10000))
    while work(case)["bytes"] > 1.2e9:
        case["requests"] -= 1
    return case


# ---------------------------------------------------------------------------
# Sizes inside a case
# ---------------------------------------------------------------------------

def _batch_shapes(case):
    r = random.Random("batch %s %d" % (case["mix"], case["pick"]))
    out = []
    for _ in range(case["count"]):
        if case["mix"] == "ragged":
            out.append((r.choice((512, 1024, 2048, 4096)), r.choice((32, 64, 128))))
        elif case["mix"] == "small":
            out.append((256, 32))
        else:   # cut-outs of any size, some with tiles the vector loads do not divide
            NT = r.choice((10, 12, 20, 25, 30, 45, 48, 50, 60, 100))
            out.append((NT * max(1, int(math.exp(r.uniform(math.log(200), math.log(2200))) / NT)),
                        NT))
    return out


def _serve_shapes(case):
    r = random.Random("serve %d" % case["pick"])
    refs = [(1024, 2048, 4096)[i % 3] for i in range(case["refs"])]
    return refs, [(r.randrange(case["refs"]), r.choice((32, 64))) for _ in range(case["requests"])]


def _pair_work(N, NT, outs=2):
    tiles = (N // NT) ** 2
    return 8 * N * N + 4 * outs * tiles, 12 * N * N


def work(case):
    kind = case["kind"]
    if kind == "pair":
        b, f = _pair_work(case["N"], case["NT"],
                          (2 if case["which"] == "both" else 1) + (4 if case["sums"] else 0))
    elif kind == "stream":
        b, f = (case["pairs"] * v for v in _pair_work(case["N"], case["NT"]))
        if case["which"] == "separate":   # two calls, each of which has to read both images
            b, f = b + case["pairs"] * 8 * case["N"] ** 2, f
    elif kind == "pyramid":
        b, f = _pair_work(case["N"], case["NT"], 6)
        ns = case["N"] // case["NT"]
        while ns % 2 == 0:
            ns //= 2
            b, f = b + 24 * ns * ns, f + 16 * ns * ns
        b += 24
    elif kind == "merge":
        b, f = 16 * case["ns"] ** 2 + 24 * (case["ns"] // case["f"]) ** 2, 4 * case["ns"] ** 2
    elif kind == "batch":
        b, f = (sum(v) for v in zip(*(_pair_work(N, NT) for N, NT in _batch_shapes(case))))
    else:
        refs, reqs = _serve_shapes(case)
        b, f = (sum(v) for v in zip(*(_pair_work(refs[r], NT) for r, NT in reqs)))
    return {"bytes": b, "flops": f}


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------

class _Sky:
    """Image pairs from a seed: every call draws the next pair."""

    def __init__(self, seed):
        self.host = random.Random("sky %d" % seed)
        self.gen = torch.Generator(device="cuda").manual_seed(seed)

    def _image(self, N, sources, blanks):
        img = torch.randn(N, N, device="cuda", generator=self.gen) * NOISE
        if sources:
            rc = torch.tensor(sources, dtype=torch.float64, device="cuda")
            rad = 11   # about 6 sigma of the beam
            k = torch.arange(-rad, rad + 1, device="cuda")
            rows = rc[:, 0].round().long()[:, None] + k
            cols = rc[:, 1].round().long()[:, None] + k
            gr = torch.exp(-(rows - rc[:, :1]) ** 2 / (2 * SIGMA ** 2))
            gc = torch.exp(-(cols - rc[:, 1:2]) ** 2 / (2 * SIGMA ** 2))
            val = (rc[:, 2, None, None] * gr[:, :, None] * gc[:, None, :]).float()
            r = rows[:, :, None].expand(val.shape).reshape(-1)
            c = cols[:, None, :].expand(val.shape).reshape(-1)
            inside = (r >= 0) & (r < N) & (c >= 0) & (c < N)
            img.view(-1).index_put_(((r * N + c)[inside],), val.reshape(-1)[inside],
                                    accumulate=True)
        if blanks:
            d = (torch.arange(N, device="cuda", dtype=torch.float32) - (N - 1) / 2) ** 2
            img[d[:, None] + d[None, :] > (N / 2) ** 2] = float("nan")
        return img

    def pair(self, N, blanks=False):
        n = max(3, round(33 * (N / 2048) ** 2))
        src = sorted(((self.host.uniform(0, N - 1), self.host.uniform(0, N - 1),
                       math.exp(self.host.uniform(math.log(1e-3), math.log(2.0))))
                      for _ in range(n)), key=lambda s: s[2])
        drop = max(1, round(n * 5 / 33))
        return self._image(N, src, blanks), self._image(N, src[drop:], blanks)

    def sums(self, ns):
        """Per-tile sums as a pass exports them: A, P, Sx, Sy of mostly empty tiles, a few bright."""
        t = torch.rand(ns * ns, 4, device="cuda", generator=self.gen) * 0.1 + 0.9
        bright = torch.rand(ns * ns, 1, device="cuda", generator=self.gen) < 0.02
        scale = torch.tensor([2.0e3, 1e-5, 4e-2, 4e-2], device="cuda")
        return (t * scale * torch.where(bright, 50.0, 1.0)).contiguous()


def _pairs_of(case, seed):
    """The image pairs (x, y, NT) of a case, in the order its outputs come."""
    sky = _Sky(seed)
    kind = case["kind"]
    if kind in ("pair", "pyramid"):
        return [(*sky.pair(case["N"], case.get("blanks", False)), case["NT"])]
    if kind == "stream":
        return [(*sky.pair(case["N"], case["blanks"]), case["NT"]) for _ in range(case["pairs"])]
    if kind == "batch":
        return [(*sky.pair(N), NT) for N, NT in _batch_shapes(case)]
    refs, reqs = _serve_shapes(case)
    images = [sky.pair(N)[0] for N in refs]
    return [(sky.pair(refs[r])[1], images[r], NT) for r, NT in reqs]


def prepare(case, seed):
    kind = case["kind"]
    if kind == "merge":
        return {"kind": kind, "sums": _Sky(seed).sums(case["ns"]), "f": case["f"]}
    pairs = _pairs_of(case, seed)
    if kind in ("pair", "pyramid"):
        x, y, NT = pairs[0]
        return {"kind": kind, "x": x, "y": y, "NT": NT, "which": case.get("which"),
                "sums": case.get("sums")}
    if kind == "batch":
        return {"kind": kind, "batch": Batch(pairs)}
    if kind == "serve":
        refs, reqs = _serve_shapes(case)
        total = sum(4 * refs[r] ** 2 for r, _ in reqs)
        srv = Server(budget_bytes=2 * total + (64 << 20))
        used = {}
        for (_, ref, _), (r, _) in zip(pairs, reqs):
            if r not in used:
                used[r] = srv.add_reference(ref)
        torch.cuda.synchronize()    # snapshots ready: the requests carry no event
        made = [srv.request(snap, used[r], NT, ready=False)
                for (snap, _, NT), (r, _) in zip(pairs, reqs)]
        return {"kind": kind, "server": srv, "requests": made}
    # stream: outputs and calls fixed once, captured into a graph
    outs = [{k: torch.empty(x.shape[0] // NT, x.shape[0] // NT, device="cuda")
             for k in ("lisi", "auglisi")} for x, _, NT in pairs]

    def calls(stream):
        for (x, y, NT), out in zip(pairs, outs):
            if case["which"] == "separate":
                lisi_tiles(x, y, NT, out=out["lisi"], stream=stream)
                auglisi_tiles(x, y, NT, out=out["auglisi"], stream=stream)
            else:
                iqa_tiles(x, y, NT, out=out, stream=stream)

    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    calls(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        calls(side)
    return {"kind": kind, "graph": graph, "pairs": pairs, "outs": outs, "stream": side}


# ---------------------------------------------------------------------------
# One pass
# ---------------------------------------------------------------------------

def run(state):
    kind = state["kind"]
    if kind == "pair":
        x, y, NT = state["x"], state["y"], state["NT"]
        if state["which"] == "lisi":
            return lisi_tiles(x, y, NT)
        if state["which"] == "auglisi":
            return auglisi_tiles(x, y, NT)
        return iqa_tiles(x, y, NT, sums=state["sums"])
    if kind == "stream":
        state["graph"].replay()
        return state["outs"]
    if kind == "pyramid":
        levels = pyramid(state["x"], state["y"], state["NT"])
        return levels, merge_tiles(levels[0].sums, levels[0].lisi.shape[0])
    if kind == "merge":
        return merge_tiles(state["sums"], state["f"])
    if kind == "batch":
        state["batch"].run()
        return [(r.lisi, r.auglisi) for r in state["batch"].results]
    srv, reqs = state["server"], state["requests"]
    srv.submit(reqs)
    srv.drain()
    srv.poll()
    return [(r.lisi, r.auglisi) for r in reqs]


# ---------------------------------------------------------------------------
# The same in 64 bits
# ---------------------------------------------------------------------------

def _f32(v):
    return float(torch.tensor(v, dtype=torch.float32))


def _exact_sums(x, y, NT):
    N = x.shape[0]
    ns = N // NT
    A = torch.empty(ns, ns, 4, dtype=torch.float64, device=x.device)
    rows = max(1, (1 << 25) // (NT * N))    # tile rows at a time: bounded temporaries
    for t in range(0, ns, rows):
        u = min(ns, t + rows)
        a, b = x[t * NT:u * NT].double(), y[t * NT:u * NT].double()
        a = torch.where(a > 0, a, 0.0)
        b = torch.where(b > 0, b, 0.0)
        s, d = a + b, (a - b).abs()
        for k, v in enumerate((s / (d + _f32(CONST)), s * d, a, b)):
            A[t:u, :, k] = v.view(u - t, NT, ns, NT).sum(dim=(1, 3))
    return A


def _exact_values(A):
    c = _f32(CONST)
    lisi = (c / 2) * A[..., 0] / (torch.maximum(A[..., 2], A[..., 3]) + c)
    aug = 1.0 - A[..., 1] / (A[..., 2] + A[..., 3] + c)
    return lisi, aug


def _exact_level(A):
    return (*_exact_values(A), A.reshape(-1, 4))


def _exact_merge(A, f):
    n = A.shape[0] // f
    return A.view(n, f, n, f, 4).sum(dim=(1, 3))


def exact(case, seed):
    kind = case["kind"]
    if kind == "merge":
        sums = _Sky(seed).sums(case["ns"]).double().view(case["ns"], case["ns"], 4)
        return _exact_level(_exact_merge(sums, case["f"]))
    pairs = _pairs_of(case, seed)
    if kind == "pyramid":
        x, y, NT = pairs[0]
        A = _exact_sums(x, y, NT)
        levels, B = [_exact_level(A)], A
        while B.shape[0] % 2 == 0:
            B = _exact_merge(B, 2)
            levels.append(_exact_level(B))
        return levels, _exact_level(_exact_merge(A, A.shape[0]))
    if kind == "pair":
        x, y, NT = pairs[0]
        A = _exact_sums(x, y, NT)
        if case["which"] != "both":
            return _exact_values(A)[0 if case["which"] == "lisi" else 1]
        lisi, aug, sums = _exact_level(A)
        return lisi, aug, sums if case["sums"] else None
    vals = [_exact_values(_exact_sums(x, y, NT)) for x, y, NT in pairs]
    if kind == "stream":
        return [{"lisi": a, "auglisi": b} for a, b in vals]
    return vals
