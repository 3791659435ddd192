"""Performance cases of the KNN filtering library: the calls that a user's program makes.

Every case is one pass through the C-ABI as its Python binding exposes it:
``knnf_filter`` (one frame), ``knnf_filter_batch`` (many frames, one launch),
``knnf_pc1``, ``knnf_svm`` and ``knnf_svm_pc1`` (the two steps that produce the
filter's inputs), the device pipeline cube -> maps and band -> filter, and a
burst of host frames through the batching server.

Inputs follow ``paper_2404_10631_amd.inputs`` (brain-like Voronoi regions,
dermatology-like lesions, smooth spectra, a one-vs-one model), drawn on the GPU
from the seed alone.

``exact`` evaluates the same definitions in binary64 with plain torch.  The
filter's neighbour order is defined on binary32 distances (with ties by linear
index), so neighbours are selected by those and everything computed from them
(distances, averages) is binary64.
"""
from __future__ import annotations

import math

import torch

from paper_2404_10631_amd import _lib
from paper_2404_10631_amd.serve import Server

DEV = "cuda"
NO_CHECK = _lib.KNNF_PLAN_NO_INPUT_CHECK

# 64 frame sizes with sides from 50 to 1000 pixels, as a scanner with a free
# region of interest delivers them (a fixed list, so that the work is the same
# for every seed); every third side is odd.
_UNEVEN = [(50 + (i * 389) % 951, 50 + (i * 617 + 211) % 951) for i in range(64)]


def listed():
    return [
        # The snapshot sensor's 50 x 50 frame, one call at a time with the
        # library's default plan (input check on): the smallest call.
        dict(name="filter_snapshot", op="filter", kind="derma", H=50, W=50, C=4, K=16, R=7,
             lam=0.01, nbr=False, check=True, search="pruned"),
        # One brain-like image resident on the GPU, inputs known to be finite:
        # the benchmark's call.
        dict(name="filter_brain", op="filter", kind="brain", H=380, W=480, C=4, K=40, R=14,
             lam=0.01, nbr=False, check=False, search="pruned"),
        # The 493 x 375 brain image with the neighbour lists kept and the
        # inputs checked: an analysis that looks at the neighbours (odd sizes).
        dict(name="filter_brain_neighbours", op="filter", kind="brain", H=375, W=493, C=4, K=40,
             R=14, lam=0.01, nbr=True, check=True, search="pruned"),
        # The fused 1000 x 1000 dermatology image: the largest single frame.
        dict(name="filter_derma_large", op="filter", kind="derma", H=1000, W=1000, C=4, K=40, R=14,
             lam=0.01, nbr=False, check=False, search="pruned"),
        # Spectral distance only (spatial weight 0).
        dict(name="filter_spectral", op="filter", kind="brain", H=380, W=480, C=4, K=40, R=14,
             lam=0.0, nbr=False, check=False, search="pruned"),
        # A recording of 1024 snapshot frames in one checked call.
        dict(name="batch_snapshots", op="batch", kind="derma", frames=1024, H=50, W=50, C=4, K=16,
             R=7, lam=0.01, check=True),
        # 64 regions of interest of uneven sizes in one call: the largest case.
        dict(name="batch_uneven", op="batch", kind="brain", frames=64, H=0, W=0, C=4, K=40, R=14,
             lam=0.01, check=False),
        # The band the filter reads, from a 128-band brain cube.
        dict(name="pc1_brain", op="pc1", kind="brain", H=380, W=480, bands=128, normalize=True),
        # The probability maps of the 100-band dermatology cube (rows that are
        # not whole cache lines).
        dict(name="svm_derma", op="svm", kind="derma", H=1000, W=1000, bands=100, C=4),
        # Both steps from one read of the brain cube.
        dict(name="svm_pc1_brain", op="svm_pc1", kind="brain", H=380, W=480, bands=128, C=4,
             normalize=True),
        # Cube to filtered maps on the device, the whole classification of one
        # 493 x 375 image.
        dict(name="pipeline_brain", op="pipeline", kind="brain", H=375, W=493, bands=128, C=4,
             K=40, R=14, lam=0.01),
        # A burst of 30 host frames (21 snapshots, 7 brain images, 2 large
        # ones) through the batching server, until all are done.
        dict(name="serve_burst", op="serve", small=21, medium=7, large=2),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["filter", "filter", "filter", "filter", "batch", "pc1", "svm", "svm_pc1",
                     "pipeline"])
    kind = rng.choice(["brain", "derma"])
    if op == "filter":
        H, W = _log_int(rng, 50, 1000), _log_int(rng, 50, 1000)
        R, K = rng.randint(4, 16), rng.randint(4, 64)
        lam = rng.choice([0.01, 0.01, 0.01, 0.1, 1.0, 0.0])
        if lam == 0.0:  # the band of two rows' windows holds at most 16,384 pixels
            W = min(W, 16384 // (2 * R + 2))
        small = H * W <= 200_000
        return dict(op=op, kind=kind, H=H, W=W, C=rng.choice([2, 3, 4, 4, 4, 7]), K=K, R=R,
                    lam=lam, nbr=rng.random() < 0.3, check=rng.random() < 0.4,
                    search="exhaustive" if lam and small and rng.random() < 0.2 else "pruned")
    if op == "batch":
        H, W = _log_int(rng, 50, 500), _log_int(rng, 50, 500)
        n = max(2, min(1024, _log_int(rng, 2, 4_000_000 // (H * W))))
        return dict(op=op, kind=kind, frames=n, H=H, W=W, C=rng.choice([3, 4, 4]),
                    K=rng.randint(8, 48), R=rng.randint(5, 15), lam=0.01,
                    check=rng.random() < 0.5)
    bands = rng.choice([25, 33, 64, 100, 128, 128, 200, 4 * rng.randint(8, 56)])
    H = _log_int(rng, 50, 1000)
    W = _log_int(rng, 50, min(1000, max(51, 100_000_000 // (bands * H))))
    if op == "pc1":
        return dict(op=op, kind=kind, H=H, W=W, bands=bands, normalize=rng.random() < 0.8)
    C = rng.choice([2, 3, 4, 4, 4, 6])
    if op == "svm":
        return dict(op=op, kind=kind, H=H, W=W, bands=bands, C=C)
    if op == "svm_pc1":
        return dict(op=op, kind=kind, H=H, W=W, bands=bands, C=C, normalize=rng.random() < 0.8)
    return dict(op=op, kind=kind, H=H, W=W, bands=bands, C=C, K=rng.randint(8, 48),
                R=rng.randint(5, 15), lam=0.01)


# ---- inputs ------------------------------------------------------------------


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _uniform(g, n, lo, hi):
    return (lo + (hi - lo) * torch.rand(n, generator=g, device=DEV, dtype=torch.float64)).tolist()


def _grid(H, W):
    y = torch.arange(H, device=DEV, dtype=torch.float32)[:, None]
    x = torch.arange(W, device=DEV, dtype=torch.float32)[None, :]
    return y, x


def _voronoi(H, W, g):
    y, x = _grid(H, W)
    sy, sx = _uniform(g, 6, 0.0, H), _uniform(g, 6, 0.0, W)
    best = torch.full((H, W), float("inf"), device=DEV)
    label = torch.zeros((H, W), device=DEV, dtype=torch.int64)
    for k in range(6):
        d = (y - sy[k]) ** 2 + (x - sx[k]) ** 2
        label = torch.where(d < best, k, label)
        best = torch.minimum(best, d)
    return label


def _blur(img, sigma=2.0):
    """Separable Gaussian, edges reflected."""
    r = 8
    w = [math.exp(-0.5 * (k / sigma) ** 2) for k in range(-r, r + 1)]
    s = sum(w)
    for dim in (0, 1):
        n = img.shape[dim]
        at = torch.arange(n, device=DEV)
        out = torch.zeros_like(img)
        for k in range(-r, r + 1):
            i = (at + k) % (2 * n)
            out += (w[k + r] / s) * img.index_select(dim, torch.where(i < n, i, 2 * n - 1 - i))
        img = out
    return img


def _lesion(H, W, g):
    """Signed distance (pixels, negative inside) to an elliptical lesion's edge."""
    y, x = _grid(H, W)
    dy, dx = _uniform(g, 2, -0.15, 0.15)
    ay, ax = _uniform(g, 2, 0.2, 0.35)
    th = _uniform(g, 1, 0.0, math.pi)[0]
    cy, cx, ay, ax = H / 2 + dy * H, W / 2 + dx * W, ay * H, ax * W
    u = (x - cx) * math.cos(th) + (y - cy) * math.sin(th)
    v = -(x - cx) * math.sin(th) + (y - cy) * math.cos(th)
    return (torch.sqrt((u / ax) ** 2 + (v / ay) ** 2) - 1.0) * min(ax, ay)


def _frame(kind, H, W, C, g, pc1, prob):
    """Fill pc1 (H, W) and prob (H, W, C) with one frame."""
    if kind == "brain":
        label = _voronoi(H, W, g)
        mu = torch.tensor(_uniform(g, 6, 0.15, 0.85), device=DEV)
        level = _blur(mu[label])
        favoured = label % C
    else:
        sd = _lesion(H, W, g)
        inside = 1.0 / (1.0 + torch.exp(sd.clamp(-60, 60)))
        lo, hi = _uniform(g, 1, 0.2, 0.4)[0], _uniform(g, 1, 0.6, 0.8)[0]
        level = inside * lo + (1.0 - inside) * hi
        favoured = torch.where(inside >= 0.5, 0, 1 % C)
    pc1.copy_(level + 0.02 * torch.randn((H, W), generator=g, device=DEV))
    logits = torch.randn((H, W, C), generator=g, device=DEV)
    logits += 2.0 * torch.nn.functional.one_hot(favoured, C)
    prob.copy_(torch.softmax(logits.double(), dim=-1))


def _cube(kind, H, W, B, g):
    """Pixel-major cube, band averages and eigenvector."""
    bands = torch.linspace(0.0, 1.0, B, device=DEV, dtype=torch.float64)
    a, b = _uniform(g, 1, 0.6, 1.4)[0], _uniform(g, 1, 0.0, 1.0)[0]
    base = 0.35 + 0.15 * torch.sin(2 * math.pi * (bands * a + b))
    if kind == "brain":
        label, sites = _voronoi(H, W, g), 6
    else:
        label, sites = (_lesion(H, W, g) > 0).long(), 2
    spectra = []
    for _ in range(sites):
        bump = torch.zeros_like(bands)
        for _ in range(2):
            c, w, h = (_uniform(g, 1, *r)[0] for r in ((0.1, 0.9), (0.05, 0.2), (-0.25, 0.25)))
            bump += h * torch.exp(-0.5 * ((bands - c) / w) ** 2)
        spectra.append((base + bump).clamp(0.0, 1.0))
    spectra = torch.stack(spectra)
    y, x = _grid(H, W)
    fy, py, fx = (_uniform(g, 1, *r)[0] for r in ((2, 6), (0, 6), (2, 6)))
    illum = (1.0 + 0.1 * torch.sin(y / H * fy + py) * torch.cos(x / W * fx)).reshape(-1, 1)
    cube = torch.randn((H * W, B), generator=g, device=DEV)
    cube *= 0.01
    cube.addcmul_(spectra.float()[label.reshape(-1)], illum.expand(-1, B))
    direction = spectra[0] - base
    return cube, base.contiguous(), (direction / direction.norm()).contiguous()


def _model(C, B, g):
    M = C * (C - 1) // 2
    w = torch.randn((M, B), generator=g, device=DEV, dtype=torch.float64) * (40.0 / math.sqrt(B))
    bias = -0.35 * w.sum(dim=1)
    bias += 0.5 * torch.randn(M, generator=g, device=DEV, dtype=torch.float64)
    A = torch.tensor(_uniform(g, M, -2.5, -0.5), device=DEV, dtype=torch.float64)
    Bp = torch.tensor(_uniform(g, M, -0.3, 0.3), device=DEV, dtype=torch.float64)
    return w, bias, A, Bp


# ---- states and passes -------------------------------------------------------

_ctx = None


def _context():
    """The process's library context (a program creates it once)."""
    global _ctx
    if _ctx is None:
        _ctx = _lib.knnf_create(torch.cuda.current_device())
    return _ctx


def _stream():
    return torch.cuda.current_stream().cuda_stream


def _c_frame(H, W, C, K, R, lam, pc1, prob, out_prob, out_class, nbr=None, dist=None):
    f = _lib.knnf_frame()
    f.H, f.W, f.C, f.K, f.R, f.lam = H, W, C, K, R, lam
    f.pc1, f.prob = pc1.data_ptr(), prob.data_ptr()
    f.out_prob, f.out_class = out_prob.data_ptr(), out_class.data_ptr()
    f.out_nbr = nbr.data_ptr() if nbr is not None else None
    f.out_dist = dist.data_ptr() if dist is not None else None
    return f


def _plan(search="pruned", check=True):
    """None (the library's own choice), or a plan where the caller asks for something else."""
    if search == "pruned" and check:
        return None
    return _lib.make_plan({"search": _lib.KNNF_SEARCH_PRUNED if search == "pruned"
                           else _lib.KNNF_SEARCH_EXHAUSTIVE,
                           "flags": 0 if check else NO_CHECK})


def _sizes(case):
    return _UNEVEN[:case["frames"]] if not case["H"] else [(case["H"], case["W"])] * case["frames"]


def _serve_specs(case):
    """(kind, H, W, K, R) of the burst's frames, the sizes mixed."""
    each = ([("derma", 50, 50, 16, 7)] * case["small"] + [("brain", 380, 480, 40, 14)] * case["medium"]
            + [("derma", 1000, 1000, 40, 14)] * case["large"])
    return [each[(7 * k) % len(each)] for k in range(len(each))]


class _Served:
    """Host frames in pinned memory, and a server over a device pool that holds them all."""

    def __init__(self, case, g):
        self.frames, need = [], 0
        for kind, H, W, K, R in _serve_specs(case):
            d1 = torch.empty((H, W), device=DEV)
            d2 = torch.empty((H, W, 4), device=DEV)
            _frame(kind, H, W, 4, g, d1, d2)
            h1 = torch.empty((H, W), pin_memory=True)
            h2 = torch.empty((H, W, 4), pin_memory=True)
            for h, d in ((h1, d1), (h2, d2)):
                h.copy_(d)
                h.to(DEV)  # as serve.HostFrame: the first copy from a pinned buffer is slow
            f = _lib.knnf_host_frame()
            f.H, f.W, f.C, f.K, f.R, f.lam = H, W, 4, K, R, 0.01
            f.pc1, f.prob, f.t_arrival = h1.data_ptr(), h2.data_ptr(), -1.0
            self.frames.append((f, h1, h2))
            need += _lib.knnf_frame_bytes(H, W, 4, K, False)
        self.server = Server(_context(), need)
        self.tickets = []

    def run(self):
        h = self.server.handle
        for t in self.tickets:  # the last burst's results have been used
            _lib.knnf_server_release(h, t)
        self.tickets = [_lib.knnf_server_submit(h, f)[1] for f, _, _ in self.frames]
        _lib.knnf_server_drain(h)
        pool, base, out = self.server.pool, self.server.pool.data_ptr(), []
        for t in self.tickets:
            v = _lib.knnf_server_result(h, t)
            n = v.H * v.W
            o, c = v.out_prob - base, v.out_class - base
            out.append(pool[o:o + 16 * n].view(torch.float32).view(v.H, v.W, 4))
            out.append(pool[c:c + 4 * n].view(torch.int32).view(v.H, v.W))
        return out

    def __del__(self):
        if getattr(self, "server", None) is not None:
            self.server.close()


def prepare(case, seed):
    _context()
    g, op = _gen(seed), case["op"]
    if op == "serve":
        return _Served(case, g)
    s = dict(case=case)
    if op == "filter":
        H, W, C, K = case["H"], case["W"], case["C"], case["K"]
        s["pc1"] = torch.empty((H, W), device=DEV)
        s["prob"] = torch.empty((H, W, C), device=DEV)
        _frame(case["kind"], H, W, C, g, s["pc1"], s["prob"])
        s["out"] = [torch.empty((H, W, C), device=DEV),
                    torch.empty((H, W), device=DEV, dtype=torch.int32)]
        if case["nbr"]:
            s["out"] += [torch.empty((H, W, K), device=DEV, dtype=torch.int32),
                         torch.empty((H, W, K), device=DEV)]
        s["frame"] = _c_frame(H, W, C, K, case["R"], case["lam"], s["pc1"], s["prob"], *s["out"])
        s["plan"] = _plan(case["search"], case["check"])
    elif op == "batch":
        C, sizes = case["C"], _sizes(case)
        n = sum(h * w for h, w in sizes)
        s["pc1"], s["prob"] = torch.empty(n, device=DEV), torch.empty((n, C), device=DEV)
        s["out"] = [torch.empty((n, C), device=DEV), torch.empty(n, device=DEV, dtype=torch.int32)]
        frames, at = [], 0
        for k, (h, w) in enumerate(sizes):
            e = at + h * w
            if case["H"] and k >= 32:  # a recording: 32 scenes, other frames are noisy repeats
                p = (k % 32) * h * w
                s["pc1"][at:e] = s["pc1"][p:p + h * w].roll(k) + 0.002 * torch.randn(
                    h * w, generator=g, device=DEV)
                s["prob"][at:e] = s["prob"][p:p + h * w].roll(k, 0)
            else:
                _frame(case["kind"], h, w, C, g, s["pc1"][at:e].view(h, w),
                       s["prob"][at:e].view(h, w, C))
            frames.append(_c_frame(h, w, C, case["K"], case["R"], case["lam"], s["pc1"][at:],
                                   s["prob"][at:], s["out"][0][at:], s["out"][1][at:]))
            at = e
        s["frames"] = _lib.frame_array(frames)
        s["plan"] = _plan("pruned", case["check"])
    else:
        H, W, B = case["H"], case["W"], case["bands"]
        n = H * W
        s["cube"], s["mean"], s["vec"] = _cube(case["kind"], H, W, B, g)
        s["band"] = torch.empty(n, device=DEV)
        if op != "pc1":
            C = case["C"]
            s["model"] = _model(C, B, g)
            s["maps"] = torch.empty((n, C), device=DEV)
        if op == "pipeline":
            s["out"] = [torch.empty((H, W, C), device=DEV),
                        torch.empty((H, W), device=DEV, dtype=torch.int32)]
            s["frame"] = _c_frame(H, W, C, case["K"], case["R"], case["lam"], s["band"], s["maps"],
                                  *s["out"])
            s["plan"] = _plan("pruned", check=False)
    return s


def run(state):
    if isinstance(state, _Served):
        return state.run()
    s, case, ctx = state, state["case"], _context()
    op = case["op"]
    if op == "filter":
        _lib.knnf_filter(ctx, s["frame"], s["plan"], _stream())
        return s["out"]
    if op == "batch":
        _lib.knnf_filter_batch(ctx, s["frames"], s["plan"], _stream())
        return s["out"]
    n, B = case["H"] * case["W"], case["bands"]
    if op == "pc1":
        _lib.knnf_pc1(ctx, s["cube"].data_ptr(), n, B, s["mean"].data_ptr(), s["vec"].data_ptr(),
                      s["band"].data_ptr(), case["normalize"], _stream())
        return s["band"]
    model = [t.data_ptr() for t in s["model"]]
    if op == "svm":
        _lib.knnf_svm(ctx, s["cube"].data_ptr(), n, B, case["C"], *model, s["maps"].data_ptr(),
                      _stream())
        return s["maps"]
    _lib.knnf_svm_pc1(ctx, s["cube"].data_ptr(), n, B, case["C"], *model, s["mean"].data_ptr(),
                      s["vec"].data_ptr(), s["maps"].data_ptr(), s["band"].data_ptr(),
                      case.get("normalize", True), _stream())
    if op == "svm_pc1":
        return [s["maps"], s["band"]]
    _lib.knnf_filter(ctx, s["frame"], s["plan"], _stream())
    return [s["maps"], s["band"]] + s["out"]


# ---- work --------------------------------------------------------------------


def _filter_work(n, C, K, nbr=False, pairs=None):
    """Inputs once, outputs once; the K neighbours' distances (8 operations each; every window
    pair's where the caller asks for the exhaustive search) and their class sums."""
    return (n * (4 + 4 * C + 4 * C + 4 + (8 * K if nbr else 0)),
            8 * (pairs if pairs else n * K) + n * C * (K + 1))


def _cube_work(n, B, C=0, band=False):
    """The cube once, the model once, the maps and the band once; 2 operations per hyperplane and
    band, 3 for the projection, and about 20 per pixel and hyperplane for the sigmoids and one
    coupling sweep."""
    M = C * (C - 1) // 2
    return (4 * n * B + 8 * (M + 2 * band) * B + 4 * n * C + (4 * n if band else 0),
            n * (2 * M * B + (3 * B if band else 0) + 20 * M))


def work(case):
    op = case["op"]
    if op == "serve":
        each = [_filter_work(H * W, 4, K) for _, H, W, K, _ in _serve_specs(case)]
        return {"bytes": sum(b for b, _ in each), "flops": sum(f for _, f in each)}
    if op == "filter":
        H, W, R = case["H"], case["W"], case["R"]
        pairs = None
        if case["search"] == "exhaustive":
            pairs = W * W * sum(min(H - 1, r + R) - max(0, r - R) + 1 for r in range(H))
        b, f = _filter_work(H * W, case["C"], case["K"], case["nbr"], pairs)
    elif op == "batch":
        b, f = _filter_work(sum(h * w for h, w in _sizes(case)), case["C"], case["K"])
    else:
        n = case["H"] * case["W"]
        b, f = _cube_work(n, case["bands"], case.get("C", 0), op != "svm")
        if op == "pipeline":
            b2, f2 = _filter_work(n, case["C"], case["K"])
            b, f = b + b2, f + f2
    return {"bytes": b, "flops": f}


# ---- the same definitions in 64 bits -----------------------------------------


def _exact_filter(pc1, prob, K, R, lam):
    """Frames (F, H, W), (F, H, W, C): averages (F, H, W, C), indices and distances (F, H, W, K)."""
    F, H, W = pc1.shape
    C = prob.shape[-1]
    lam32 = torch.tensor(lam, device=DEV, dtype=torch.float32)
    fr, fc = (lam32 * torch.arange(n, device=DEV, dtype=torch.float32) for n in (H, W))
    out = torch.empty((F, H, W, C), device=DEV, dtype=torch.float64)
    nbr = torch.empty((F, H, W, K), device=DEV, dtype=torch.int64)
    dist = torch.empty((F, H, W, K), device=DEV, dtype=torch.float64)
    b = (fc[:, None] - fc[None, :]).double()
    flat = prob.reshape(F, H * W, C).double()
    for r in range(H):
        lo, hi = max(0, r - R), min(H - 1, r + R) + 1
        n = (hi - lo) * W
        a = fr[r] - fr[lo:hi]
        spatial = ((b * b)[:, None, :] + (a * a).double()[None, :, None]).float()  # W, rows, W
        step = max(1, int(48_000_000 // (F * n)))
        for c0 in range(0, W, step):
            c1 = min(W, c0 + step)
            e = (pc1[:, r, c0:c1, None, None] - pc1[:, None, lo:hi, :]).double()
            d32 = (e * e + spatial[c0:c1].double()).float().reshape(F, c1 - c0, n)
            key = d32.view(torch.int32).long() * (1 << 31)
            key += torch.arange(lo * W, hi * W, device=DEV)
            idx = torch.topk(key, K, dim=-1, largest=False, sorted=True).values % (1 << 31)
            nbr[:, r, c0:c1] = idx
            i, j = idx // W, idx % W
            lam64 = float(lam32)
            de = pc1[:, r, c0:c1, None].double() - torch.gather(
                pc1.reshape(F, -1).double(), 1, idx.reshape(F, -1)).view(idx.shape)
            cq = torch.arange(c0, c1, device=DEV)[None, :, None]
            dist[:, r, c0:c1] = de * de + (lam64 * (r - i)) ** 2 + (lam64 * (cq - j)) ** 2
            rows = torch.gather(flat, 1, idx.reshape(F, -1, 1).expand(-1, -1, C))
            out[:, r, c0:c1] = rows.view(F, c1 - c0, K, C).sum(dim=2) / K
    return out, nbr, dist


def _exact_maps(cube, model, C):
    w, bias, A, Bp = model
    M = C * (C - 1) // 2
    pairs = [(i, j) for i in range(C) for j in range(i + 1, C)]
    out = torch.empty((cube.shape[0], C), device=DEV, dtype=torch.float64)
    for p0 in range(0, cube.shape[0], 1 << 17):
        x = cube[p0:p0 + (1 << 17)].double()
        f = torch.stack([(x * w[m]).sum(dim=1) for m in range(M)], dim=1) + bias
        r1 = (1.0 / (1.0 + torch.exp(f * A + Bp))).clamp(1e-7, 1.0 - 1e-7)
        n = x.shape[0]
        r = torch.zeros((n, C, C), device=DEV, dtype=torch.float64)
        for m, (i, j) in enumerate(pairs):
            r[:, i, j] = r1[:, m]
            r[:, j, i] = 1.0 - r1[:, m]
        Q = -(r.transpose(1, 2) * r)
        for t in range(C):
            Q[:, t, t] = (r[:, :, t] ** 2).sum(dim=1)
        p = torch.full((n, C), 1.0 / C, device=DEV, dtype=torch.float64)
        for _ in range(100):
            qp = (Q * p[:, None, :]).sum(dim=2)
            live = (qp - (p * qp).sum(dim=1, keepdim=True)).abs().amax(dim=1) >= 0.005 / C
            if not bool(live.any()):
                break
            z = p.clone()
            for t in range(C):
                qz = (Q * z[:, None, :]).sum(dim=2)
                z[:, t] += ((z * qz).sum(dim=1) - qz[:, t]) / Q[:, t, t]
                z = z / z.sum(dim=1, keepdim=True)
            p = torch.where(live[:, None], z, p)
        out[p0:p0 + n] = p
    return out


def _exact_band(cube, mean, vec, normalize):
    out = torch.cat([((cube[p:p + (1 << 17)].double() - mean) * vec).sum(dim=1)
                     for p in range(0, cube.shape[0], 1 << 17)])
    if normalize:
        lo, hi = out.min(), out.max()
        out = (out - lo) / (hi - lo) if bool(hi > lo) else torch.zeros_like(out)
    return out


def exact(case, seed):
    op = case["op"]
    if op == "serve" or (op == "batch" and not case["H"]):
        return None  # millions of pixels' windows: more than 20 seconds
    s = prepare(case, seed)
    if op == "filter":
        out, _, dist = _exact_filter(s["pc1"][None], s["prob"][None], case["K"], case["R"],
                                     case["lam"])
        return [out[0], None] + ([None, dist[0]] if case["nbr"] else [])
    if op == "batch":
        F, H, W, C = case["frames"], case["H"], case["W"], case["C"]
        out = torch.empty((F, H, W, C), device=DEV, dtype=torch.float64)
        pc1, prob = s["pc1"].view(F, H, W), s["prob"].view(F, H, W, C)
        step = max(1, int(40_000_000 // (W * W * (2 * case["R"] + 1))))
        for f0 in range(0, F, step):
            out[f0:f0 + step] = _exact_filter(pc1[f0:f0 + step], prob[f0:f0 + step], case["K"],
                                              case["R"], case["lam"])[0]
        return [out.view(-1, C), None]
    if op == "pc1":
        return _exact_band(s["cube"], s["mean"], s["vec"], case["normalize"])
    maps = _exact_maps(s["cube"], s["model"], case["C"])
    if op == "svm":
        return maps
    band = _exact_band(s["cube"], s["mean"], s["vec"], case.get("normalize", True))
    if op == "svm_pc1":
        return [maps, band]
    # the filter's inputs are the binary32 maps and band
    H, W, C = case["H"], case["W"], case["C"]
    out = _exact_filter(band.float().view(1, H, W), maps.float().view(1, H, W, C), case["K"],
                        case["R"], case["lam"])[0]
    return [maps, band, out[0], None]
