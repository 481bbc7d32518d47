"""The work that a user of this library has it do, as cases that can be timed
and compared: single frames, stacks, batches, served requests, a training
step, gradients, and the evaluation tools, over the sizes, layouts, methods
and options that they take in use.

listed() names the fixed cases, draw() gives further ones of the same ranges;
prepare() makes what a program has in hand before the call, run() is one pass
through the public entry points, work() the bytes and operations a pass cannot
do without, and exact() its outputs in 64-bit arithmetic.

The inputs are synthetic scenes as a depth camera sees them: a wall at 4 m,
tilted plates and spheres in front of it with step edges around them, noise of
standard deviation 0.001 z^2, 2% of the pixels without depth (0).
"""
import math

import numpy as np
import torch

import paper_2209_08241_amd as bn

# frame sizes of the mixed workloads (rows, columns): the sizes of this
# repository's batch and serving workloads, and odd ones between them
MIX = [(240, 320), (480, 640), (720, 1280), (1080, 1920)]
ODD = [(241, 322), (479, 637), (719, 1279), (375, 1242), (576, 640)]


def listed():
    """The fixed cases."""
    return [
        # one camera frame at a time, each result wanted at once: the smallest
        # call, outputs allocated by it
        case("frame_qvga", "frame", H=240, W=320, keep=False),
        # a video loop at 1080p that keeps its output buffers
        case("frame_hd", "frame", H=1080, W=1920),
        # a region of interest cut out of a larger image: odd size, rows that
        # start at any element, the absolute threshold, the synthetic alpha
        case("frame_crop", "frame", H=1429, W=2555, alpha=1, mode="abs", crop=True),
        # a 12-megapixel still
        case("frame_12mp", "frame", H=3072, W=4096),
        # an offline pass that drops only the pairs across an edge
        case("stack_pairs", "stack", n=12, H=720, W=1280, method="pair_removal"),
        # the single-pair estimator averaged over three offsets
        case("stack_scales", "stack", n=6, H=1080, W=1920, method="multiscale", alpha=3, scales=3),
        # the 256-frame batch of mixed sizes, its plan replayed
        case("batch_mix", "batch", n=256),
        # a dozen cameras of different sizes, new buffers at each step
        case("cameras", "cameras", n=12),
        # requests served by continuous batching
        case("served", "served", n=16),
        # a training step on 16 frames: forward, cosine loss, backward
        case("train", "train", n=16, H=480, W=640),
        # gradients of a batch of odd-sized crops (a refinement loop)
        case("grad_crop", "grad", n=4, H=719, W=1277, crop=True),
        # an evaluation step: 5x5 plane fit, angle images, angle errors
        case("evaluate", "evaluate", H=1080, W=1920, radius=2),
    ]


def case(name, kind, n=1, H=0, W=0, method="four_pair", alpha=2, scales=0, mode="rel",
         crop=False, keep=True, radius=2):
    c = dict(kind=kind, n=n, H=H, W=W, method=method, alpha=alpha, scales=scales, mode=mode,
             crop=crop, keep=keep, radius=radius)
    if name:
        c["name"] = name
    return c


def draw(rng):
    """One more case of the same ranges."""
    kind = rng.choice(["frame", "frame", "frame", "stack", "stack", "stack", "batch", "cameras",
                       "served", "train", "grad", "grad", "evaluate", "evaluate"])

    def size(lo, hi):
        # pixels over their logarithm, the usual aspect ratios; half of the
        # widths whole groups of 16, the rest any
        px = math.exp(rng.uniform(math.log(lo), math.log(hi)))
        w = max(8, int(math.sqrt(px * rng.choice([1.0, 4 / 3, 16 / 9, 3.3]))))
        if rng.random() < 0.5:
            w = max(16, w // 16 * 16)
        return max(8, int(px / w)), w

    c = dict(crop=rng.random() < 0.3, mode=rng.choice(["rel", "rel", "rel", "abs", "none"]))
    if kind in ("frame", "stack", "cameras", "served"):
        c["method"] = rng.choice(["four_pair", "four_pair", "pair_removal", "multiscale"])
    multi = c.get("method") == "multiscale"
    c["alpha"] = rng.choice([1, 2, 3, 4]) if multi else rng.choice([1, 2, 2, 2, 3, 4, 5, 6, 7, 8])
    c["scales"] = rng.choice([1, 2, 3, 4, 5, 6]) if multi else 0
    if kind == "frame":
        c["H"], c["W"] = size(4096, 12 << 20)
        c["keep"] = rng.random() < 0.5
    elif kind in ("stack", "train", "grad"):
        c["n"] = rng.randint(2, 24)
        c["H"], c["W"] = size(16384, (6 << 20) / c["n"] if kind == "train" else (12 << 20) / c["n"])
    elif kind == "batch":
        c["n"] = rng.randint(17, 224)
    elif kind in ("cameras", "served"):
        c["n"] = rng.randint(2, 16)
    else:
        c["radius"] = rng.choice([1, 2, 2, 2, 3])
        c["H"], c["W"] = size(16384, 2 << 20)
        c.update(alpha=2, mode="rel")
    return case(None, kind, **c)


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def intrinsics(H, W):
    f = 525.0 * W / 640.0
    return (f, f, 0.5 * (W - 1), 0.5 * (H - 1))


def scenes(n, H, W, seed, crop=False):
    """n scenes: depth [n, H, W] float32 (with crop, a view into larger
    images) and the analytic camera-facing normals [n, H, W, 3] float32."""
    rng = np.random.RandomState(seed % (1 << 31))
    dev = "cuda"
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)
    fx, fy, cx, cy = intrinsics(H, W)
    u = ((torch.arange(W, device=dev, dtype=torch.float32) - cx) / fx).view(1, 1, W)
    v = ((torch.arange(H, device=dev, dtype=torch.float32) - cy) / fy).view(1, H, 1)
    z = torch.full((n, H, W), 4.0, device=dev)
    normal = torch.zeros((n, H, W, 3), device=dev)
    normal[..., 2] = -1.0
    half = np.array([cx / fx, cy / fy])
    for k in range(5):
        # the centre's ray within the picture, its distance, and the shape
        c = rng.uniform(-0.7, 0.7, size=(n, 2)) * half
        dist = rng.uniform(1.0, 3.0, size=(n, 1))
        C = np.concatenate([c * dist, dist], axis=1)
        par = lambda a: torch.as_tensor(a, device=dev, dtype=torch.float32).view(n, 1, 1)  # noqa: E731
        if k < 2:  # a tilted round plate
            th, ph = np.radians(rng.uniform(15, 50, n)), rng.uniform(0, 2 * np.pi, n)
            N = -np.stack([np.sin(th) * np.cos(ph), np.sin(th) * np.sin(ph), np.cos(th)], axis=1)
            den = par(N[:, 0]) * u + par(N[:, 1]) * v + par(N[:, 2])
            t = par((N * C).sum(1)) / den
            r2 = (t * u - par(C[:, 0])) ** 2 + (t * v - par(C[:, 1])) ** 2 + (t - par(C[:, 2])) ** 2
            hit = (r2 < par(rng.uniform(0.3, 0.8, n) ** 2)) & (t > 0.3) & (t < z)
            nn = [par(N[:, i]) for i in range(3)]
        else:  # a sphere
            R = rng.uniform(0.2, 0.5, n)
            rr = u * u + v * v + 1.0
            rc = par(C[:, 0]) * u + par(C[:, 1]) * v + par(C[:, 2])
            disc = rc * rc - rr * par((C * C).sum(1) - R * R)
            t = (rc - disc.clamp(min=0).sqrt()) / rr
            hit = (disc > 0) & (t > 0.3) & (t < z)
            nn = [(t * u - par(C[:, 0])) / par(R), (t * v - par(C[:, 1])) / par(R),
                  (t - par(C[:, 2])) / par(R)]
        z = torch.where(hit, t, z)
        for i in range(3):
            normal[..., i] = torch.where(hit, nn[i], normal[..., i])
    z = z + 0.001 * z * z * torch.randn(z.shape, device=dev, generator=gen)
    z = torch.where(torch.rand(z.shape, device=dev, generator=gen) < 0.02, 0.0, z)
    if crop:
        wide = torch.full((n, H + 2, W + 7), 2.5, device=dev)
        view = wide[:, 1:1 + H, 3:3 + W]
        view.copy_(z)
        z = view
    return z, normal


def sizes(c):
    """(rows, columns) of the frames of a case of mixed sizes, in order."""
    if c["kind"] == "batch":  # 64 : 96 : 64 : 32, as in the 256-frame mix
        share = [0.25, 0.375, 0.25]
        k = [int(round(s * c["n"])) for s in share]
        k.append(c["n"] - sum(k))
        return [s for s, m in zip(MIX, k) for _ in range(m)]
    pool = MIX[:3] + ODD
    return [pool[(5 * i + c["n"]) % len(pool)] for i in range(c["n"])]


class Frames:
    """Frames of mixed sizes: depth views, and outputs as views of three
    buffers (one allocation each, as a program that keeps them would)."""

    def __init__(self, c, seed):
        self.sizes = sizes(c)
        self.depth, by_size = [None] * len(self.sizes), {}
        for i, s in enumerate(self.sizes):
            by_size.setdefault(s, []).append(i)
        for j, (s, where) in enumerate(sorted(by_size.items())):
            d, _ = scenes(len(where), *s, seed * 64 + j, c["crop"])
            for k, i in enumerate(where):
                self.depth[i] = d[k]

    def outputs(self):
        px = [h * w for h, w in self.sizes]
        at = np.concatenate([[0], np.cumsum([-(-p // 16) * 16 for p in px])])
        self.normals = torch.zeros((int(at[-1]), 3), device="cuda")
        self.mask = torch.zeros(int(at[-1]), dtype=torch.uint8, device="cuda")
        self.stats = bn.new_stats(len(px))
        self.list = [bn.BatchFrame(self.depth[i], *intrinsics(h, w),
                                   normals=self.normals[at[i]:at[i] + px[i]].view(h, w, 3),
                                   mask=self.mask[at[i]:at[i] + px[i]].view(h, w),
                                   stats=self.stats[i])
                     for i, (h, w) in enumerate(self.sizes)]
        self.at = at
        return self


def tau_of(c):
    # the absolute threshold is in squared depth units: |n| of a plane facing
    # the camera at 3 m with the case's pixel spacing, times four
    if c["mode"] != "abs":
        return 4.0
    H, W = (c["H"], c["W"]) if c["W"] else (480, 640)
    fx, fy, _, _ = intrinsics(H, W)
    return float(np.float32(4.0 * 9.0 * c["alpha"] ** 2 / (fx * fy)))


def options(c):
    return dict(alpha=c["alpha"], mode=c["mode"], tau=tau_of(c), method=c["method"],
                scales=c["scales"])


def prepare(c, seed):
    kind, n, H, W = c["kind"], c["n"], c["H"], c["W"]
    s = {"case": c, "options": options(c)}
    if kind == "frame":
        d, _ = scenes(1, H, W, seed, c["crop"])
        s["depth"] = d[0]
        if c["keep"]:
            s["keep"] = dict(normals=torch.zeros((H, W, 3), device="cuda"),
                             mask=torch.zeros((H, W), dtype=torch.uint8, device="cuda"),
                             stats=bn.new_stats())
    elif kind == "stack":
        s["depth"], _ = scenes(n, H, W, seed, c["crop"])
        s["keep"] = dict(normals=torch.zeros((n, H, W, 3), device="cuda"),
                         mask=torch.zeros((n, H, W), dtype=torch.uint8, device="cuda"),
                         stats=bn.new_stats(n))
    elif kind == "batch":
        s["frames"] = Frames(c, seed).outputs()
        s["plan"] = bn.BatchPlan(s["frames"].list, **s["options"])
    elif kind == "cameras":
        s["frames"] = Frames(c, seed).outputs()
        s["plan"] = bn.BatchPlan(s["frames"].list, **s["options"])
    elif kind == "served":
        s["frames"] = Frames(c, seed)
        s["server"] = bn.Server(1 << 30, **s["options"])
        s["open"] = []
    elif kind == "train":
        s["depth"], s["target"] = scenes(n, H, W, seed, c["crop"])
        s["target_mask"] = torch.zeros((n, H, W), dtype=torch.uint8, device="cuda")
    elif kind == "grad":
        s["depth"], t = scenes(n, H, W, seed, c["crop"])
        s["cotangent"] = -t / (n * H * W)
        s["keep"] = torch.zeros((n, H, W), device="cuda")
    else:
        d, t = scenes(1, H, W, seed, c["crop"])
        s["depth"], s["target"] = d[0], t[0].contiguous()
        # an estimate near the truth, 14% of its pixels masked
        gen = torch.Generator(device="cuda")
        gen.manual_seed(seed + 1)
        e = t[0] + 0.1 * torch.randn(t[0].shape, device="cuda", generator=gen)
        e = e / e.norm(dim=-1, keepdim=True)
        s["mask"] = (torch.rand((H, W), device="cuda", generator=gen) < 0.14).to(torch.uint8)
        s["estimate"] = torch.where((s["mask"] == 0)[..., None], e, 0.0).contiguous()
    return s


class Slot:
    """A request's output in the server's memory, for torch.as_tensor."""

    def __init__(self, ptr, shape, typestr):
        self.__cuda_array_interface__ = dict(shape=shape, typestr=typestr, data=(ptr, False),
                                             version=2)


def run(s):
    c, opt = s["case"], s["options"]
    kind = c["kind"]
    if kind == "frame":
        n, m, st = bn.estimate_normals(s["depth"], *intrinsics(c["H"], c["W"]), **opt,
                                       **s.get("keep", {}))
        return dict(normals=n, mask=m, stats=st)
    if kind == "stack":
        n, m, st = bn.estimate_normals_stack(s["depth"], intrinsics(c["H"], c["W"]), **opt,
                                             **s["keep"])
        return dict(normals=n, mask=m, stats=st)
    if kind == "batch":
        s["plan"].run()
        f = s["frames"]
        return dict(normals=f.normals, mask=f.mask, stats=f.stats)
    if kind == "cameras":
        f = s["frames"]
        s["plan"].update(f.list)
        s["plan"].launch()
        return dict(normals=f.normals, mask=f.mask, stats=f.stats)
    if kind == "served":
        srv = s["server"]
        for rid in s["open"]:          # the last pass's results are no longer read
            srv.release(rid)
        f = s["frames"]
        s["open"] = [srv.submit(d, *intrinsics(*hw)) for d, hw in zip(f.depth, f.sizes)]
        out = []
        for rid, (h, w) in zip(s["open"], f.sizes):
            info = srv.wait(rid)
            out.append([torch.as_tensor(Slot(info["normals"], (h, w, 3), "<f4"), device="cuda"),
                        torch.as_tensor(Slot(info["mask"], (h, w), "|u1"), device="cuda")])
        return out
    if kind == "train":
        x = s["depth"].detach().requires_grad_(True)
        n, m = bn.normals_with_grad_stack(x, intrinsics(c["H"], c["W"]), c["alpha"], c["mode"],
                                          opt["tau"])
        loss = bn.cosine_loss(n, s["target"], m, s["target_mask"])
        loss.backward()
        return dict(loss=loss.detach(), grad=x.grad, mask=m)
    if kind == "grad":
        g = bn.normals_vjp_stack(s["depth"], intrinsics(c["H"], c["W"]), s["cotangent"],
                                 c["alpha"], c["mode"], opt["tau"], grad_depth=s["keep"])
        return dict(grad=g)
    fit, fit_mask = bn.plane_fit_normals(s["depth"], *intrinsics(c["H"], c["W"]), c["radius"])
    theta, phi = bn.normal_angles(s["estimate"])
    mse = bn.angle_mse(s["estimate"], s["mask"], s["target"], None, sync=False)
    return dict(fit=fit, fit_mask=fit_mask, theta=theta, phi=phi, mse=mse)


def work(c):
    """Each input read once and each output written once; the operations of
    the definitions (products, sums, compares, roots)."""
    kind = c["kind"]
    px = sum(h * w for h, w in sizes(c)) if kind in ("batch", "cameras", "served") \
        else c["n"] * c["H"] * c["W"]
    ops = {"four_pair": 34, "pair_removal": 95, "multiscale": 14 + 16 * c["scales"]}[c["method"]]
    if kind == "train":
        # forward 17, loss 12 + 12 + 1 + 1 read, its gradient 12 + 1 + 1 read
        # and 12 written, adjoint 4 + 12 read and 4 written
        return dict(bytes=(17 + 26 + 26 + 20) * px, flops=(34 + 6 + 4 + 70) * px)
    if kind == "grad":
        return dict(bytes=20 * px, flops=70 * px)
    if kind == "evaluate":
        # fit 4 read and 13 written; angles 12 read and 8 written; errors 25 read
        taps = (2 * c["radius"] + 1) ** 2
        return dict(bytes=(17 + 20 + 25) * px, flops=(14 * taps + 120 + 40 + 80) * px)
    return dict(bytes=17 * px, flops=ops * px)


# ---------------------------------------------------------------------------
# the same outputs in 64 bits, in plain torch
# ---------------------------------------------------------------------------

def exact(c, seed):
    s = inputs_only(c, seed)
    kind = c["kind"]
    if kind in ("batch", "cameras", "served"):
        f = s["frames"]
        got = [exact_normals(c, f.depth[i][None], hw)[0] for i, hw in enumerate(f.sizes)]
        if kind == "served":
            return [[g, None] for g in got]
        pad = [torch.cat([g.reshape(-1, 3), g.new_zeros(-(h * w) % 16, 3)])
               for g, (h, w) in zip(got, f.sizes)]
        return dict(normals=torch.cat(pad), mask=None, stats=None)
    hw = (c["H"], c["W"])
    if kind == "frame":
        return dict(normals=exact_normals(c, s["depth"][None], hw)[0], mask=None, stats=None)
    if kind == "stack":
        return dict(normals=exact_normals(c, s["depth"], hw), mask=None, stats=None)
    if kind == "train":
        d = s["depth"].double().requires_grad_(True)
        n, codes = exact_normals(c, s["depth"], hw, d, True)
        U = codes == 0
        cos = (n * s["target"].double()).sum(-1)
        loss = torch.where(U, 1.0 - cos, torch.zeros_like(cos)).sum() / U.sum().clamp(min=1)
        loss.backward()
        return dict(loss=loss.detach(), grad=d.grad, mask=None)
    if kind == "grad":
        d = s["depth"].double().requires_grad_(True)
        n = exact_normals(c, s["depth"], hw, d)
        (n * s["cotangent"].double()).sum().backward()
        return dict(grad=d.grad)
    return exact_evaluation(c, s)


def inputs_only(c, seed):
    """prepare()'s inputs, without plans and outputs."""
    if c["kind"] in ("batch", "cameras", "served"):
        return {"frames": Frames(c, seed)}
    if c["kind"] in ("frame", "stack"):
        d, _ = scenes(c["n"], c["H"], c["W"], seed, c["crop"])
        return {"depth": d[0] if c["kind"] == "frame" else d}
    return prepare(c, seed)


def shifted(d, dx, dy):
    """The image whose pixel (x, y) is d's (x + dx, y + dy), 0 outside."""
    H, W = d.shape[-2:]
    out = torch.zeros_like(d)
    ys, xs = slice(max(0, -dy), min(H, H - dy)), slice(max(0, -dx), min(W, W - dx))
    if ys.start < ys.stop and xs.start < xs.stop:
        out[..., ys, xs] = d[..., ys.start + dy:ys.stop + dy, xs.start + dx:xs.stop + dx]
    return out


def fma32(a, b, c):
    return (a.double() * b.double() + c.double()).float()


def exact_normals(c, d32, hw, d64=None, want_codes=False):
    """Unit normals [n, H, W, 3] in 64 bits; which pixels hold one is decided
    in binary32, in the order that the header of the library gives."""
    H, W = hw
    fx, fy, cx, cy = (float(np.float32(v)) for v in intrinsics(H, W))
    alpha, K, tau = c["alpha"], c["scales"], tau_of(c)
    method = c["method"]
    if d64 is None:
        d64 = d32.double()
    x = torch.arange(W, device=d32.device, dtype=torch.float32).view(1, 1, W)
    y = torch.arange(H, device=d32.device, dtype=torch.float32).view(1, H, 1)
    xc, yc = x - cx, y - cy
    offs = [i * alpha for i in range(1, K + 1)] if method == "multiscale" else [alpha]
    reach = offs[-1]
    lo = 0 if method == "multiscale" else reach
    ok = ((x >= lo) & (x + reach < W) & (y >= lo) & (y + reach < H)).expand(d32.shape).clone()
    rel, none = c["mode"] == "rel", c["mode"] == "none"
    t32 = float(np.float32(tau))
    scale = {"four_pair": 4.0 * fx * fy * t32 / alpha, "pair_removal": fx * fy * t32 / alpha,
             "multiscale": K * fx * fy * t32}[method]
    k_abs = torch.tensor(math.inf if none else float(np.float32(scale * scale)),
                         device=d32.device, dtype=torch.float32)
    tt = float(np.float32(t32) * np.float32(t32))
    good = lambda t: torch.isfinite(t) & (t > 0)  # noqa: E731
    q_good = lambda q: torch.isfinite(q) & (q >= 2.0 ** -126)  # noqa: E731
    taps32 = lambda a, b: shifted(d32, a, b)  # noqa: E731
    taps64 = lambda a, b: shifted(d64, a, b)  # noqa: E731
    ok &= good(d32)
    xd, yd = xc.double(), yc.double()

    def closed(tap, f, mul_add, xo, yo):
        d2, d3, d4, d5 = tap(alpha, 0), tap(0, alpha), tap(-alpha, 0), tap(0, -alpha)
        P, S, Q, T = d2 - d4, d2 + d4, d3 - d5, d3 + d5
        a, b, w = T * P, S * Q, f(alpha) * (S * T)
        return fx * a, fy * b, mul_add(xo, a, yo, b, w), w

    plain = lambda xo, a, yo, b, w: (xo * a + yo * b) + w  # noqa: E731
    fused = lambda xo, a, yo, b, w: fma32(xo, a, fma32(yo, b, w))  # noqa: E731
    if method == "four_pair":
        for a, b in ((alpha, 0), (0, alpha), (-alpha, 0), (0, -alpha)):
            ok &= good(taps32(a, b))
        mx, my, mz, w = closed(taps32, float, plain, xc, yc)
        q = (mx * mx + my * my) + mz * mz
        fire = q > (tt * (w * w) if rel else k_abs)
        ok &= q_good(q)
        m = torch.stack(closed(taps64, float, plain, xd, yd)[:3], -1)
    elif method == "pair_removal":
        pairs = [(1, 1), (-1, 1), (-1, -1), (1, -1)]
        keeps, vecs = [], []
        for sh, sv in pairs:
            def vector(tap, d1, mul_add, xo, yo):
                dh, dv = tap(sh * alpha, 0), tap(0, sv * alpha)
                A, B = sh * ((dh - d1) * dv), sv * (dh * (dv - d1))
                w = (float(alpha) * dh) * dv
                return fx * A, fy * B, mul_add(xo, A, yo, B, w), w
            ok &= good(taps32(sh * alpha, 0)) & good(taps32(0, sv * alpha))
            mx, my, mz, w = vector(taps32, d32, fused, xc, yc)
            q = fma32(mx, mx, fma32(my, my, mz * mz))
            keeps.append(~(q > ((tt * w) * w if rel else k_abs)))
            ok &= q_good(q)
            vecs.append(vector(taps64, d64, plain, xd, yd)[:3])
        every = keeps[0] & keeps[1] & keeps[2] & keeps[3]
        fire = ~(keeps[0] | keeps[1] | keeps[2] | keeps[3])
        whole = closed(taps64, float, plain, xd, yd)[:3]
        m = torch.stack([torch.where(every, whole[i],
                                     sum(k.double() * v[i] for k, v in zip(keeps, vecs)))
                         for i in range(3)], -1)
    else:
        M32 = [torch.zeros_like(d32) for _ in range(4)]
        M64 = [torch.zeros_like(d64) for _ in range(4)]
        for off in offs:
            def vector(tap, d1, mul_add, xo, yo):
                d2, d3 = tap(off, 0), tap(0, off)
                A, B, w = (d2 - d1) * d3, d2 * (d3 - d1), float(off) * (d2 * d3)
                return fx * A, fy * B, mul_add(xo, A, yo, B, w), w
            ok &= good(taps32(off, 0)) & good(taps32(0, off))
            o32 = torch.tensor(float(off), device=d32.device)
            M32 = [fma32(o32, v, t) for v, t in zip(vector(taps32, d32, fused, xc, yc), M32)]
            M64 = [off * v + t for v, t in zip(vector(taps64, d64, plain, xd, yd), M64)]
        q = fma32(M32[0], M32[0], fma32(M32[1], M32[1], M32[2] * M32[2]))
        fire = q > (tt * (M32[3] * M32[3]) if rel else k_abs)
        ok &= q_good(q)
        m = torch.stack(M64[:3], -1)
    codes = torch.where(ok, fire.int(), 2)
    valid = codes == 0
    m = torch.where(valid[..., None], m, torch.ones_like(m))
    m = m * torch.tensor([1.0, 1.0, -1.0], device=m.device, dtype=torch.float64)
    out = torch.where(valid[..., None], m / m.norm(dim=-1, keepdim=True), torch.zeros_like(m))
    return (out, codes) if want_codes else out


def exact_evaluation(c, s):
    H, W = c["H"], c["W"]
    R = c["radius"]
    fx, fy, cx, cy = (float(np.float32(v)) for v in intrinsics(H, W))
    d = s["depth"].double()
    x = torch.arange(W, device=d.device, dtype=torch.float64).view(1, W)
    y = torch.arange(H, device=d.device, dtype=torch.float64).view(H, 1)
    ok = ((x >= R) & (x + R < W) & (y >= R) & (y + R < H)).expand(H, W).clone()
    X = torch.stack([(x - cx) / fx * d, (y - cy) / fy * d, d])
    window = [(i, j) for j in range(-R, R + 1) for i in range(-R, R + 1)]
    total = torch.zeros_like(X)
    for i, j in window:
        t = shifted(d, i, j)
        ok &= torch.isfinite(t) & (t > 0)
        total += shifted(X, i, j)
    mean = total / len(window)
    A = torch.zeros((3, 3, H, W), device=d.device, dtype=torch.float64)
    for i, j in window:
        p = shifted(X, i, j) - mean
        A += p[:, None] * p[None, :]
    A = A.permute(2, 3, 0, 1)[ok]
    v = torch.linalg.eigh(A.cpu())[1][:, :, 0].to(d.device)
    ray = torch.stack([((x - cx) / fx).expand(H, W), ((y - cy) / fy).expand(H, W),
                       torch.ones((H, W), device=d.device, dtype=torch.float64)], -1)
    v = torch.where((v * ray[ok]).sum(-1, keepdim=True) > 0, -v, v)
    fit = torch.zeros((H, W, 3), device=d.device, dtype=torch.float64)
    fit[ok] = v

    def angles(n):
        n = n.double()
        phi = torch.atan2(n[..., 1], n[..., 0])
        return (torch.atan2(torch.hypot(n[..., 0], n[..., 1]), n[..., 2]),
                torch.where(phi < 0, phi + 2 * math.pi, phi))

    theta, phi = angles(s["estimate"])
    t2, p2 = angles(s["target"])
    both = s["mask"] == 0
    k = both.sum().double()
    mse = torch.stack([((theta - t2)[both] ** 2).sum() / k, ((phi - p2)[both] ** 2).sum() / k, k])
    return dict(fit=fit, fit_mask=None, theta=theta, phi=phi, mse=mse)
