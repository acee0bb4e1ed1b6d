"""Workloads of the rasterizer as a program that uses it has them, for timing and comparing builds.

`listed()` names the fixed cases and `draw()` gives further ones of the same ranges; `prepare()` makes
what such a program holds before the call, `run()` is one pass through the public entry points,
`work()` the bytes and operations the pass cannot do without and `exact()` its outputs in 64 bits
(plain torch, nothing of the package).

A case is a dict of plain values:
  do      "grad"    render() and the gradient of its image through torch.autograd
          "frame"   Rasterizer.bin + render_fwd, nothing kept for a backward (a viewer's frame)
          "step"    TrainStep captured once into a HIP graph and replayed (forward + backward)
          "train"   LossTrainStep replayed: L1 loss, backward, statistics and Adam on raw parameters
          "densify" one clone / split / prune step
  n, deg  Gaussians and SH degree;  scene "sphere" (radius 1..5 around the camera) or "roaming"
          (blobs and a shell, radius 2..20, some on the seam)
  views   sizes joined by "+", "WxH*k" for k equirectangular views, "cubeF" for the six FxF pinhole
          faces of a cubemap;  poses "identity", "yaw" or "any" (centres in a 1 m cube but for identity)
  tile, footprint, depth, bg: settings of the rasterizer
"""
import math

import torch

from paper_2410_20686_amd.densify import DensifyStats, densify
from paper_2410_20686_amd.optim import GaussianParams, LossTrainStep
from paper_2410_20686_amd.rasterizer import Rasterizer, TrainStep, render

NAMES = ("means", "scales", "quats", "opacities", "sh")
ADAM_STEP = 1000            # iterations a training state has behind it
TAU = (2e-5, 1e-4)          # densification thresholds at the equator and the pole
EXTENT = 20.0               # scene extent of a densification step


def _case(name, do, n, deg, scene, views, poses="identity", tile=16, footprint="affine", depth=False, bg=0.0):
    c = dict(do=do, n=n, deg=deg, scene=scene, views=views, poses=poses, tile=tile, footprint=footprint, depth=depth, bg=bg)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest call: a thumbnail fitted through torch.autograd, one view, constant colours
        _case("grad_2k_256x128", "grad", 2000, 0, "sphere", "256x128"),
        # the same as a captured loop: what is left of it is kernels and the gaps between them
        _case("step_6k_512x256", "step", 6007, 1, "sphere", "512x256", bg=0.5),
        # a viewer's frame of a small scene; sides that are multiples of 16 but not of 32
        _case("frame_30k_1008x496", "frame", 30011, 3, "roaming", "1008x496", "any"),
        # a frame with its depth map, from a full-size scene
        _case("frame_depth_300k_2048x1024", "frame", 300000, 3, "roaming", "2048x1024", "yaw", depth=True),
        # training step on one panorama at a time, the way the method's trainer takes its images
        _case("step_100k_2048x1024", "step", 100000, 3, "sphere", "2048x1024"),
        # one large panorama
        _case("step_500k_4096x2048", "step", 500000, 3, "roaming", "4096x2048"),
        # the benchmark's workload: a batch of eight views
        _case("step_500k_8x2048x1024", "step", 500000, 3, "roaming", "2048x1024*8", "yaw"),
        # views of uneven sizes under any rotation
        _case("step_300k_mixed", "step", 300000, 3, "roaming", "4096x2048*2+2048x1024*3+1024x512*3", "any"),
        # a cubemap's faces next to its panorama, SH degree 2, through torch.autograd
        _case("grad_60k_cube_and_panorama", "grad", 60013, 2, "roaming", "cube512+1024x512", "yaw", bg=1.0),
        # the exact (spherical) footprint
        _case("step_spherical_200k_2x2048x1024", "step", 200000, 3, "roaming", "2048x1024*2", "yaw", footprint="spherical"),
        # a whole training iteration at the captures' own size, 32x32 tiles as the autotuner picks there
        _case("train_250k_4x1920x960", "train", 250000, 3, "roaming", "1920x960*4", "yaw", tile=32),
        # densification of a grown scene
        _case("densify_800k", "densify", 800009, 3, "roaming", "2048x1024"),
    ]


def draw(rng):
    do = rng.choice(["grad", "frame", "step", "step", "train", "densify"])
    scene = rng.choice(["sphere", "roaming"])
    deg = rng.choice([0, 1, 2, 3, 3, 3])

    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    if do == "densify":
        return _case(None, do, log_int(5000, 800000), deg, scene, "2048x1024")
    footprint = "spherical" if do != "train" and rng.random() < 0.2 else "affine"
    tile = rng.choice([16, 16, 16, 32])
    step = 32 if tile == 32 else 16
    kinds, pixels, count = [], 0, 0
    most = 6.0e6 if footprint == "spherical" else 1.2e7
    for _ in range(rng.randint(1, 3)):
        if footprint == "affine" and rng.random() < 0.2:
            f = step * log_int(4, 24)
            size, k, px = "cube%d" % f, 6, 6 * f * f
        else:
            h = step * log_int(max(1, 128 // step), 2048 // step)
            w = step * int(round(h / step * rng.choice([2.0, 2.0, 1.75, 2.25])))
            k = max(1, min(rng.randint(1, 4), int(most // (w * h))))
            size, px = "%dx%d" % (w, h) + ("*%d" % k if k > 1 else ""), k * w * h
        if kinds and pixels + px > most:
            continue
        kinds.append(size)
        pixels += px
        count += k
    poses = rng.choice(["identity", "yaw", "any"])
    n = log_int(1000, min(100000 if scene == "sphere" else 500000, 2_000_000 // count, 400000 if footprint == "affine" else 150000))
    depth = do == "frame" and rng.random() < 0.4
    return _case(None, do, n, deg, scene, "+".join(kinds), poses, tile, footprint, depth, rng.choice([0.0, 0.0, 1.0, 0.25]))


# ---- inputs ------------------------------------------------------------------------------------

CUBE = (((0, 0, 1), (0, 1, 0)), ((0, 0, -1), (0, 1, 0)), ((1, 0, 0), (0, 1, 0)),
        ((-1, 0, 0), (0, 1, 0)), ((0, 1, 0), (0, 0, -1)), ((0, -1, 0), (0, 0, 1)))  # (forward, down)


def _views(text):
    """Sizes, pinhole intrinsics by view and, for a cubemap's faces, the face number of each view."""
    wh, pin, face = [], {}, []
    for part in text.split("+"):
        if part.startswith("cube"):
            f = int(part[4:])
            for k in range(6):
                pin[len(wh)] = (f / 2, f / 2, f / 2, f / 2)
                wh.append((f, f))
                face.append(k)
        else:
            size, _, k = part.partition("*")
            w, h = (int(x) for x in size.split("x"))
            wh += [(w, h)] * int(k or 1)
            face += [-1] * int(k or 1)
    return wh, pin, face


def _cams(case, seed):
    wh, _, face = _views(case["views"])
    g = torch.Generator().manual_seed(seed + 77)
    rows, R, c = [], None, None
    for v in range(len(wh)):
        if face[v] <= 0:  # a cubemap's six faces share one centre and one frame
            c = torch.rand(3, generator=g, dtype=torch.float64) - 0.5
            a = 2 * math.pi * float(torch.rand(1, generator=g, dtype=torch.float64))
            q, r = torch.linalg.qr(torch.randn(3, 3, generator=g, dtype=torch.float64))
            q = q * torch.sign(torch.diagonal(r))
            if case["poses"] == "identity":
                R, c = torch.eye(3, dtype=torch.float64), torch.zeros(3, dtype=torch.float64)
            elif case["poses"] == "yaw":
                R = torch.tensor([[math.cos(a), 0, -math.sin(a)], [0, 1, 0], [math.sin(a), 0, math.cos(a)]], dtype=torch.float64)
            else:
                R = q * torch.sign(torch.linalg.det(q))
        M = R
        if face[v] >= 0:
            z, y = (torch.tensor(t, dtype=torch.float64) for t in CUBE[face[v]])
            M = torch.stack([torch.linalg.cross(y, z), y, z]) @ R
        rows.append(torch.cat([M.reshape(-1), -(M @ c)]))
    return torch.stack(rows).float().cuda()


def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _scene(case, seed):
    """(means, scales, quats, opacities, sh), float32 on the GPU."""
    n, g = case["n"], _gen(seed)
    f = dict(generator=g, device="cuda")
    d = torch.randn(3, n, **f)
    d /= d.norm(dim=0)
    if case["scene"] == "sphere":
        means = d * (1 + 4 * torch.rand(n, **f))
    else:  # 70% in 50 blobs, 30% uniform in volume in the shell 2..20
        b = torch.randn(3, 50, **f)
        b = b / b.norm(dim=0) * (2 + 18 * torch.rand(50, **f))
        blob = b[:, torch.randint(0, 50, (n,), **f)] + 0.5 * torch.randn(3, n, **f)
        shell = d * (8 + (8000 - 8) * torch.rand(n, **f)) ** (1 / 3)
        means = torch.where(torch.rand(n, **f) < 0.7, blob, shell)
    lo, hi = math.log(0.01), math.log(0.2)
    scales = torch.exp(lo + (hi - lo) * torch.rand(3, n, **f))
    if case["scene"] == "roaming":  # 5% moved onto the +-pi direction, within two of their largest scales
        off = math.pi + (2 * torch.rand(n, **f) - 1) * 2 * scales.amax(0) / means.norm(dim=0).clamp_min(1e-6)
        rho = torch.hypot(means[0], means[2])
        on = torch.rand(n, **f) < 0.05
        means = torch.stack([torch.where(on, rho * torch.sin(off), means[0]), means[1], torch.where(on, rho * torch.cos(off), means[2])])
    quats = torch.randn(4, n, **f)
    quats /= quats.norm(dim=0)
    opac = torch.sigmoid(torch.randn(n, **f))
    K = (case["deg"] + 1) ** 2
    sh = 0.2 * torch.randn(3 * K, n, **f)
    sh[:3] = math.sqrt(math.pi) * (2 * torch.rand(3, n, **f) - 1)
    return tuple(t.contiguous() for t in (means, scales, quats, opac, sh))


def _upstream(case, seed, pixels):
    """The image's upstream gradient, or the target image of a training iteration."""
    g = _gen(seed + 1000)
    if case["do"] == "train":
        return torch.rand(3 * pixels, generator=g, device="cuda")
    return torch.randn(3 * pixels, generator=g, device="cuda")


def _moments(case, params, seed):
    """Adam moments of a run in progress: of the size that the gradients of a mean image loss have."""
    g = _gen(seed + 2000)
    m = tuple(3e-8 * torch.randn(t.shape, generator=g, device="cuda") for t in params)
    v = tuple(1e-14 * torch.exp(torch.randn(t.shape, generator=g, device="cuda")) for t in params)
    return m, v


def _statistics(case, seed):
    """(grad_sum, tau_sum, count, noise, faint) after a few dozen views: a tenth of the Gaussians above
    the threshold, and the fiftieth part (`faint`, none of them above it) grown nearly transparent."""
    n, g = case["n"], _gen(seed + 3000)
    f = dict(generator=g, device="cuda")
    count = torch.randint(1, 40, (n,), dtype=torch.int32, **f)
    tau = count * (TAU[0] + (TAU[1] - TAU[0]) * 0.5 * torch.rand(n, **f))
    ratio = 0.9 * torch.rand(n, **f)
    order = torch.randperm(n, **f)
    above, faint = order[:n // 10], order[n - n // 50:]
    ratio[above] = 1.1 + ratio[above]
    return tau * ratio, tau, count, torch.randn(2, 3, n, **f), faint


def _settings(case):
    _, pin, _ = _views(case["views"])
    return dict(tile=case["tile"], footprint=case["footprint"], bg=(case["bg"], 0.5 * case["bg"], 0.25 * case["bg"]), pinhole=pin or None)


class State:
    pass


def prepare(case, seed):
    s = State()
    s.case = case
    s.params = _scene(case, seed)
    if case["do"] == "densify":
        grad, tau, count, s.noise, faint = _statistics(case, seed)
        s.params[3][faint] = 0.003
        s.stats = DensifyStats(case["n"], tau_min=TAU[0], tau_max=TAU[1])
        s.stats.grad_sum.copy_(grad)
        s.stats.tau_sum.copy_(tau)
        s.stats.count.copy_(count)
        return s
    wh, _, _ = _views(case["views"])
    s.cams = _cams(case, seed)
    s.rast = Rasterizer(case["n"], case["deg"], wh, _settings(case))
    if case["do"] == "train":
        means, scales, quats, opac, sh = s.params
        s.gp = GaussianParams(means, scales.log(), quats, torch.logit(opac), sh, case["deg"])
        s.params = s.gp.act
    s.rast.bin_checked(*s.params, s.cams)  # the pair list's capacity grows to the scene here
    if case["do"] == "frame":
        s.depth = torch.empty(s.rast.pixels, device="cuda") if case["depth"] else None
        return s
    s.dL = _upstream(case, seed, s.rast.pixels)
    if case["do"] == "grad":
        s.leaves = tuple(t.requires_grad_() for t in s.params)
    elif case["do"] == "step":
        s.step = TrainStep(s.rast, s.params, s.cams, s.dL)
        s.step.capture()
    else:
        s.stats = DensifyStats(case["n"], tau_min=TAU[0], tau_max=TAU[1])
        s.step = LossTrainStep(s.rast, s.gp, s.cams, s.dL, stats=s.stats)
        before = tuple(t.clone() for t in (*s.gp.raw, *s.gp.act))
        s.step.capture()  # runs one iteration on the way: back to where the training state was
        m, v = _moments(case, s.params, seed)
        for t, old in zip((*s.gp.raw, *s.gp.act, *s.gp.m, *s.gp.v), (*before, *m, *v)):
            t.copy_(old)
        s.gp.step_count.fill_(ADAM_STEP)
        s.stats.reset()
    return s


def run(s):
    do = s.case["do"]
    if do == "densify":
        new, src, counts = densify(s.params, s.stats, s.noise, EXTENT, s.case["deg"])
        return dict(zip(NAMES, new), src=src, counts=list(counts))
    if do == "frame":
        s.rast.bin(*s.params, s.cams)
        rgb, T = s.rast.render_fwd(out_depth=s.depth)
        return dict(rgb=rgb, T=T, **({} if s.depth is None else {"depth": s.depth}))
    if do == "grad":
        rgb, T = render(*s.leaves, s.cams, s.rast)
        grads = torch.autograd.grad(rgb, s.leaves, s.dL)
        return dict(zip(NAMES, grads), rgb=rgb.detach(), T=T)
    s.step.replay()
    if do == "step":
        return dict(zip(NAMES, s.step.grads), rgb=s.step.rgb)
    return dict(raw=s.gp.raw, m=s.gp.m, v=s.gp.v, loss=s.step.loss, grad_sum=s.stats.grad_sum,
                tau_sum=s.stats.tau_sum, count=s.stats.count)


def work(case):
    """Bytes: parameters, images and gradients each once.  Operations: about 400 per (Gaussian, view)
    projected and as many again for the adjoint; per pixel about 40 Gaussians composited before it
    is opaque or the list ends, at 23 operations each forward and 50 in reverse."""
    n, width = case["n"], 4 * (11 + 3 * (case["deg"] + 1) ** 2)
    if case["do"] == "densify":
        return {"bytes": n * (2.1 * width + 12 + 4), "flops": 30 * n}
    wh, _, _ = _views(case["views"])
    pixels = sum(w * h for w, h in wh)
    items = n * len(wh)
    seen = min(40.0, 0.02 * n)
    nbytes, flops = n * width + 16 * pixels, 400 * items + 23 * seen * pixels
    if case["depth"]:
        nbytes += 4 * pixels
    if case["do"] != "frame":
        nbytes += n * width + 12 * pixels
        flops += 400 * items + 50 * seen * pixels
    if case["do"] == "train":
        nbytes += 5 * n * width + 12 * n
    return {"bytes": nbytes, "flops": flops}


# ---- the same in 64 bits -----------------------------------------------------------------------

def _sh(d, K):
    """Real spherical harmonics of unit directions d [3, n], degree by degree, m = -l..l."""
    x, y, z = d
    Y = [torch.full_like(x, 0.5 / math.sqrt(math.pi))]
    if K > 1:
        c = math.sqrt(3 / (4 * math.pi))
        Y += [c * y, c * z, c * x]
    if K > 4:
        a, b = math.sqrt(15 / math.pi) / 2, math.sqrt(5 / math.pi) / 4
        Y += [a * x * y, a * y * z, b * (2 * z * z - x * x - y * y), a * x * z, a / 2 * (x * x - y * y)]
    if K > 9:
        p = math.pi
        a, b, c = math.sqrt(35 / (2 * p)) / 4, math.sqrt(105 / p) / 2, math.sqrt(21 / (2 * p)) / 4
        e, f = math.sqrt(7 / p) / 4, math.sqrt(105 / p) / 4
        Y += [a * y * (3 * x * x - y * y), b * x * y * z, c * y * (4 * z * z - x * x - y * y),
              e * z * (2 * z * z - 3 * x * x - 3 * y * y), c * x * (4 * z * z - x * x - y * y),
              f * z * (x * x - y * y), a * x * (x * x - 3 * y * y)]
    return Y


def _dot(a, b):
    return a[0] * b[0] + a[1] * b[1] + a[2] * b[2]


def _sandwich(R, S):
    """R S R^T for 3x3 lists of numbers or tensors (R may have two rows)."""
    RS = [[sum(r[k] * S[k][j] for k in range(3)) for j in range(3)] for r in R]
    return [[sum(RS[i][k] * R[j][k] for k in range(3)) for j in range(len(R))] for i in range(len(R))]


def _project(P, cam, wh, pin, deg, spherical):
    """Per-Gaussian quantities of one view: leaves of the compositing (first six, or nine with the
    spherical footprint, of the shape, then opacity and colour), and plain values."""
    m, s, q, o, sh = P
    W, H = wh
    near, far, dilation, pole = (float(torch.tensor(v, dtype=torch.float32)) for v in (0.2, 1e4, 0.3, 1e-4))
    R = [[cam[3 * i + j] for j in range(3)] for i in range(3)]
    mu = [_dot(R[i], m) + cam[9 + i] for i in range(3)]
    w, x, y, z = q / q.norm(dim=0)
    Rq = [[1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y)],
          [2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x)],
          [2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)]]
    D = [[s[i] ** 2 if i == j else 0.0 for j in range(3)] for i in range(3)]
    S = _sandwich(R, _sandwich(Rq, D))
    r2 = _dot(mu, mu)
    r, p = r2.sqrt(), mu[0] ** 2 + mu[2] ** 2
    rho = p.sqrt()
    zero = torch.zeros_like(r)
    if pin:
        fx, fy, cx, cy = pin
        depth, tx, ty = mu[2], mu[0] / mu[2], mu[1] / mu[2]
        kept = (depth > near) & (depth < far) & (tx.abs() <= 1.3 * W / (2 * fx)) & (ty.abs() <= 1.3 * H / (2 * fy))
        u, v = fx * tx + cx, fy * ty + cy
        J = [[fx / depth, zero, -fx * tx / depth], [zero, fy / depth, -fy * ty / depth]]
    else:
        depth = r
        kept = (r > near) & (r < far) & (rho > pole * r)
        a1, a2 = W / (2 * math.pi), H / math.pi
        u, v = a1 * torch.atan2(mu[0], mu[2]) + W / 2, a2 * torch.atan2(mu[1], rho) + H / 2
        J = [[a1 * mu[2] / p, zero, -a1 * mu[0] / p],
             [-a2 * mu[0] * mu[1] / (r2 * rho), a2 * rho / r2, -a2 * mu[1] * mu[2] / (r2 * rho)]]
    c = [-sum(R[k][i] * cam[9 + k] for k in range(3)) for i in range(3)]
    d = torch.stack([m[i] - c[i] for i in range(3)])
    d = d / d.norm(dim=0)
    K = (deg + 1) ** 2
    Y = _sh(d, K)
    col = [(sum(sh[3 * k + ch] * Y[k] for k in range(K)) + 0.5).clamp_min(0) for ch in range(3)]
    pmin = -torch.log(255 * o.detach())
    kept = kept & (pmin < 0)
    with torch.no_grad():
        k = (-2 * pmin).clamp_min(0).sqrt()
    if spherical:
        delta = dilation * (math.pi / H) ** 2
        C = [[S[i][j] / r2 + (delta if i == j else 0.0) for j in range(3)] for i in range(3)]
        co = [[C[(i + 1) % 3][(j + 1) % 3] * C[(i + 2) % 3][(j + 2) % 3] - C[(i + 1) % 3][(j + 2) % 3] * C[(i + 2) % 3][(j + 1) % 3]
               for j in range(3)] for i in range(3)]
        det = _dot(C[0], co[0])
        kept = kept & (det > 0)
        A = [co[i][j] / det for i, j in ((0, 0), (0, 1), (0, 2), (1, 1), (1, 2), (2, 2))]
        leaf = A + [mu[i] / r for i in range(3)]
        with torch.no_grad():
            sb = k * (s.amax(0) ** 2 / r2 + delta).sqrt() * 1.001
            beta = torch.asin(sb.clamp(max=1.0))
            theta = torch.atan2(mu[1], rho)  # downwards
            whole = (sb >= 1) | (theta.abs() + beta >= math.pi / 2)
            eu = W / (2 * math.pi) * torch.asin((torch.sin(beta) / torch.cos(theta)).clamp(-1, 1)) + 0.01
            eu = torch.where(whole, torch.full_like(eu, float(W)), eu)
            ev = torch.where(sb >= 1, torch.full_like(eu, float(H)), beta * H / math.pi + 0.01)
    else:
        cov = _sandwich([[_dot(J[i], [R[k][j] for k in range(3)]) for j in range(3)] for i in range(2)],
                        _sandwich(Rq, D))
        uu, uv, vv = cov[0][0] + dilation, cov[0][1], cov[1][1] + dilation
        det = uu * vv - uv * uv
        kept = kept & (det > 0)
        leaf = [u, v, vv / det, -uv / det, uu / det]
        with torch.no_grad():
            eu, ev = k * uu.sqrt() * 1.001 + 0.01, k * vv.sqrt() * 1.001 + 0.01
    return leaf + [o] + col, dict(u=u.detach(), v=v.detach(), eu=eu, ev=ev, kept=kept, depth=depth.detach(),
                                  pmin=pmin, ct=(rho / r).detach())


TILE = 16


def _lists(x, wh, pin, block=TILE):
    """(tile, Gaussian) pairs of the footprint rectangles, ordered by (tile, float depth, index)."""
    W, H = wh
    nx, ny = -(-W // block), -(-H // block)
    at = x["kept"].nonzero()[:, 0]
    at = at[torch.sort(x["depth"][at].float(), stable=True)[1]]
    u, v, eu, ev = (x[k][at] for k in ("u", "v", "eu", "ev"))
    c0, c1 = torch.floor((u - eu) / block), torch.floor((u + eu) / block)
    r0, r1 = torch.floor((v - ev) / block).clamp_min(0), torch.floor((v + ev) / block).clamp_max(ny - 1)
    if pin:
        c0, c1 = c0.clamp_min(0), c1.clamp_max(nx - 1)
    else:
        full = c1 - c0 + 1 >= nx
        c0, c1 = torch.where(full, torch.zeros_like(c0), c0), torch.where(full, torch.full_like(c1, nx - 1), c1)
    nc, nr = (c1 - c0 + 1).clamp_min(0).long(), (r1 - r0 + 1).clamp_min(0).long()
    num = nc * nr
    own = torch.repeat_interleave(torch.arange(len(at), device=at.device), num)
    k = torch.arange(len(own), device=at.device) - torch.repeat_interleave(num.cumsum(0) - num, num)
    tile = (r0.long()[own] + k // nc[own]) * nx + (c0.long()[own] + k % nc[own]) % nx
    tile, order = torch.sort(tile, stable=True)
    visible = torch.zeros_like(x["kept"])
    visible[at[num > 0]] = True
    length = torch.bincount(tile, minlength=nx * ny)
    return at[own[order]], length, nx, visible


def _composite(leaf, x, wh, pin, spherical, bg, dL, most=24_000_000):
    """(rgb [3, H, W], T, depth map) of one view; with an upstream gradient dL [3, H, W] its gradient
    is added to .grad of the leaves."""
    W, H = wh
    rgb = torch.tensor(bg, dtype=torch.float64, device="cuda").view(3, 1).expand(3, W * H).clone()
    T_out = torch.ones(W * H, dtype=torch.float64, device="cuda")
    D_out = torch.zeros_like(T_out)
    gauss, length, nx, visible = _lists(x, wh, pin)
    first = length.cumsum(0) - length
    size, tiles = torch.sort(length, descending=True)
    size, at = size.tolist(), 0
    cell = torch.arange(TILE * TILE, device="cuda")
    while at < len(size) and size[at] > 0:
        L = size[at]
        B = max(1, most // (L * TILE * TILE))
        t = tiles[at:at + B]
        at += B
        j = torch.arange(L, device="cuda")
        valid = j < length[t][:, None]
        idx = gauss[(first[t][:, None] + j).clamp_max(len(gauss) - 1)]
        px, py = (t % nx)[:, None] * TILE + cell % TILE, (t // nx)[:, None] * TILE + cell // TILE
        inside = (px < W) & (py < H)
        pix = (py * W + px)[inside]
        G = [q[idx][:, :, None] for q in leaf]
        X, Yc = px[:, None, :].double() + 0.5, py[:, None, :].double() + 0.5
        if spherical:
            a11, a12, a13, a22, a23, a33, m1, m2, m3, o, c0, c1, c2 = G
            phi, th = (X - W / 2) * (2 * math.pi / W), (H / 2 - Yc) * (math.pi / H)
            d1, d2, d3 = torch.cos(th) * torch.sin(phi), -torch.sin(th), torch.cos(th) * torch.cos(phi)
            v1, v2, v3 = a11 * m1 + a12 * m2 + a13 * m3, a12 * m1 + a22 * m2 + a23 * m3, a13 * m1 + a23 * m2 + a33 * m3
            b = v1 * d1 + v2 * d2 + v3 * d3
            a = a11 * d1 * d1 + a22 * d2 * d2 + a33 * d3 * d3 + 2 * (a12 * d1 * d2 + a13 * d1 * d3 + a23 * d2 * d3)
            power = -0.5 * (m1 * v1 + m2 * v2 + m3 * v3 - b * b / a)
            ok = b.detach() > 0
        else:
            u, v, ca, cb, cc, o, c0, c1, c2 = G
            du, dv = X - u, Yc - v
            if not pin:
                du = du - W * torch.floor(du.detach() / W + 0.5)
            power = -0.5 * (ca * du * du + cc * dv * dv) - cb * du * dv
            ok = True
        ok = ok & (power.detach() >= x["pmin"][idx][:, :, None]) & valid[:, :, None]
        alpha = torch.where(ok, (o * torch.exp(power)).clamp(max=0.99), torch.zeros_like(power))
        alive = torch.cumsum(torch.log1p(-alpha.detach()), 1) >= math.log(1e-4)
        alpha = torch.where(alive, alpha, torch.zeros_like(alpha))
        lg = torch.log1p(-alpha)
        after = torch.cumsum(lg, 1)
        wgt = alpha * torch.exp(after - lg)
        T = torch.exp(after[:, -1])
        out = [(wgt * c).sum(1) + T * b0 for c, b0 in zip((c0, c1, c2), bg)]
        if dL is not None:
            loss = sum((out[ch][inside] * dL[ch].reshape(-1)[pix]).sum() for ch in range(3))
            loss.backward()
        with torch.no_grad():
            for ch in range(3):
                rgb[ch, pix] = out[ch].detach()[inside]
            T_out[pix] = T.detach()[inside]
            D_out[pix] = (wgt.detach() * x["depth"][idx][:, :, None]).sum(1)[inside]
    return rgb.view(3, H, W), T_out, D_out, visible


def _render64(case, params, cams, upstream, l1=False):
    """Images, gradients and statistics of all views; with `l1` the upstream array is the target of
    a mean absolute loss, whose gradient takes its place."""
    wh, pin, _ = _views(case["views"])
    spherical = case["footprint"] == "spherical"
    st = _settings(case)
    bg = [float(torch.tensor(b, dtype=torch.float32)) for b in st["bg"]]
    P = [t.double().requires_grad_(upstream is not None) for t in params]
    cams = cams.double().tolist()
    got, off, total = dict(rgb=[], T=[], depth=[]), 0, 3 * sum(w * h for w, h in wh)
    loss = 0.0
    stats = [torch.zeros(case["n"], dtype=torch.float64, device="cuda") for _ in range(2)]
    for k, (w, h) in enumerate(wh):
        full, x = _project(P, cams[k], (w, h), pin.get(k), case["deg"], spherical)
        leaf = [t.detach().requires_grad_(upstream is not None) for t in full]
        dL = None if upstream is None else upstream[off:off + 3 * w * h].double().view(3, h, w)
        if l1:
            with torch.no_grad():
                rgb = _composite([t.detach() for t in leaf], x, (w, h), pin.get(k), spherical, bg, None)[0]
            loss += float((rgb - dL).abs().sum()) / total
            dL = torch.sign(rgb - dL) / total
        rgb, T, D, visible = _composite(leaf, x, (w, h), pin.get(k), spherical, bg, dL)
        if upstream is not None:
            grads = [torch.zeros_like(t) if t.grad is None else t.grad for t in leaf]
            keep = [torch.where(x["kept"], g, torch.zeros_like(g)) for g in grads]
            use = x["kept"].nonzero()[:, 0]
            torch.autograd.backward([t[use] for t in full], [g[use] for g in keep])
            if l1:
                gu, gv = keep[0] * (w / 2), keep[1] * (h / 2)
                stats[0] += torch.where(visible, torch.hypot(gu, gv), torch.zeros_like(gu))
                lo, hi = (float(torch.tensor(t, dtype=torch.float32)) for t in TAU)
                stats[1] += torch.where(visible, lo + (1 - x["ct"]) * (hi - lo), torch.zeros_like(gu))
        got["rgb"].append(rgb.reshape(-1))
        got["T"].append(T)
        got["depth"].append(D)
        off += 3 * w * h
    out = {k: torch.cat(v) for k, v in got.items()}
    return out, [t.grad for t in P], loss, stats


def _exact_train(case, seed, params, cams, target):
    means, scales, quats, opac, sh = params
    raw = [t.double() for t in (means, scales.log(), quats, torch.logit(opac), sh)]
    act = (means, torch.exp(scales.log()), quats, torch.sigmoid(torch.logit(opac)), sh)
    _, grads, loss, stats = _render64(case, act, cams, target, l1=True)
    m, v = _moments(case, params, seed)
    f32 = lambda x: float(torch.tensor(x, dtype=torch.float32))  # noqa: E731
    b1, b2, eps = f32(0.9), f32(0.999), f32(1e-15)
    lr = [f32(x) for x in (1.6e-4, 5e-3, 1e-3, 5e-2, 2.5e-3, 2.5e-3 / 20)]
    out = dict(raw=[], m=[], v=[], loss=torch.tensor([loss], dtype=torch.float64), grad_sum=stats[0], tau_sum=stats[1], count=None)
    t = ADAM_STEP + 1
    for k, g in enumerate(grads):
        a = act[k].double()
        g = g * (a if k == 1 else a * (1 - a) if k == 3 else 1.0)
        mm, vv = b1 * m[k].double() + (1 - b1) * g, b2 * v[k].double() + (1 - b2) * g * g
        rate = torch.full_like(g, lr[k])
        if k == 4:
            rate[3:] = lr[5]
        out["raw"].append(raw[k] - rate / (1 - b1 ** t) * mm / (vv.sqrt() / math.sqrt(1 - b2 ** t) + eps))
        out["m"].append(mm)
        out["v"].append(vv)
    return out


def _exact_densify(case, seed, params):
    means, scales, quats, opac, sh = params
    grad, tau, count, noise, faint = _statistics(case, seed)
    opac[faint] = 0.003
    f32 = lambda x: torch.tensor(x, dtype=torch.float32, device="cuda")  # noqa: E731
    sel = (count > 0) & (grad >= tau)
    small = scales.amax(0) <= f32(1e-3) * f32(EXTENT)
    drop = opac < f32(0.005)
    orig, clone, child = ((a & ~drop).nonzero()[:, 0] for a in (~(sel & ~small), sel & small, sel & ~small))
    q = quats.double()[:, child]
    w, x, y, z = q / q.norm(dim=0)
    R = [[1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y)],
         [2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x)],
         [2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)]]
    src = torch.cat([orig, clone, child, child])
    out = [t.double()[..., src] for t in params]
    base = len(orig) + len(clone)
    for ch in range(2):
        lo, hi = base + ch * len(child), base + (ch + 1) * len(child)
        l = (scales.double() * noise[ch].double())[:, child]
        for k in range(3):
            out[0][k, lo:hi] += _dot(R[k], l)
        out[1][:, lo:hi] /= 1.6
    return dict(zip(NAMES, out), src=None, counts=[None] * 4)


def exact(case, seed):
    params = _scene(case, seed)
    if case["do"] == "densify":
        return _exact_densify(case, seed, params)
    wh, _, _ = _views(case["views"])
    cams = _cams(case, seed)
    pixels = sum(w * h for w, h in wh)
    up = None if case["do"] == "frame" else _upstream(case, seed, pixels)
    if case["do"] == "train":
        return _exact_train(case, seed, params, cams, up)
    out, grads, _, _ = _render64(case, params, cams, up)
    if case["do"] == "frame":
        return dict(rgb=out["rgb"], T=out["T"], **({"depth": out["depth"]} if case["depth"] else {}))
    got = dict(zip(NAMES, grads), rgb=out["rgb"])
    return dict(got, T=out["T"]) if case["do"] == "grad" else got
