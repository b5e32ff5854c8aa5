"""The work this library is measured on: the lattice operations of a point-cloud
network, called as a training or an inference program calls them.

Five kinds of call, over clouds made on the GPU from a seed:

  head      the output layer alone on a ready lattice: DeformSlice fused with the
            classifier (logits), and with train=True its backward pass down to the
            point features
  conv      one lattice convolution on a ready lattice, sliced back onto the points
  step      a whole pass over a new cloud: splat, neighbour table, the convolutions,
            then the slice or (tail="deform") DeformSlice with the classifier; with
            train=True the backward pass of every stage too
  unet      the same with one coarser level: a second lattice at twice the scale,
            downsample, upsample, slice
  pointnet  the input layer over a new cloud: lattice, Distribute + PointNet, slice;
            with train=True the gradients of its parameters

Vertices have no fixed order from run to run, so every pass ends on the points or
in the gradients of weights, which do not depend on it.
"""
import math

import torch

from paper_2108_03917_amd import Lattice

DEV = "cuda" if torch.cuda.is_available() else "cpu"
WIDTHS = (16, 32, 64)       # the PointNet blocks of the input layer


def _case(name, op, cloud, points, sigma, chain, dtype="bf16", **more):
    c = {"name": name, "op": op, "cloud": cloud, "points": points, "sigma": sigma, "chain": chain, "dtype": dtype,
         "objects": 1, "classes": 0, "train": False, "tail": "slice", "f_d": 0}
    c.update(more)
    return c


def listed():
    return [
        # one part-segmentation object (their mean size), its logits: the smallest call there is
        _case("object_head", "head", "objects", 2613, 0.04, "64", "f32", classes=50),
        # the smallest whole pass: three spheres, few channels
        _case("tiny_step", "step", "spheres", 4096, 0.05, "8-16", "f32"),
        # one object at a time, as part segmentation runs them at inference
        _case("object_step", "step", "objects", 2613, 0.04, "64-64", tail="deform", classes=50),
        # a training step on a batch of 16 objects, convolutions in 32 bits
        _case("objects_train", "step", "objects", 40000, 0.04, "64-64", "f32", objects=16, tail="deform",
              classes=50, train=True),
        # a training step of one U-Net level on the same batch
        _case("objects_unet_train", "unet", "objects", 40000, 0.04, "64-64", objects=16, train=True),
        # an indoor room, inference
        _case("room_step", "step", "room", 200000, 0.04, "64-64-128"),
        # the largest indoor room, output layer forward and backward
        _case("room_head_train", "head", "room", 537211, 0.04, "64", "f32", classes=20, train=True),
        # a mean indoor room through the input layer: colour and normal per point
        _case("room_pointnet", "pointnet", "room", 145003, 0.04, "64", "f32", f_d=6),
        # one LiDAR scan, wide channels, semantic logits
        _case("scan_step", "step", "scan", 103889, 0.3, "128-128", tail="deform", classes=20),
        # a small LiDAR scan through a 32-bit convolution whose width is no power of two
        _case("scan_conv_ragged", "conv", "scan", 82411, 0.3, "96-96", "f32"),
        # four LiDAR scans in space and time (d = 4): the largest inference pass
        _case("frames_step", "step", "frames", 421398, 0.3, "64-64", objects=4),
        # the same four scans through the input layer with its gradients: the largest training pass
        _case("frames_pointnet_train", "pointnet", "frames", 421398, 0.3, "64", "f32", objects=4, f_d=1, train=True),
    ]


def draw(rng):
    """A case of the same ranges: every cloud and call, sizes spread over their logarithm."""
    op = rng.choice(["head", "conv", "step", "step", "unet", "pointnet"])
    cloud = rng.choice(["objects", "room", "scan", "frames"])
    train = rng.random() < 0.4
    dtype = rng.choice(["bf16", "bf16", "f32"])
    lo, hi = {"objects": (1500, 60000), "room": (9000, 300000), "scan": (30000, 130000),
              "frames": (60000, 420000)}[cloud]
    if dtype == "f32" and op in ("conv", "step", "unet"):
        hi = min(hi, 120000)
    points = int(math.exp(rng.uniform(math.log(lo), math.log(hi))))
    objects = 1
    if cloud == "objects":
        objects = max(1, min(32, points // 2613))
    elif cloud == "frames":
        objects = rng.choice([2, 3, 4])
    sigma = {"objects": 0.04, "room": 0.04, "scan": 0.3, "frames": 0.3}[cloud] * rng.choice([1, 1.5, 2])
    sigma = round(sigma, 3)
    widths = [32, 64, 64, 96, 128] if train or dtype == "f32" else [32, 48, 64, 64, 96, 100, 128]
    c = rng.choice(widths)
    if op == "step":
        chain = "-".join(str(w) for w in [c] + [rng.choice([c, rng.choice(widths)]) for _ in range(rng.choice([1, 2]))])
    elif op in ("conv", "unet"):
        chain = "%d-%d" % (c, c if op == "unet" else rng.choice([c, rng.choice(widths)]))
    else:
        chain, dtype = ("64" if op == "pointnet" else str(c)), "f32"
    if op in ("conv", "step", "unet"):      # no dearer than the largest listed case: about this many operations
        ch = [int(w) for w in chain.split("-")]
        macs = sum(a * b for a, b in zip(ch, ch[1:])) + (2 * ch[-1] ** 2 if op == "unet" else 0)
        ops = 2 * 1.7 * 9 * macs * (3 if train and op != "conv" else 1)
        points = max(min(points, int((4e10 if dtype == "f32" else 1.5e11) / ops)), lo // 2)
    tail = "slice"
    if op == "head" or (op == "step" and rng.random() < 0.5):
        tail = "deform"
    classes = rng.choice([8, 20, 26, 50]) if tail == "deform" else 0
    case = _case("", op, cloud, points, sigma, chain, dtype, objects=objects, classes=classes,
                 train=train and op != "conv", tail=tail if op == "step" else "slice",
                 f_d=(rng.choice([1, 3, 6]) if op == "pointnet" else 0))
    del case["name"]
    return case


def _dim(case):
    return 4 if case["cloud"] == "frames" else 3


def _chain(case):
    return [int(c) for c in case["chain"].split("-")]


# -- clouds ------------------------------------------------------------------

class _Rng:
    """Seeded draws on the GPU."""

    def __init__(self, seed):
        self.g = torch.Generator(device=DEV)
        self.g.manual_seed(int(seed))

    def uniform(self, lo, hi, *shape):
        return torch.rand(*shape, generator=self.g, device=DEV) * (hi - lo) + lo

    def normal(self, *shape):
        return torch.randn(*shape, generator=self.g, device=DEV)

    def pick(self, p, n):
        """n indices with probabilities proportional to p."""
        edges = (p.double() / p.double().sum()).cumsum(0)
        u = torch.rand(n, generator=self.g, device=DEV, dtype=torch.float64)
        return torch.searchsorted(edges, u).clamp_(max=p.numel() - 1)

    def perm(self, n):
        return torch.randperm(n, generator=self.g, device=DEV)


def _rotations(r, n):
    q = r.normal(n, 4)
    w, x, y, z = (q / q.norm(dim=1, keepdim=True)).unbind(1)
    return torch.stack([1 - 2 * (y * y + z * z), 2 * (x * y - z * w), 2 * (x * z + y * w),
                        2 * (x * y + z * w), 1 - 2 * (x * x + z * z), 2 * (y * z - x * w),
                        2 * (x * z - y * w), 2 * (y * z + x * w), 1 - 2 * (x * x + y * y)], 1).view(n, 3, 3)


def _spheres(case, r):
    m = case["points"]
    rad = r.uniform(0.1, 0.3, 3)
    centre = rad[:, None] + r.uniform(0, 1, 3, 3) * (1 - 2 * rad[:, None])
    s = r.pick(rad * rad, m)
    v = r.normal(m, 3)
    return centre[s] + rad[s, None] * v / v.norm(dim=1, keepdim=True), None


def _objects(case, r):
    """Objects of three boxes or cylinders each, points on their surfaces, scaled to the unit ball."""
    m, n = case["points"], case["objects"]
    obj = torch.arange(m, device=DEV) * n // m
    prim = obj * 3 + r.pick(torch.ones(3, device=DEV), m)
    half = r.uniform(0.05, 0.5, 3 * n, 3)
    round_ = r.uniform(0, 1, 3 * n) < 0.5
    u = r.uniform(-1, 1, m, 3)
    # a box: one coordinate of the cube goes to its face
    axis = r.pick(torch.ones(3, device=DEV), m)
    box = u.scatter(1, axis[:, None], u.gather(1, axis[:, None]).sign())
    # a cylinder: side or caps
    th = math.pi * u[:, 0]
    cap = r.uniform(0, 1, m) < 0.3
    rad = torch.where(cap, u[:, 1].abs().sqrt(), torch.ones_like(th))
    cyl = torch.stack([rad * th.cos(), rad * th.sin(), torch.where(cap, u[:, 2].sign(), u[:, 2])], 1)
    p = torch.where(round_[prim, None], cyl, box) * half[prim]
    p = (_rotations(r, 3 * n)[prim] @ p[:, :, None])[:, :, 0] + r.uniform(-0.5, 0.5, 3 * n, 3)[prim]
    cnt = torch.zeros(n, 1, device=DEV).index_add_(0, obj, torch.ones(m, 1, device=DEV))
    p = p - (torch.zeros(n, 3, device=DEV).index_add_(0, obj, p) / cnt)[obj]
    p = p / torch.zeros(n, device=DEV).scatter_reduce_(0, obj, p.norm(dim=1), "amax")[obj, None]
    o = r.perm(m)
    return p[o], (obj[o].int() if n > 1 else None)


def _room(case, r):
    """A room of 8 x 8 x 3 m with 20 boxes on the floor, points on the surfaces with 5 mm of noise."""
    m, L, H = case["points"], 8.0, 3.0
    e = torch.eye(3, device=DEV)
    zero = torch.zeros(3, device=DEV)
    rects = [(zero, L * e[0], L * e[1]), (zero, L * e[1], H * e[2]), (L * e[0], L * e[1], H * e[2]),
             (zero, L * e[0], H * e[2]), (L * e[1], L * e[0], H * e[2])]
    o, u, v = (torch.stack(t) for t in zip(*rects))
    n = 20
    size = r.uniform(0, 1, n, 3) * torch.tensor([1.7, 1.7, 1.2], device=DEV) + 0.3
    yaw, at = r.uniform(0, 2 * math.pi, n), r.uniform(1.0, L - 1.0, n, 2)
    ax = torch.stack([yaw.cos(), yaw.sin(), 0 * yaw], 1) * size[:, :1]
    ay = torch.stack([-yaw.sin(), yaw.cos(), 0 * yaw], 1) * size[:, 1:2]
    az = torch.stack([0 * yaw, 0 * yaw, size[:, 2]], 1)
    c = torch.cat([at, 0 * yaw[:, None]], 1) - 0.5 * (ax + ay)
    o = torch.cat([o, c, c + ax, c, c + ay, c + az])
    u = torch.cat([u, ay, ay, ax, ax, ax])
    v = torch.cat([v, az, az, az, az, ay])
    nrm = torch.linalg.cross(u, v)
    area = nrm.norm(dim=1)
    nrm = nrm / area[:, None]
    s = r.pick(area, m)
    ab = r.uniform(0, 1, m, 2)
    p = o[s] + ab[:, :1] * u[s] + ab[:, 1:] * v[s] + nrm[s] * (0.005 * r.normal(m, 1))
    return p, None, torch.cat([r.uniform(0, 1, o.shape[0], 3)[s], nrm[s]], 1)


def _raycast(r, m, centre, half, yaw):
    """m returns of a 64-beam sensor at 1.73 m in scan order: ground and boxes within 50 m, 2 cm of noise."""
    n_az = -(-m * 5 // (64 * 4))
    while True:
        az = torch.arange(n_az, device=DEV) * (2 * math.pi / n_az)
        el = torch.deg2rad(torch.linspace(-25.0, 3.0, 64, device=DEV))
        d = torch.stack([el.cos()[None] * az.cos()[:, None], el.cos()[None] * az.sin()[:, None],
                         el.sin()[None].expand(n_az, 64)], 2).reshape(-1, 3)
        org = torch.tensor([0.0, 0.0, 1.73], device=DEV)
        best = torch.where(d[:, 2] < 0, -org[2] / d[:, 2], torch.full_like(d[:, 2], math.inf))
        rot = torch.stack([yaw.cos(), -yaw.sin(), 0 * yaw, yaw.sin(), yaw.cos(), 0 * yaw, 0 * yaw, 0 * yaw,
                           0 * yaw + 1], 1).view(-1, 3, 3)
        lo = ((org - centre)[:, None] @ rot)[:, 0]
        inv = 1 / (d @ rot.permute(1, 0, 2).reshape(3, -1)).view(-1, yaw.numel(), 3)
        t1, t2 = (-half - lo) * inv, (half - lo) * inv
        near = torch.minimum(t1, t2).amax(2)
        far = torch.maximum(t1, t2).amin(2)
        hit = torch.where((far >= near) & (near > 0), near, torch.full_like(near, math.inf)).amin(1)
        best = torch.minimum(best, hit)
        keep = torch.nonzero(best <= 50.0)[:, 0]
        if keep.numel() >= m:
            break
        n_az = n_az * 9 // 8 + 1
    keep = keep[r.perm(keep.numel())[:m].sort().values]
    return org + (best[keep] + 0.02 * r.normal(m))[:, None] * d[keep]


def _scan(case, r):
    m, n, k = case["points"], 40, max(1, case["objects"])
    rad = r.uniform(9.0, 2025.0, n).sqrt()
    ang = r.uniform(0, 2 * math.pi, n)
    half = r.uniform(0, 1, n, 3) * torch.tensor([2.75, 1.25, 1.25], device=DEV) + 0.25
    centre = torch.stack([rad * ang.cos(), rad * ang.sin(), half[:, 2]], 1)
    yaw = r.uniform(0, 2 * math.pi, n)
    if case["cloud"] == "scan":
        return _raycast(r, m, centre, half, yaw), None
    # every fourth box moves by up to 2 m from scan to scan; time is the fourth axis, half a unit a scan
    step = r.uniform(-1.4, 1.4, n, 3) * torch.tensor([1.0, 1.0, 0.0], device=DEV)
    step[torch.arange(n, device=DEV) % 4 != 0] = 0
    out = []
    for t in range(k):
        mt = (t + 1) * m // k - t * m // k
        p = _raycast(r, mt, centre + t * step, half, yaw)
        out.append(torch.cat([p, torch.full((mt, 1), 0.5 * t, device=DEV)], 1))
    return torch.cat(out), None


_CLOUDS = {"spheres": _spheres, "objects": _objects, "room": _room, "scan": _scan, "frames": _scan}


def _inputs(case, seed):
    """Positions, batch ids, point features, weights and point gradients of a case."""
    r = _Rng(seed)
    got = _CLOUDS[case["cloud"]](case, r)
    pos, batch = got[0].float().contiguous(), got[1]
    m, d, ch = case["points"], _dim(case), _chain(case)
    taps = 2 * (d + 1) + 1
    i = {"pos": pos, "batch": batch}
    if case["op"] in ("step", "unet"):
        if len(got) > 2:    # colour and normal, lifted to the first layer's width
            i["feat"] = (got[2] @ r.normal(6, ch[0])) / math.sqrt(6.0)
        else:
            i["feat"] = r.normal(m, ch[0])
    if case["op"] == "pointnet":
        f = case["f_d"]
        i["raw"] = got[2][:, :f].contiguous() if len(got) > 2 and f <= 6 else r.uniform(0, 1, m, f)
        k, i["layers"] = d + f, []
        for w in WIDTHS:
            i["layers"].append((1 + 0.1 * r.normal(k), 0.1 * r.normal(k), r.normal(w, k) * math.sqrt(2.0 / k),
                                0.01 * r.normal(w)))
            k = w
    else:
        def weight(a, b):
            w = r.normal(b, taps, a) / math.sqrt(2.0 * a)
            return w.bfloat16() if case["dtype"] == "bf16" else w
        i["w"] = [weight(a, b) for a, b in zip(ch, ch[1:])]
        if case["op"] == "unet":
            i["w_down"], i["w_up"] = weight(ch[-1], ch[-1]), weight(ch[-1], ch[-1])
    if case["op"] in ("head", "conv"):      # a smooth field of unit variance over the lattice
        i["freq"], i["phase"] = 0.15 * r.normal(d + 1, ch[0]), r.uniform(0, 2 * math.pi, ch[0])
    n_out = ch[-1]
    if case["classes"]:
        n_out = case["classes"]
        i["w_delta"], i["b_delta"] = r.normal(ch[-1]) / math.sqrt(ch[-1]), 0.25
        i["w_cls"], i["b_cls"] = r.normal(n_out, ch[-1]) / math.sqrt(ch[-1]), 0.1 * r.normal(n_out)
    if case["train"]:
        i["g"] = r.normal(m, n_out)
    return i


def _field(keys, i):
    return (1.4142135 * torch.sin(keys.double() @ i["freq"].double() + i["phase"].double())).float()


# -- the passes ----------------------------------------------------------------

def prepare(case, seed):
    i = _inputs(case, seed)
    s = dict(i, case=case)
    s["L"] = Lattice(_dim(case), case["sigma"], max_points=case["points"])
    if case["op"] == "unet":
        s["Lc"] = Lattice(_dim(case), 2 * case["sigma"], max_points=case["points"])
    if case["op"] == "pointnet":
        s["params"] = Lattice.pack_pointnet([[t.cpu() for t in b] for b in i["layers"]]).to(DEV)
    if case["op"] in ("head", "conv"):
        s["L"].splat(s["pos"], None, s["batch"], want_weight=False)
        s["x"] = _field(s["L"].keys(), i)
        if case["op"] == "conv":
            s["L"].build_neighbors()
            if case["dtype"] == "bf16":
                s["x"] = s["x"].bfloat16()
    return s


def _convs(s, stored_last):
    """The chain's convolutions; a row is stored in 16 bits where the next layer reads it so."""
    L, dt = s["L"], s["case"]["dtype"]
    x, _ = L.splat(s["pos"], s["feat"], s["batch"], want_weight=False, values_dtype=dt)
    L.build_neighbors()
    xs = [x]
    for k, w in enumerate(s["w"]):
        last = k == len(s["w"]) - 1
        xs.append(L.conv(xs[-1], w, dtype=dt, out_dtype=stored_last if last else dt))
    return xs


def _convs_backward(s, xs, g):
    """From the gradient of the last layer's rows to the point features': (dL/dfeat, every dL/dW)."""
    L, dt = s["L"], s["case"]["dtype"]
    gws = []
    for k in reversed(range(len(s["w"]))):
        g, gw, _ = L.conv_backward(g, s["w"][k], xs[k], dtype=dt, grad_in_dtype=dt if k else "f32")
        gws.append(gw)
    return [L.splat_backward(g)] + gws[::-1]


def _run_head(s):
    L, train = s["L"], s["case"]["train"]
    out = [L.deform_slice(s["x"], s["w_delta"], s["b_delta"], s["w_cls"], s["b_cls"])]
    if train:
        g = L.deform_slice_backward(s["x"], s["w_delta"], s["b_delta"], s["g"], w_cls=s["w_cls"])
        out += [L.splat_backward(g[0])] + list(g[1:])
    return out


def _run_conv(s):
    L = s["L"]
    return [L.slice(L.conv(s["x"], s["w"][0], dtype=s["case"]["dtype"]))]


def _run_step(s):
    L, case = s["L"], s["case"]
    xs = _convs(s, "f32")
    if case["tail"] == "deform":
        out = [L.deform_slice(xs[-1], s["w_delta"], s["b_delta"], s["w_cls"], s["b_cls"])]
    else:
        out = [L.slice(xs[-1])]
    if case["train"]:
        if case["tail"] == "deform":
            g = L.deform_slice_backward(xs[-1], s["w_delta"], s["b_delta"], s["g"], w_cls=s["w_cls"],
                                        grad_dtype=case["dtype"])
            out += list(g[1:])
        else:
            g = [L.slice_backward(s["g"], out_dtype=case["dtype"])]
        out += _convs_backward(s, xs, g[0])
    return out


def _run_unet(s):
    L, Lc, dt = s["L"], s["Lc"], s["case"]["dtype"]
    xs = _convs(s, dt)
    Lc.splat(s["pos"], None, s["batch"], want_weight=False)
    xc = L.downsample(Lc, xs[-1], s["w_down"], dtype=dt, out_dtype=dt)
    out = [L.slice(Lc.upsample(L, xc, s["w_up"], dtype=dt))]
    if s["case"]["train"]:
        g = L.slice_backward(s["g"])
        gc, gw_up, _ = Lc.upsample_backward(L, g, s["w_up"], x=xc, dtype=dt, grad_in_dtype=dt)
        gf, gw_down, _ = L.downsample_backward(Lc, gc, s["w_down"], x=xs[-1], dtype=dt, grad_in_dtype=dt)
        out += [gw_up, gw_down] + _convs_backward(s, xs, gf)
    return out


def _run_pointnet(s):
    L = s["L"]
    L.splat(s["pos"], None, s["batch"], want_weight=False)
    x = L.distribute_pointnet(s["pos"], s["raw"], s["params"], groups="default")
    out = [L.slice(x)]
    if s["case"]["train"]:
        g = L.slice_backward(s["g"])
        out.append(L.distribute_pointnet_backward(s["pos"], s["raw"], s["params"], g, groups="default"))
    return out


def run(state):
    return {"head": _run_head, "conv": _run_conv, "step": _run_step, "unet": _run_unet,
            "pointnet": _run_pointnet}[state["case"]["op"]](state)


# -- the same in 64 bits ---------------------------------------------------------

class _Ref:
    """The lattice of a cloud in plain torch.  Which simplex holds a point is decided in
    32 bits, each operation rounded by itself, as the library's interface states; weights
    and values are in 64 bits from there on."""

    def __init__(self, pos, batch, sigma):
        m, d = pos.shape
        n = d + 1
        sig = torch.tensor(sigma, dtype=torch.float32).double().item()
        S = torch.zeros(m, device=pos.device)
        x = [None] * n
        for j in range(d, 0, -1):
            f = torch.tensor(n * math.sqrt(2.0 / 3.0) / (sig * math.sqrt(j * (j + 1.0)))).float().item()
            s = pos[:, j - 1] * f
            x[j] = S - s * float(j)
            S = S + s
        x[0] = S
        x = torch.stack(x, 1)
        r = torch.round(x * torch.tensor(1.0 / n).float().item()).long() * n
        delta = x - r.float()
        a, b = delta[:, :, None], delta[:, None, :]
        lower = torch.ones(n, n, device=pos.device).tril(-1).bool()[None]      # j < i
        rank = ((b > a) | ((b == a) & lower)).sum(2)
        rank = rank + (r.sum(1) // n)[:, None]
        neg, big = rank < 0, rank > d
        rank = rank + n * neg.long() - n * big.long()
        r = r + n * neg.long() - n * big.long()
        z = torch.zeros(m, n, device=pos.device, dtype=torch.float64)
        z.scatter_(1, rank, (x.double() - r) / n)
        self.bary = torch.cat([(1 - z[:, :1] + z[:, d:])] + [z[:, d - k:d - k + 1] - z[:, n - k:n - k + 1]
                                                               for k in range(1, n)], 1)
        k = torch.arange(n, device=pos.device)[None, :, None]
        keys = r[:, None, :] + k - n * (rank[:, None, :] > d - k).long()
        bid = batch.long()[:, None, None] if batch is not None else torch.zeros_like(keys[:, :1, :1])
        rows = torch.cat([bid.expand(m, n, 1), keys[:, :, :d]], 2).reshape(m * n, n)
        self.table, idx = torch.unique(self._pack(rows), return_inverse=True)
        self.idx = idx.view(m, n)
        self.V, self.d, self.n = self.table.numel(), d, n
        self.rows = torch.empty(self.V, n, dtype=torch.long, device=pos.device)
        self.rows[idx] = rows
        self.keys = torch.cat([self.rows[:, 1:], -self.rows[:, 1:].sum(1, keepdim=True)], 1)

    def _pack(self, rows):
        """(batch, c_0 .. c_{d-1}) in one ordered integer; coordinates and batch ids keep within 12 bits here."""
        p = torch.zeros(rows.shape[0], dtype=torch.long, device=rows.device)
        for j in range(rows.shape[1]):
            p = p * 8192 + (rows[:, j] + 4096)
        return p

    def find(self, keys, bid):
        q = self._pack(torch.cat([bid, keys[:, :self.d]], 1))
        at = torch.searchsorted(self.table, q).clamp_(max=self.V - 1)
        return torch.where(self.table[at] == q, at, torch.full_like(at, -1))

    def offsets(self):
        o = self.n * torch.eye(self.n, dtype=torch.long, device=self.rows.device) - 1
        return torch.cat([torch.zeros_like(o[:1]), o, -o])

    def neighbors(self):
        return [self.find(self.keys + o, self.rows[:, :1]) for o in self.offsets()]

    def down(self, fine):
        return [fine.find(2 * self.keys + o, self.rows[:, :1]) for o in fine.offsets()]

    def up(self, coarse):
        got = []
        for o in self.offsets():
            k = self.keys + o
            at = coarse.find(torch.div(k, 2, rounding_mode="floor"), self.rows[:, :1])
            got.append(torch.where((k % 2 == 0).all(1), at, torch.full_like(at, -1)))
        return got

    def splat(self, f):
        w = self.bary[:, :, None] * f[:, None, :]
        return torch.zeros(self.V, f.shape[1], dtype=f.dtype, device=f.device).index_add(
            0, self.idx.reshape(-1), w.reshape(-1, f.shape[1]))

    def slice(self, x):
        return (self.bary[:, :, None] * x[self.idx]).sum(1)


def _ref_conv(x, table, w):
    x = torch.cat([x, torch.zeros_like(x[:1])])      # row -1: an absent neighbour
    y = 0
    for t, at in enumerate(table):
        y = y + x[at] @ w[:, t].t()
    return y


def _ref_deform(ref, x, i):
    q = ref.bary[:, :, None] * x[ref.idx]
    db = torch.tanh(i["b_delta"] + (q - q.max(1, keepdim=True).values) @ i["w_delta"])
    f = ((ref.bary + db)[:, :, None] * x[ref.idx]).sum(1)
    return f @ i["w_cls"].t() + i["b_cls"]


def _ref_pointnet(ref, i, layers):
    pos, n = i["pos"].double(), ref.n
    at = ref.idx.reshape(-1)
    rep = pos.repeat_interleave(n, 0)
    cnt = torch.zeros(ref.V, 1, dtype=pos.dtype, device=pos.device).index_add(0, at, torch.ones_like(rep[:, :1]))
    mean = torch.zeros(ref.V, ref.d, dtype=pos.dtype, device=pos.device).index_add(0, at, rep) / cnt
    h = torch.cat([rep - mean[at], i["raw"].double().repeat_interleave(n, 0)], 1)
    cloud = i["batch"].long().repeat_interleave(n) if i["batch"] is not None else torch.zeros_like(at)
    nb = int(cloud.max()) + 1
    num = torch.zeros(nb, 1, dtype=pos.dtype, device=pos.device).index_add(0, cloud, torch.ones_like(rep[:, :1]))

    def mean_of(v):
        return (torch.zeros(nb, v.shape[1], dtype=v.dtype, device=v.device).index_add(0, cloud, v) / num)[cloud]
    for gamma, beta, w, b in layers:     # as many groups as channels: every channel by itself
        h = h - mean_of(h)
        h = h / torch.sqrt(mean_of(h * h) + 1e-5)
        h = torch.relu(gamma * h + beta) @ w.t() + b
    return torch.full((ref.V, 64), -math.inf, dtype=h.dtype, device=h.device).scatter_reduce(
        0, at[:, None].expand(-1, 64), h, "amax", include_self=False)


def exact(case, seed):
    i = _inputs(case, seed)
    ref = _Ref(i["pos"], i["batch"], case["sigma"])

    def leaf(t):
        return t.double().requires_grad_(case["train"])
    d = {k: leaf(i[k]) for k in ("feat", "w_delta", "w_cls", "b_cls", "w_down", "w_up") if k in i}
    ws = [leaf(w) for w in i.get("w", ())]
    layers = [[leaf(t) for t in b] for b in i.get("layers", ())]
    if "b_delta" in i:
        d["b_delta"] = leaf(torch.tensor([i["b_delta"]], device=DEV))
    if case["op"] in ("step", "unet"):
        x = ref.splat(d["feat"])
        table = ref.neighbors()
        for w in ws:
            x = _ref_conv(x, table, w)
    if case["op"] == "head":
        x = leaf(_field(ref.keys, i))
        out = _ref_deform(ref, x, d)
        wrt = [x] + [d[k] for k in ("w_delta", "b_delta", "w_cls", "b_cls")]
    elif case["op"] == "conv":
        x = _field(ref.keys, i)
        x = x.bfloat16() if case["dtype"] == "bf16" else x
        out = ref.slice(_ref_conv(x.double(), ref.neighbors(), ws[0]))
    elif case["op"] == "step":
        deform = case["tail"] == "deform"
        out = _ref_deform(ref, x, d) if deform else ref.slice(x)
        wrt = ([d[k] for k in ("w_delta", "b_delta", "w_cls", "b_cls")] if deform else []) + [d["feat"]] + ws
    elif case["op"] == "unet":
        coarse = _Ref(i["pos"], i["batch"], 2 * case["sigma"])
        x = _ref_conv(x, coarse.down(ref), d["w_down"])
        out = ref.slice(_ref_conv(x, ref.up(coarse), d["w_up"]))
        wrt = [d["w_up"], d["w_down"], d["feat"]] + ws
    else:
        out = ref.slice(_ref_pointnet(ref, i, layers))
        wrt = [t for b in layers for t in b]
    if not case["train"]:
        return [out]
    g = list(torch.autograd.grad(out, wrt, i["g"].double()))
    if case["op"] == "head":
        g[0] = ref.slice(g[0])
    if case["op"] == "pointnet":
        g = [torch.cat([t.reshape(-1) for t in g])]
    return [out.detach()] + g


# -- what a pass cannot do without -------------------------------------------------

def work(case):
    """Bytes: every array that goes into or comes out of a call read or written once, with the lattice's
    own records (a vertex and a weight a pair, the ring table).  Operations: multiplications and additions."""
    i = _inputs(case, 1)
    V = _Ref(i["pos"], i["batch"], case["sigma"]).V
    m, n, ch, k = case["points"], _dim(case) + 1, _chain(case), case["classes"]
    taps, train = 2 * n + 1, case["train"]
    e = 2 if case["dtype"] == "bf16" else 4
    pairs, ring = 8 * m * n, 4 * V * taps
    b = f = 0

    def conv(a, c, ea, ec, rows_in, rows_out):
        nonlocal b, f
        b += rows_in * a * ea + rows_out * c * ec + a * c * taps * e + 4 * rows_out * taps
        f += 2 * rows_out * taps * a * c
        if train:       # input and weight gradients
            b += rows_in * a * (ea + e) + rows_out * c * ec + a * c * taps * (e + 4) + 4 * rows_out * taps
            f += 4 * rows_out * taps * a * c
    if case["op"] in ("step", "unet"):
        b += 4 * m * (n - 1) + 4 * m * ch[0] + pairs + e * V * ch[0] + ring     # splat, neighbour table
        f += 2 * m * n * ch[0]
        for a, c in zip(ch, ch[1:]):
            conv(a, c, e, 4, V, V)
        if train:
            b += 4 * m * ch[0] + pairs
            f += 2 * m * n * ch[0]
    if case["op"] == "unet":
        Vc = _Ref(i["pos"], i["batch"], 2 * case["sigma"]).V
        b += 4 * m * (n - 1) + 4 * taps * (V + Vc)
        conv(ch[-1], ch[-1], e, e, V, Vc)
        conv(ch[-1], ch[-1], e, 4, Vc, V)
    if case["op"] == "conv":
        conv(ch[0], ch[1], e, 4, V, V)
    if case["op"] == "pointnet":
        c0 = n - 1 + case["f_d"]
        mac = 16 * c0 + 32 * 16 + 64 * 32
        b += 8 * m * (n - 1) + 4 * m * case["f_d"] + 2 * pairs + 4 * V * 64
        f += 2 * m * n * mac
        if train:
            b += 4 * m * c0 + pairs + 2 * 4 * V * 64
            f += 6 * m * n * mac
    c = ch[-1]
    if k:               # DeformSlice and the classifier
        b += 4 * V * c + pairs + 4 * m * k + 4 * c * k
        f += m * (6 * n * c + 2 * c * k)
        if train:
            b += 8 * V * c + pairs + 4 * m * k + 8 * c * k
            f += m * (12 * n * c + 4 * c * k)
            if case["op"] == "head":
                b += 4 * V * c + pairs + 4 * m * c
                f += 2 * m * n * c
    else:
        b += 4 * V * c + pairs + 4 * m * c
        f += 2 * m * n * c
        if train:
            b += e * V * c + pairs + 4 * m * c
            f += 2 * m * n * c
    return {"bytes": b, "flops": f}


def tolerance(case):
    """About four times what the passes show against exact() and between two runs (vertex order, and with it the
    order of sums, changes from run to run)."""
    if case["op"] == "pointnet" and case["train"]:      # near ties of the maximum: 1.3e-3 against 64 bits
        return {"rel": 5e-3}
    deform = case["op"] == "head" or case["tail"] == "deform"
    if case["op"] != "head" and deform and case["train"]:
        # which vertex wins the maximum follows from rounded rows: a flip moves a whole gradient term
        # (2.7e-2 against 64 bits with 16-bit rows, 9.2e-4 with 32-bit ones)
        return {"rel": 0.1 if case["dtype"] == "bf16" else 4e-3}
    if case["dtype"] == "bf16":                         # 3.4e-3
        return {"rel": 1.5e-2}
    if deform and case["train"]:                        # one flip in a small cloud
        return {"rel": 1e-4}
    return {"rel": 3e-5 if deform or case["op"] == "pointnet" else 1e-5}   # 7.8e-6; 1.3e-6
