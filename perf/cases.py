"""The work that a user of the library has it do, as cases that can be timed.

Every case goes through the public calls of paper_2603_18401_amd on synthetic
image pairs made on the GPU from a seed.  A pair is two views of 3-D points
5-15 m away under one of the four motions that set the epipole (near-pure
sideways, exactly sideways, forward, general), 70 % of the smaller keypoint
set true partners with 0.5 px noise, the rest uniform outliers; descriptors
are unit rows with N(0, 0.05^2) noise between the views.  The image sizes,
keypoint counts, tolerances and batch shapes are those of the repository's
benchmark workloads.

A case's "do" names the call that it stands for:

  query    Index + query_match / query_match_bf16 / query_match_fp8
  match    Index + query, then match over that CSR
  replay   Batch.launch of a recorded batch, F read on the device
  mutual   both directions, the cross-check and the GMS filter
  train    one minibatch of the tolerance network (gradient and Adam)
  infer    keypoint features and the predicted tolerances
  encode   the reduced formats and their rounding-error bounds
"""

import math
import random

import numpy as np
import torch

import paper_2603_18401_amd as epm
from paper_2603_18401_amd import learned_eps

SIZES = ((640, 480), (1920, 1080), (4032, 3024), (6048, 4032))
IN, HID, NPARAM = 6, 64, learned_eps.NPARAM
SHAPES = ((HID, IN), (HID,), (HID, HID), (HID,), (1, HID), (1,))


def _case(name, do, pairs=1, kp_min=1000, kp_max=1000, size=3, eps=2.0, eps_per_keypoint=False,
          dtype="f32", ratio=0.8, sync=False, **more):
    return dict(name=name, do=do, pairs=pairs, kp_min=kp_min, kp_max=kp_max, size=size, eps=eps,
                eps_per_keypoint=eps_per_keypoint, dtype=dtype, ratio=ratio, sync=sync, **more)


def listed():
    return [
        # one frame pair of a sequence as it arrives: a thousand keypoints,
        # its candidate count waited for, as the call does by default -- launches and latency
        _case("vga_pair_f32", "query", size=0, sync=True),
        # a few multi-megapixel pairs of an SfM run at tolerances of 1-4 px
        _case("six_24mp_pairs_f32", "query", pairs=6, kp_min=20000, kp_max=20000,
              eps_per_keypoint=True, ratio=0.0),
        # the batching workload: 512 uneven pairs at once, BF16 rows
        _case("batch_512_bf16", "query", pairs=512, kp_min=500, kp_max=30000, size=-1,
              dtype="bf16", ratio=0.0),
        # a service that replays one recorded batch on new inputs and new F
        _case("replay_48_bf16", "replay", pairs=48, kp_min=500, kp_max=10000, size=-1,
              dtype="bf16"),
        # the paper's own tolerances (25-100 px): over a thousand candidates a query
        _case("six_50k_wide_f32", "query", pairs=6, kp_min=50000, kp_max=50000, eps=50.0,
              eps_per_keypoint=True, ratio=0.0),
        # one very dense pair with the map's descriptors kept in FP8
        _case("dense_60k_fp8", "query", kp_min=60001, kp_max=60001, dtype="fp8"),
        # candidates first, matching over them afterwards: BF16 and binary rows
        _case("csr_60k_bf16", "match", kp_min=60000, kp_max=60000, dtype="bf16"),
        _case("csr_60k_bin256", "match", kp_min=60000, kp_max=60000, dtype="bin256"),
        # both directions with cross-check and GMS over a small group of pairs
        _case("mutual_8_gms", "mutual", pairs=8, kp_min=7000, kp_max=9000, size=2, eps=3.0),
        # a training step of the tolerance network at its default batch
        dict(name="train_65536", do="train", batch=65536),
        # the learned tolerances of a batch of 200 pairs of 10000 keypoints
        dict(name="infer_2m", do="infer", pairs=200, kp=10000),
        # a map's descriptors brought into the reduced formats
        dict(name="encode_500k", do="encode", rows=500003),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    do = rng.choice(("query", "query", "query", "match", "match", "replay", "mutual", "train",
                     "infer", "encode"))
    if do == "train":
        return dict(do=do, batch=_log_int(rng, 256, 65536))
    if do == "infer":
        return dict(do=do, pairs=rng.randint(1, 200), kp=_log_int(rng, 100, 10000))
    if do == "encode":
        return dict(do=do, rows=_log_int(rng, 1000, 500000))
    dtype = {"query": ("f32", "bf16", "fp8"), "match": ("f32", "bf16", "bin256"),
             "replay": ("f32", "bf16"), "mutual": ("f32",)}[do]
    kp_max = _log_int(rng, 500, 60000)
    c = _case("", do, pairs=_log_int(rng, 1, 64), kp_min=max(100, int(kp_max * rng.uniform(0.05, 1))),
              kp_max=kp_max, size=rng.randint(-1, 3), eps=math.exp(rng.uniform(0.0, math.log(50.0))),
              eps_per_keypoint=rng.random() < 0.5, dtype=rng.choice(dtype),
              ratio=rng.choice((0.0, 0.8)), sync=do == "query" and rng.random() < 0.3)
    del c["name"]
    # at most 300000 keypoints and 100 million candidates in all (30 million
    # where a separate match, or a second direction, reads the rows again)
    c["pairs"] = max(1, min(c["pairs"], 300000 // c["kp_max"]))
    most = 1e8 if do == "query" else 3e7
    while _candidates(c) > most and c["eps"] > 1.0:
        c["eps"] = max(1.0, c["eps"] * 0.7)
    return c


# ------------------------------------------------------------------ shapes

def _shapes(case):
    """(W, H, m, n) of every pair: the same for every seed."""
    rng = random.Random("%(pairs)d %(kp_min)d %(kp_max)d %(size)d" % case)
    out = []
    for _ in range(case["pairs"]):
        W, H = SIZES[case["size"] if case["size"] >= 0 else rng.randint(1, 3)]
        out.append((W, H, _log_int(rng, case["kp_min"], case["kp_max"]),
                    _log_int(rng, case["kp_min"], case["kp_max"])))
    return out


def _mean_eps(case):
    return case["eps"] * (7.0 / 6.0 if case["eps_per_keypoint"] else 1.0)


def _candidates(case):
    """Expected candidates: a band of 2 eps along a line of about 0.9 W."""
    return sum(m * n * 1.8 * _mean_eps(case) / H for W, H, m, n in _shapes(case))


# ------------------------------------------------------------------ scenes

def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) + 2603)
    return g


def _rotation(axis, angle):
    a = axis / np.linalg.norm(axis)
    k = np.array([[0, -a[2], a[1]], [a[2], 0, -a[0]], [-a[1], a[0], 0]])
    return np.eye(3) + np.sin(angle) * k + (1 - np.cos(angle)) * (k @ k)


def _pose(rng, kind):
    """Rotation and centre of camera 2 (X2 = R (X1 - C), |C| = 1 m)."""
    sign = 1.0 if rng.random() < 0.5 else -1.0
    if kind == 0:    # near-pure sideways: the epipole far outside the image
        return _rotation(np.array([0.0, 1.0, 0.0]),
                         sign * np.deg2rad(10.0 ** rng.uniform(-4.0, 1.0))), np.array([1.0, 0.0, 0.0])
    if kind == 3:    # exactly sideways: the epipole at infinity
        return np.eye(3), np.array([1.0, 0.0, 0.0])
    if kind == 1:    # forward: the epipole inside the image
        C = np.array([rng.uniform(-0.1, 0.1), rng.uniform(-0.1, 0.1), 1.0])
        return _rotation(rng.standard_normal(3), np.deg2rad(rng.uniform(0.0, 2.0))), C / np.linalg.norm(C)
    C = rng.standard_normal(3)
    return _rotation(rng.standard_normal(3), np.deg2rad(rng.uniform(0.0, 15.0))), C / np.linalg.norm(C)


def _skew(t):
    return np.array([[0, -t[2], t[1]], [t[2], 0, -t[0]], [-t[1], t[0], 0]])


def _scene(case, seed):
    """Keypoints, tolerances, cameras and descriptors of a batch of pairs."""
    g = _generator(seed)
    rng = np.random.default_rng(int(seed))
    shapes = _shapes(case)
    P, dev = len(shapes), "cuda"
    F, Ks, Rs, ts = [], [], [], []
    for p, (W, H, m, n) in enumerate(shapes):
        R, C = _pose(rng, 3 if p == 0 and P >= 8 else p % 3)
        f, t = 0.5622 * W, -R @ C
        Ki = np.array([[1 / f, 0, -0.5 * W / f], [0, 1 / f, -0.5 * H / f], [0, 0, 1.0]])
        F.append(Ki.T @ _skew(t) @ R @ Ki)
        Ks.append((f, 0.5 * W, 0.5 * H))
        Rs.append(R)
        ts.append(t)

    def rows(counts):
        return torch.repeat_interleave(torch.arange(P, device=dev), torch.tensor(counts, device=dev))

    def uniform(n, c=1):
        return torch.rand((n, c), generator=g, device=dev, dtype=torch.float64)

    m, n = [s[2] for s in shapes], [s[3] for s in shapes]
    n1, n2 = sum(m), sum(n)
    true = [int(0.7 * min(a, b)) for a, b in zip(m, n)]
    start = [np.concatenate([[0], np.cumsum(c)])[:-1] for c in (m, n)]
    pt = rows(true)
    within = torch.arange(sum(true), device=dev) - torch.tensor(
        np.concatenate([[0], np.cumsum(true)])[:-1], device=dev)[pt]
    i1 = torch.tensor(start[0], device=dev)[pt] + within
    i2 = torch.tensor(start[1], device=dev)[pt] + within
    K, R, t = (torch.tensor(np.array(v), device=dev) for v in (Ks, Rs, ts))
    wh = torch.tensor([[s[0], s[1]] for s in shapes], device=dev, dtype=torch.float64)
    kp1 = uniform(n1, 2) * wh[rows(m)]
    kp2 = uniform(n2, 2) * wh[rows(n)]
    # image-1 pixels at a depth, seen from camera 2; those it does not see stay outliers
    z = 5.0 + 10.0 * uniform(len(pt))
    X = torch.cat([(kp1[i1] - K[pt, 1:]) / K[pt, :1], torch.ones_like(z)], 1) * z
    X = (R[pt] * X[:, None, :]).sum(2) + t[pt]
    x = X[:, :2] / X[:, 2:] * K[pt, :1] + K[pt, 1:]
    seen = (X[:, 2:] > 1e-3) & (x >= 0).all(1, keepdim=True) & (x < wh[pt]).all(1, keepdim=True)
    noise = 0.5 * torch.randn((2, len(pt), 2), generator=g, device=dev, dtype=torch.float64)
    kp1[i1] += noise[0]
    kp2[i2] = torch.where(seen, x + noise[1], kp2[i2])
    # every image lists its keypoints in an order of its own
    o1 = torch.argsort(rows(m) + uniform(n1)[:, 0])
    o2 = torch.argsort(rows(n) + uniform(n2)[:, 0])
    s = {"F": F, "g": g, "m": m, "n": n, "n1": n1, "n2": n2, "shapes": shapes,
         "kp1": kp1[o1].float(), "kp2": kp2[o2].float()}
    s["specs"] = [epm.PairSpec(f, W, H, a, b) for f, (W, H, a, b) in zip(F, shapes)]

    def tolerances(k):
        if not case["eps_per_keypoint"]:
            return None
        return case["eps"] * 2.0 ** torch.randint(-1, 2, (k,), generator=g, device=dev).float()

    s["eps2"], s["eps1"] = tolerances(n2), tolerances(n1)
    if case["dtype"] == "bin256":
        def bits(k):
            return torch.randint(-2 ** 31, 2 ** 31, (k, 8), generator=g, device=dev).int()
        b1, b2 = bits(n1), bits(n2)
        flips = torch.zeros((len(pt), 8), dtype=torch.int64, device=dev)
        for b in range(32):
            flips += (torch.rand((len(pt), 8), generator=g, device=dev) < 0.08).long() << b
        b2[i2] = torch.where(seen, b1[i1] ^ flips.int(), b2[i2])
        s["d1"], s["d2"] = b1[o1].contiguous(), b2[o2].contiguous()
    else:
        def unit(x):
            return x / x.norm(dim=1, keepdim=True)
        d1 = unit(torch.randn((n1, 128), generator=g, device=dev))
        d2 = unit(torch.randn((n2, 128), generator=g, device=dev))
        both = unit(torch.randn((len(pt), 128), generator=g, device=dev))
        noisy = [unit(both + 0.05 * torch.randn(both.shape, generator=g, device=dev)) for _ in range(2)]
        d1[i1] = torch.where(seen, noisy[0], d1[i1])
        d2[i2] = torch.where(seen, noisy[1], d2[i2])
        s["d1"], s["d2"] = d1[o1], d2[o2]
    return s


# ---------------------------------------------------------- tolerance network

def _parameters(rng):
    parts = []
    for shape in SHAPES:
        lim = math.sqrt(6.0 / shape[-1]) if len(shape) == 2 else 0.05
        parts.append(rng.uniform(-lim, lim, shape) * (0.3 if shape == (1, HID) else 1.0))
    parts[5][:] = 1.9
    return np.concatenate([p.reshape(-1) for p in parts]).astype(np.float32)


def _split(params):
    out, at = [], 0
    for shape in SHAPES:
        k = int(np.prod(shape))
        out.append(params[at:at + k].reshape(shape))
        at += k
    return out


def _network(params, x):
    w1, b1, w2, b2, w3, b3 = _split(params)
    a1 = x @ w1.T + b1
    a2 = torch.relu(a1) @ w2.T + b2
    return a1, a2, (torch.relu(a2) @ w3.T + b3)[:, 0]


def _attributes(g, n):
    """Keypoint scale (px), detector response and orientation."""
    u = torch.rand((n, 3), generator=g, device="cuda")
    return torch.stack([12.0 ** u[:, 0], u[:, 1], (2 * u[:, 2] - 1) * math.pi], 1).contiguous()


def _training(case, seed):
    """Features, residual targets and a minibatch, some way into a training."""
    g = _generator(seed)
    rng = np.random.default_rng(int(seed))
    rows = 4 * case["batch"]
    x = torch.cat([_attributes(g, rows), 2 * torch.rand((rows, 2), generator=g, device="cuda") - 1,
                   7 * torch.rand((rows, 1), generator=g, device="cuda")], 1).contiguous()
    y = (0.15 * x[:, 0] * torch.randn(rows, generator=g, device="cuda")).abs()
    params = _parameters(rng)
    # a sample on a kink of the network or of the loss has two gradients:
    # the minibatch is drawn from the others
    a1, a2, z = _network(torch.tensor(params, device="cuda").double(), x.double())
    away = torch.minimum(torch.minimum(a1.abs().amin(1), a2.abs().amin(1)),
                         (torch.nn.functional.softplus(z) - y).abs())
    pick = torch.rand(rows, generator=g, device="cuda") + 2.0 * (away < 2e-5)
    order = torch.argsort(pick)[:case["batch"]].int()
    v = np.square(rng.uniform(0.5, 2.0, NPARAM) * 1e-2).astype(np.float32)
    m = (rng.standard_normal(NPARAM) * 3e-3).astype(np.float32)
    return {"x": x, "y": y, "order": order, "params": params, "m": m, "v": v, "t": 500}


# ------------------------------------------------------------------ the calls

def prepare(case, seed):
    do = case["do"]
    if do == "train":
        s = _training(case, seed)
        tr = learned_eps.Trainer(s["params"], torch.device("cuda"))
        tr.m.copy_(torch.tensor(s["m"]))
        tr.v.copy_(torch.tensor(s["v"]))
        tr.t = s["t"]
        return {"case": case, "trainer": tr, "x": s["x"], "y": s["y"], "order": s["order"]}
    if do == "infer":
        c = dict(case, do="query", kp_min=case["kp"], kp_max=case["kp"], size=3, eps=2.0,
                 eps_per_keypoint=False, dtype="bin256")
        s = _scene(c, seed)
        params = torch.tensor(_parameters(np.random.default_rng(int(seed))), device="cuda")
        return {"case": case, "specs": s["specs"], "kp2": s["kp2"],
                "attrs": _attributes(s["g"], s["n2"]), "params": params, "F": s["F"]}
    if do == "encode":
        d = torch.randn((case["rows"], 128), generator=_generator(seed), device="cuda")
        return {"case": case, "d": d / d.norm(dim=1, keepdim=True)}
    s = _scene(case, seed)
    s["case"] = case
    if do == "mutual":
        s["sizes"] = [(W, H) for W, H, _, _ in s["shapes"]]
        s["rspecs"] = epm.reversed_specs(s["specs"], s["sizes"])
        return s
    if case["dtype"] == "bf16":
        s["c1"], s["c2"] = epm.quantize(s["d1"], "bf16"), epm.quantize(s["d2"], "bf16")
    if case["dtype"] == "fp8":
        s["c2"], s["scale2"] = epm.quantize(s["d2"], "fp8")
        s["err2"] = epm.rounding_error(s["d2"], s["c2"], "fp8", s["scale2"])
    # a program that calls again and again keeps its workspace and its output
    # buffers, the columns with room for more than it expects
    room = int(2.5 * _candidates(case)) + 8192
    idx = epm.Index(s["specs"], s["kp2"], eps2=s["eps2"], eps=case["eps"])
    s["workspace"] = idx.workspace
    idx.close()
    if do == "replay":
        code = {"bf16": dict(desc1_f32=s["d1"], desc2_f32=s["d2"])}.get(case["dtype"], {})
        Fd = torch.tensor(np.array(s["F"]).reshape(-1, 9), device="cuda")
        s["batch"] = epm.Batch(s["specs"], s["kp1"], s["kp2"], s.get("c1", s["d1"]),
                               s.get("c2", s["d2"]), room, eps2=s["eps2"], eps=case["eps"],
                               dtype=case["dtype"], ratio=case["ratio"], workspace=s["workspace"],
                               F_dev=Fd, **code)
        s["batch"].col_indices.zero_()
        return s
    s["offsets"] = torch.zeros(s["n1"] + 1, dtype=torch.int64, device="cuda")
    s["cols"] = torch.zeros(room, dtype=torch.int32, device="cuda")
    s["out"] = (torch.zeros(s["n1"], dtype=torch.int32, device="cuda"),
                torch.zeros(s["n1"], dtype=torch.float32, device="cuda"),
                torch.zeros(s["n1"], dtype=torch.float32, device="cuda"))
    return s


def run(s):
    case = s["case"]
    do = case["do"]
    if do == "train":
        tr = s["trainer"]
        loss = tr.step(s["x"], s["y"], s["order"])
        return {"loss": loss, "grad": tr.grad_buf, "params": tr.params, "m": tr.m, "v": tr.v}
    if do == "infer":
        f = learned_eps.features(s["specs"], s["kp2"], s["attrs"])
        return {"features": f, "eps": learned_eps.infer(f, s["params"])}
    if do == "encode":
        codes, scale = epm.quantize(s["d"], "fp8")
        err = epm.rounding_error(s["d"], codes, "fp8", scale)
        half = epm.quantize(s["d"], "bf16")
        return {"fp8": codes, "scale": scale, "error": err, "bf16": half,
                "bf16_error": epm.rounding_error(s["d"], half, "bf16")}
    if do == "replay":
        s["batch"].launch()
        b = s["batch"]
        return {"offsets": b.row_offsets, "cols": b.col_indices, "best": b.best_idx,
                "dist": b.best_dist, "second": b.second_dist}
    if do == "mutual":
        fwd = epm.Index(s["specs"], s["kp2"], eps2=s["eps2"], eps=case["eps"])
        rev = epm.Index(s["rspecs"], s["kp1"], eps2=s["eps1"], eps=case["eps"])
        _, _, b12, d12, s12 = fwd.query_match(s["kp1"], s["d1"], s["d2"], ratio=case["ratio"])
        _, _, b21, d21, s21 = rev.query_match(s["kp2"], s["d2"], s["d1"], ratio=case["ratio"])
        both = fwd.mutual(b12, b21)
        kept = fwd.gms(s["sizes"], s["kp1"], s["kp2"], b12)
        return {"best12": b12, "dist12": d12, "second12": s12, "best21": b21, "dist21": d21,
                "second21": s21, "mutual": both, "gms": kept}
    idx = epm.Index(s["specs"], s["kp2"], eps2=s["eps2"], eps=case["eps"],
                    workspace=s["workspace"])
    kept = dict(row_offsets=s["offsets"], col_indices=s["cols"], sync=case["sync"])
    if do == "match":
        offs, cols = idx.query(s["kp1"], **kept)
        code = dict(desc1_f32=s["d1"], desc2_f32=s["d2"]) if case["dtype"] == "bf16" else {}
        best, dist, second = idx.match(offs, cols, s.get("c1", s["d1"]), s.get("c2", s["d2"]),
                                       dtype=case["dtype"], ratio=case["ratio"], out=s["out"], **code)
    else:
        kept.update(out=s["out"], ratio=case["ratio"])
        if case["dtype"] == "bf16":
            got = idx.query_match_bf16(s["kp1"], s["c1"], s["c2"], s["d1"], s["d2"], **kept)
        elif case["dtype"] == "fp8":
            got = idx.query_match_fp8(s["kp1"], s["c2"], s["scale2"], s["err2"], s["d1"], s["d2"],
                                      **kept)
        else:
            got = idx.query_match(s["kp1"], s["d1"], s["d2"], **kept)
        offs, _, best, dist, second = got
    # the whole column buffer: its first offsets[-1] entries are the candidates
    return {"offsets": offs, "cols": s["cols"], "best": best, "dist": dist, "second": second}


# ------------------------------------------------------------------ the least work

def work(case):
    do = case["do"]
    net = 2 * (IN * HID + HID * HID + HID)
    if do == "train":
        b = case["batch"]
        return {"bytes": b * (4 + 4 * IN + 4) + 4 * NPARAM * 7, "flops": 3 * net * b}
    if do == "infer":
        n = case["pairs"] * case["kp"]
        return {"bytes": n * (8 + 12 + 4 * IN + 4) + 4 * NPARAM, "flops": net * n}
    if do == "encode":
        return {"bytes": case["rows"] * (512 + 128 + 4 + 256 + 8), "flops": case["rows"] * 128 * 8}
    n1 = sum(s[2] for s in _shapes(case))
    n2 = sum(s[3] for s in _shapes(case))
    k = _candidates(case)
    row = {"f32": (512, 512), "bf16": (768, 768), "fp8": (512, 512 + 128 + 8),
           "bin256": (32, 32)}[case["dtype"]]
    per = 8 + (24 if case["dtype"] == "bin256" else 3 * 128)
    eps = 4 if case["eps_per_keypoint"] else 0
    one = n1 * (8 + row[0]) + n2 * (8 + eps + row[1])
    if do == "mutual":  # the rows are read once, the CSRs are written all the same
        return {"bytes": one + 2 * (4 * k + 10 * (n1 + n2)) + 8 * n1, "flops": 2 * k * per}
    return {"bytes": one + 8 * (n1 + 1) + 4 * k + 12 * n1, "flops": k * per}


# ------------------------------------------------------------------ in 64 bits

def _two_smallest(F, kp1, kp2, eps, d1, d2):
    """Squared distances to the nearest and the second nearest candidate of
    every image-1 keypoint (inf where there is none)."""
    one = torch.ones((len(kp1), 1), dtype=torch.float64, device="cuda")
    lines = torch.cat([kp1.double(), one], 1) @ torch.tensor(np.asarray(F), device="cuda").T
    x, y = kp2.double().T
    binary = d1.dtype == torch.int32
    if binary:
        shifts = torch.arange(32, device="cuda", dtype=torch.int32)
        d1 = ((d1[:, :, None] >> shifts) & 1).reshape(len(d1), 256)
        d2 = ((d2[:, :, None] >> shifts) & 1).reshape(len(d2), 256)
    d1, d2 = d1.double(), d2.double()
    q1, q2 = (d1 * d1).sum(1), (d2 * d2).sum(1)
    near = [torch.full((len(kp1),), math.inf, dtype=torch.float64, device="cuda") for _ in range(2)]
    if not len(kp2):
        return near
    step = max(1, 100_000_000 // len(kp2))
    for b in range(0, len(kp1), step):
        a, bb, c = (lines[b:b + step, k:k + 1] for k in range(3))
        inside = (a * x + bb * y + c).abs() <= eps * torch.sqrt(a * a + bb * bb)
        inside &= (a != 0) | (bb != 0)
        d = torch.addmm(q2, d1[b:b + step], d2.T, alpha=-2.0) + q1[b:b + step, None]
        d.masked_fill_(~inside, math.inf)
        got = torch.topk(d, min(2, len(kp2)), dim=1, largest=False)[0]
        for k in range(got.shape[1]):
            near[k][b:b + step] = got[:, k].clamp_min(0.0)
    return near


def _exact_pairs(case, s, back=False):
    first, second = [], []
    q = k = 0
    for f, m, n in zip(s["F"], s["m"], s["n"]):
        a, b = slice(q, q + m), slice(k, k + n)
        own = s["eps1"] if back else s["eps2"]
        eps = float(np.float32(case["eps"])) if own is None else own[a if back else b].double()
        one = (s["kp1"][a], s["kp2"][b], s["d1"][a], s["d2"][b])
        if back:
            got = _two_smallest(np.asarray(f).T, one[1], one[0], eps, one[3], one[2])
        else:
            got = _two_smallest(f, one[0], one[1], eps, one[2], one[3])
        first.append(got[0])
        second.append(got[1])
        q, k = q + m, k + n
    return torch.cat(first), torch.cat(second)


def exact(case, seed):
    do = case["do"]
    if do == "train":
        s = _training(case, seed)
        p = torch.tensor(s["params"], device="cuda").double().requires_grad_()
        x, y = s["x"][s["order"].long()].double(), s["y"][s["order"].long()].double()
        u = y - torch.nn.functional.softplus(_network(p, x)[2])
        q = float(np.float32(0.99))
        loss = torch.where(u >= 0, q * u, (q - 1.0) * u).mean()
        loss.backward()
        b1, b2, lr, eps = (float(np.float32(k)) for k in (0.9, 0.999, 1e-3, 1e-8))
        g, t = p.grad, s["t"] + 1
        m = b1 * torch.tensor(s["m"], device="cuda").double() + (1 - b1) * g
        v = b2 * torch.tensor(s["v"], device="cuda").double() + (1 - b2) * g * g
        new = p.detach() - lr * (m / (1 - b1 ** t)) / (torch.sqrt(v / (1 - b2 ** t)) + eps)
        return {"loss": loss.detach().reshape(1), "grad": g, "params": new, "m": m, "v": v}
    if do == "infer":
        s = prepare(case, seed)
        feats, epss = [], []
        W, H = SIZES[3]
        params = s["params"].bfloat16().double()
        for p, f in enumerate(s["F"]):
            at = slice(p * case["kp"], (p + 1) * case["kp"])
            xy = s["kp2"][at].double()
            e = np.linalg.svd(np.asarray(f).T)[2][2]
            if abs(e[2]) * 1e12 < np.linalg.norm(e[:2]):
                rel = torch.full((case["kp"],), 1000.0, dtype=torch.float64, device="cuda")
            else:
                d = torch.hypot(xy[:, 0] - e[0] / e[2], xy[:, 1] - e[1] / e[2])
                rel = (d / math.hypot(W, H)).clamp_max(1000.0)
            x = torch.cat([s["attrs"][at].double(), ((xy[:, :1] - W / 2) / (W / 2)),
                           ((xy[:, 1:] - H / 2) / (W / 2)), torch.log1p(rel)[:, None]], 1)
            feats.append(x)
            epss.append(torch.nn.functional.softplus(_network(params, x)[2]).clamp(0.5, 8.0))
        return {"features": torch.cat(feats), "eps": torch.cat(epss)}
    if do == "encode":
        d = prepare(case, seed)["d"].double()
        scale = d.abs().amax(1) / 448.0
        half = (d - d.bfloat16().double()).norm(dim=1)
        # the FP8 error is the norm against the codes' own values, whose
        # rounding follows the FP32 quotient: no value without those codes
        return {"fp8": None, "scale": scale, "error": None, "bf16": None, "bf16_error": half}
    s = _scene(case, seed)
    dist, second = _exact_pairs(case, s)
    if do == "mutual":
        d21, s21 = _exact_pairs(case, s, back=True)
        return {"best12": None, "dist12": dist, "second12": second, "best21": None, "dist21": d21,
                "second21": s21, "mutual": None, "gms": None}
    return {"offsets": None, "cols": None, "best": None, "dist": dist, "second": second}
