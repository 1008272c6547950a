"""The work that a user of this package has it do, as timed cases.

``listed()`` gives the cases, ``draw(rng)`` one more of the same ranges,
``prepare(case, seed)`` what a program holds before the call, ``run(state)``
one pass through the public entry points, ``work(case)`` the bytes and
operations a pass cannot do without, and ``exact(case, seed)`` the same
outputs in 64 bits, in plain torch.

Kinds of case (``op``):

``forward``  object-frame rays rendered through the differentiable surface
``step``     the same with its backward pass: a torch loss's gradient
``render``   a view of one object into host images (evaluation, previews)
``query``    densities at points on the device
``mesh``     a triangle mesh of one object, copied to the host
``train``    a burst of training steps of one or many objects, then the
             weights read back into page-locked buffers the program keeps

Ray, sample and cell positions follow the documented FP32 expression order,
as they decide integers; everything after them is taken in 64 bits.
"""
import ctypes
import math

import numpy as np
import torch

import paper_2304_05735_amd as pk
from paper_2304_05735_amd.field import RomapFieldFn

M32 = 0xFFFFFFFF
_stream = None


def stream():
    """The stream that contexts and torch share (a context orders its work on it)."""
    global _stream
    if _stream is None:
        _stream = torch.cuda.Stream()
    return _stream


def case_of(name, op, **kw):
    c = dict(name=name, op=op, levels=16, base=16, top=1024, log2T=19, samples=64, bf16=False,
             layers=1)
    c.update(kw)
    return c


def listed():
    return [
        # the smallest call: a preview or unit of a user's own loop on the small model
        case_of("forward_small", "forward", levels=8, top=128, log2T=12, samples=32, rays=256),
        # a full ray batch of one object in evaluation
        case_of("forward_batch", "forward", rays=4096),
        # one iteration of a torch training loop around the surface: the default shape ...
        case_of("step_batch", "step", rays=4096),
        # ... and a ragged one with the BF16 MLP and long rays on the paper's table size
        case_of("step_bf16_ragged", "step", log2T=16, samples=128, rays=1999, bf16=True),
        # an evaluation view at the image size of the benchmark scenes
        case_of("render_view", "render", W=640, H=480, fill=0.35, bf16=True),
        # a small odd-sized preview of a mapped object with empty space skipped
        case_of("render_preview", "render", log2T=17, samples=128, W=173, H=131, fill=0.8,
                occupancy=0.3),
        # densities for a caller's own grid or collision test
        case_of("query_points", "query", points=100003, log2T=18),
        # the per-object mesh of the paper (64 cells a side)
        case_of("mesh_64", "mesh", res=64, log2T=18),
        # a newly detected small object: few rays, many short steps
        case_of("train_small", "train", objects=1, levels=8, top=128, log2T=12, log2T_lo=12,
                samples=32, rays=256, steps=48),
        # one object at full size with the FP32 MLP
        case_of("train_one", "train", objects=1, log2T_lo=19, rays=4096, steps=16),
        # a room of objects of mixed size in one batched step (the headline)
        case_of("train_room", "train", objects=24, log2T_lo=15, rays=1050, bf16=True, steps=16),
        # a frame of incremental mapping: a few steps with long rays and empty-space skipping
        case_of("train_frame", "train", objects=12, log2T=18, log2T_lo=18, samples=128, rays=2500,
                bf16=True, steps=4, occupancy=0.3),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["forward", "step", "render", "query", "mesh", "train", "train", "train"])
    c = case_of("", op, levels=rng.choice([8, 12, 16, 16]), top=rng.choice([128, 512, 1024, 2048]),
                log2T=rng.randint(12, 19), samples=rng.choice([32, 64, 64, 128]),
                bf16=rng.random() < 0.5, layers=rng.choice([1, 1, 1, 2, 3]))
    if op in ("forward", "step"):
        c["rays"] = _log_int(rng, 65, 4096)
    elif op == "render":
        c.update(W=_log_int(rng, 64, 640), H=_log_int(rng, 48, 480), fill=rng.uniform(0.1, 0.9),
                 occupancy=rng.choice([1.0, 0.3]))
    elif op == "query":
        c["points"] = _log_int(rng, 1000, 200000)
    elif op == "mesh":
        c["res"] = rng.randint(17, 80)
    else:
        n = rng.choice([1, 1, 2, 5, 11, 24])
        c.update(objects=n, log2T_lo=max(12, c["log2T"] - rng.randint(0, 4)),
                 rays=_log_int(rng, 200, 4096 if n == 1 else 1000), steps=rng.choice([1, 4, 10, 16]),
                 occupancy=rng.choice([1.0, 1.0, 0.3]))
    del c["name"]
    return c


# ---------------------------------------------------------------------------
# inputs, from the seed alone

def _levels(case, log2T):
    """(N_l, T_l, hashed, first entry) of each level, and the entries in all."""
    L, lo, hi = case["levels"], case["base"], case["top"]
    b = math.exp((math.log(hi) - math.log(lo)) / (L - 1))
    out, off = [], 0
    for l in range(L):
        N = int(math.floor(lo * b ** l + 1e-6))
        dense = (N + 1) ** 3
        hashed = dense > (1 << log2T)
        T = (1 << log2T) if hashed else dense
        out.append((N, T, hashed, off))
        off += T
    return out, off


def _mats(case):
    return [(64, 2 * case["levels"])] + [(64, 64)] * (case["layers"] - 1) + [(16, 64), (64, 15), (3, 64)]


def _n_mlp(case):
    return sum(a * b for a, b in _mats(case))


def _gen(seed, *key):
    g = torch.Generator(device="cuda")
    g.manual_seed(hash((int(seed),) + key) & 0x7FFFFFFFFFFF)
    return g


def _uniform(g, lo, hi, *shape):
    return torch.rand(*shape, generator=g, device="cuda") * (hi - lo) + lo


def _params(case, seed, k, log2T):
    """Parameters of trained size: grid U(-0.5, 0.5), MLP Glorot-uniform."""
    g = _gen(seed, 1, k)
    parts = [_uniform(g, -0.5, 0.5, 2 * _levels(case, log2T)[1])]
    for o, i in _mats(case):
        lim = math.sqrt(6.0 / (o + i))
        parts.append(_uniform(g, -lim, lim, o * i))
    p = torch.cat(parts)
    if case["op"] in ("render", "query", "mesh"):
        _solid(case, p, log2T)
    return p


def _solid(case, p, log2T):
    """Makes a trained-looking body of the parameters: the first feature of the
    coarsest level falls off with the radius and leads the density (sigma = 10
    at about half the box), everything else is texture on it."""
    N, T, hashed, _ = _levels(case, log2T)[0][0]
    v = torch.arange((N + 1) ** 3, device="cuda")
    c = torch.stack([v % (N + 1), v // (N + 1) % (N + 1), v // (N + 1) ** 2], 1)
    h = (c[:, 0] ^ ((c[:, 1] * 2654435761) & M32) ^ ((c[:, 2] * 805459861) & M32)) & (T - 1)
    grid, W = _split(case, p)
    grid[h if hashed else v, 0] = 0.7 - (2.0 * c / N - 1.0).norm(dim=1)
    first, last = W[0], W[-3]
    first[:2] = 0.0
    first[0, 0], first[1, 0] = 1.0, -1.0
    for w in W[1:-3]:  # deeper density MLP: pass the two units on
        w[:2] = 0.0
        w[0, 0] = w[1, 1] = 1.0
    last[0] *= 0.1
    last[0, 0], last[0, 1] = 12.0, -12.0


def _moments(case, seed, k, n):
    """Adam moments of a model in training: sqrt(v) over a decade above what one
    sample adds to a table entry (a fixed decade for the MLP), m below it."""
    g = _gen(seed, 2, k)
    rv = torch.exp(_uniform(g, 0.0, math.log(10.0), n))
    rv[:n - _n_mlp(case)] *= 4.0 / (case["rays"] * case["samples"])
    rv[n - _n_mlp(case):] *= 1e-3
    return rv * _uniform(g, -0.3, 0.3, n), rv * rv


def _occupancy(case, seed, k):
    """64^3 bits of an object: a shell-like band of cells, or None (no skipping)."""
    share = case.get("occupancy", 1.0)
    if share >= 1.0:
        return None
    r = np.random.default_rng([int(seed), 3, k])
    x = (np.arange(64) + 0.5) / 32 - 1
    rad = np.sqrt(x[None, None, :] ** 2 + x[None, :, None] ** 2 + x[:, None, None] ** 2)
    mid = r.uniform(0.6, 0.8)
    on = np.abs(rad - mid) < share * 0.7
    return np.packbits(on.reshape(-1), bitorder="little")


def _half(seed, k):
    return np.random.default_rng([int(seed), 4, k]).uniform(0.25, 0.6, 3).astype(np.float32)


def _config(case, seed, **kw):
    return pk.default_config(n_levels=case["levels"], base_res=case["base"], max_res=case["top"],
                             log2_table_size=case["log2T"], samples_per_ray=case["samples"],
                             precision=pk.PREC_BF16 if case["bf16"] else pk.PREC_FP32,
                             mlp_layers=case["layers"], seed=int(seed) & 0x7FFFFFFF, **kw)


def _look_at(eye, target):
    f = np.asarray(target, float) - np.asarray(eye, float)
    f /= np.linalg.norm(f)
    x = np.cross(f, [0.0, 0.0, 1.0])
    x /= np.linalg.norm(x)
    T = np.zeros((3, 4))
    T[:, 0], T[:, 1], T[:, 2], T[:, 3] = x, np.cross(f, x), f, eye
    return T.astype(np.float32)


def _camera(T, W, H, f):
    return dict(T_wc=T, W=W, H=H, fx=float(f), fy=float(f), cx=W / 2.0, cy=H / 2.0)


def _view(case, seed):
    """A camera that sees the object's box over about `fill` of the image's width."""
    r = np.random.default_rng([int(seed), 5])
    a = r.uniform(0, 2 * math.pi)
    eye = 2.5 * np.array([math.cos(a), math.sin(a), r.uniform(0.2, 0.6)])
    W, H = case["W"], case["H"]
    extent = 2 * float(np.linalg.norm(_half(seed, 0)))
    return _camera(_look_at(eye, r.uniform(-0.05, 0.05, 3)), W, H,
                   case["fill"] * W * np.linalg.norm(eye) / extent)


def _object_rays(case, seed):
    """Rays (origin, unit direction, t_near, t_far) from around the box into it;
    some pass beside it (an empty segment)."""
    g = _gen(seed, 6)
    n = case["rays"]
    half = torch.from_numpy(_half(seed, 0)).cuda()
    o = torch.randn(n, 3, generator=g, device="cuda")
    o = o / o.norm(dim=1, keepdim=True) * 1.6
    d = _uniform(g, -1.1, 1.1, n, 3) * half - o
    d = d / d.norm(dim=1, keepdim=True)
    t0, t1 = (-half - o) / d, (half - o) / d
    tn = torch.minimum(t0, t1).amax(1).clamp_min(0)
    tf = torch.maximum(t0, t1).amin(1)
    return torch.cat([o, d, tn[:, None], tf[:, None]], 1).contiguous()


def _points(case, seed):
    half = torch.from_numpy(_half(seed, 0)).cuda()
    return (_uniform(_gen(seed, 7), -1.02, 1.02, case["points"], 3) * half).contiguous()


def _room(case, seed):
    """Boxes, ray counts and tables of a training case, and its keyframes:
    a ring of 12 cameras, masks of each object's inscribed ball, images of
    smooth colour, depth on every 200th pixel."""
    r = np.random.default_rng([int(seed), 8])
    n = case["objects"]
    spec = []
    side = max(1, math.ceil(math.sqrt(n)))
    for k in range(n):
        half = _half(seed, k)
        t = np.array([(k % side - (side - 1) / 2) * 1.5, (k // side - (side - 1) / 2) * 1.5,
                      float(half[2])]) + r.uniform(-0.1, 0.1, 3)
        span = case["log2T"] - case["log2T_lo"]
        log2T = case["log2T"] - (k * span // max(1, n - 1) if n > 1 else 0)
        rays = case["rays"] if n == 1 else max(64, int(case["rays"] * r.uniform(0.4, 1.6)))
        spec.append(dict(t=t.astype(np.float32), yaw=float(np.float32(r.uniform(0, 6.28))), half=half,
                         log2T=log2T, rays=rays))
    small = case["rays"] < 1000 and n == 1
    W, H = (64, 64) if small else (640, 480)
    dist = 1.5 + 1.1 * side
    u, v = np.meshgrid(np.arange(W), np.arange(H))
    frames = []
    for j in range(12):
        a = 2 * math.pi * j / 12 + 0.1
        cam = _camera(_look_at((dist * math.cos(a), dist * math.sin(a), 1.5), (0, 0, 0.3)), W, H, W * 0.8)
        T = cam["T_wc"].astype(float)
        mask = np.zeros((H, W), np.int32)
        depth = np.zeros((H, W), np.float32)
        cen = [(T[:, :3].T @ (s["t"].astype(float) - T[:, 3]), k, s) for k, s in enumerate(spec)]
        for p, k, s in sorted(cen, key=lambda q: -q[0][2]):
            rad = float(s["half"].min())
            px, py = p[0] / p[2] * cam["fx"] + cam["cx"], p[1] / p[2] * cam["fy"] + cam["cy"]
            on = (u + 0.5 - px) ** 2 + (v + 0.5 - py) ** 2 < (rad / p[2] * cam["fx"]) ** 2
            mask[on] = k + 1
            depth[on] = p[2] - rad
        depth.reshape(-1)[np.arange(W * H) % 200 != 0] = 0
        ph = r.uniform(0, 6.28, 3)
        rgb = np.stack([127.5 + 127 * np.sin(0.05 * u + 0.03 * v + ph[c]) for c in range(3)], -1)
        frames.append((cam, rgb.astype(np.uint8), mask, depth))
    return spec, frames


def prepare(case, seed):
    op = case["op"]
    st = dict(case=case)
    with torch.cuda.stream(stream()):
        if op == "train":
            spec, frames = _room(case, seed)
            # a frame's ray counts change with every frame: nothing is tuned for them
            ctx = pk.Context(_config(case, seed, autotune=1 if case["steps"] > 4 else 0, alpha_deg=0.0),
                             stream=stream())
            ids, bufs = [], []
            for k, s in enumerate(spec):
                i = ctx.add_object(k + 1, s["t"], s["yaw"], s["half"], s["log2T"])
                p = _params(case, seed, k, s["log2T"])
                m, v = _moments(case, seed, k, p.numel())
                for kind, x in ((pk.PARAMS, p), (pk.ADAM_M, m), (pk.ADAM_V, v)):
                    ctx.set_params(i, x.cpu().numpy(), kind)
                occ = _occupancy(case, seed, k)
                if occ is not None:
                    ctx.set_occupancy(i, occ)
                ids.append(i)
                bufs.append(torch.empty(p.numel(), pin_memory=True))
            for f in frames:
                ctx.add_keyframe(*f)
            seen = [k for k, i in enumerate(ids) if ctx.object_info(i).n_keyframes > 0]
            st.update(ctx=ctx, ids=[ids[k] for k in seen], rays=[spec[k]["rays"] for k in seen],
                      bufs=[bufs[k] for k in seen])
        else:
            ctx = pk.Context(_config(case, seed), stream=stream())
            oid = ctx.add_object(1, np.zeros(3), 0.3, _half(seed, 0))
            p = _params(case, seed, 0, case["log2T"])
            occ = _occupancy(case, seed, 0)
            st.update(ctx=ctx, oid=oid)
            if occ is not None:
                ctx.set_occupancy(oid, occ)
            if op in ("forward", "step"):
                st["params"] = p
                st["rays"] = _object_rays(case, seed)
                if op == "step":
                    st["params"].requires_grad_(True)
                    st["target"] = torch.rand(case["rays"], 3, generator=_gen(seed, 9), device="cuda")
            else:
                ctx.set_params(oid, p.cpu().numpy())
            if op == "render":
                st["cam"] = _view(case, seed)
            elif op == "query":
                st["xyz"] = _points(case, seed)
            elif op == "mesh":
                # a vertex buffer that a viewer keeps: room for 16 triangles per surface cell
                st["tris"] = np.zeros((16 * case["res"] ** 2, 3, 3), np.float32)
                st["count"] = ctypes.c_int64()
    torch.cuda.synchronize()
    return st


def _torch_loss(rgb, depth, tend, target):
    n = rgb.shape[0]
    return ((rgb - target) ** 2).sum() / n + 0.1 * depth.sum() / n + 0.05 * tend.sum() / n


def run(st):
    case, ctx = st["case"], st["ctx"]
    op = case["op"]
    with torch.cuda.stream(stream()):
        if op == "forward":
            return ctx.field_forward(st["oid"], st["rays"], st["params"])
        if op == "step":
            p = st["params"]
            p.grad = None
            rgb, depth, tend = RomapFieldFn.apply(p, st["rays"], ctx, st["oid"])
            loss = _torch_loss(rgb, depth, tend, st["target"])
            loss.backward()
            return dict(loss=loss.detach(), rgb=rgb.detach(), grad=p.grad)
        if op == "render":
            return ctx.render(st["oid"], st["cam"])
        if op == "query":
            return ctx.query_density(st["oid"], st["xyz"])
        if op == "mesh":
            t, n = st["tris"], st["count"]
            rc = pk.lib().romap_extract_mesh(ctx.h, st["oid"], case["res"], 10.0, 1,
                                             ctypes.c_void_p(t.ctypes.data), len(t),
                                             ctypes.byref(n), 0)
            assert rc == pk.ROMAP_OK and n.value <= len(t)
            return t
        stats = ctx.train(case["steps"], st["ids"], st["rays"])
        for i, b in zip(st["ids"], st["bufs"]):
            rc = pk.lib().romap_get_params(ctx.h, i, pk.PARAMS, ctypes.c_void_p(b.data_ptr()),
                                           b.numel(), None)
            assert rc == pk.ROMAP_OK
        return dict(loss=stats.loss_mean, weights=st["bufs"])


# ---------------------------------------------------------------------------
# what a pass cannot do without

def _mlp_flops(case):
    return 2.0 * _n_mlp(case)


def _table_bytes(case, log2T, samples):
    """Each entry at most once, and no more than the samples' eight corners."""
    return sum(8.0 * min(T, 8 * samples) for _, T, _, _ in _levels(case, log2T)[0])


def _encode_flops(case):
    return 32.0 * case["levels"]


def work(case):
    op, N = case["op"], case["samples"]
    per = _mlp_flops(case) + _encode_flops(case)
    if op in ("forward", "step"):
        S = case["rays"] * N
        tab = _table_bytes(case, case["log2T"], S) + 4.0 * _n_mlp(case)
        b = tab + case["rays"] * (32 + 20)
        if op == "forward":
            return dict(bytes=b, flops=S * per)
        P = 2 * _levels(case, case["log2T"])[1] + _n_mlp(case)
        return dict(bytes=b + case["rays"] * 12 + 4.0 * P, flops=3 * S * per)
    if op == "render":
        pix = case["W"] * case["H"]
        S = pix * N * min(1.0, 0.5 * case["fill"] ** 2 * case["W"] / case["H"]) * case.get("occupancy", 1.0)
        return dict(bytes=_table_bytes(case, case["log2T"], S) + 20.0 * pix, flops=S * per)
    if op in ("query", "mesh"):
        n = case["points"] if op == "query" else (case["res"] + 1) ** 3
        per = 2.0 * (_n_mlp(case) - 15 * 64 - 3 * 64 - 15 * 64) + _encode_flops(case)
        out = 16.0 * n if op == "query" else 36.0 * 6 * case["res"] ** 2
        return dict(bytes=_table_bytes(case, case["log2T"], n) + out, flops=n * per)
    n, b, fl = case["objects"], 0.0, 0.0
    for k in range(n):
        span = case["log2T"] - case["log2T_lo"]
        log2T = case["log2T"] - (k * span // max(1, n - 1) if n > 1 else 0)
        P = 2 * _levels(case, log2T)[1] + _n_mlp(case)
        S = case["rays"] * N * case.get("occupancy", 1.0)
        b += case["steps"] * (24.0 * P + 64.0 * case["rays"]) + 4.0 * P
        fl += case["steps"] * (3 * S * per + 14.0 * P)
    return dict(bytes=b, flops=fl)


# ---------------------------------------------------------------------------
# 64 bits, in plain torch

def _corners(p, N, T, hashed):
    """Entry indices and 64-bit weights of the 8 corners of positions p (FP32)."""
    g = p * float(N)
    c = g.floor().clamp(0, N - 1)
    f = (g - c).double()
    c = c.long()
    idx, w = [], []
    for b in range(8):
        bit = [b & 1, (b >> 1) & 1, b >> 2]
        vx, vy, vz = (c[:, a] + bit[a] for a in range(3))
        if hashed:
            i = (vx ^ ((vy * 2654435761) & M32) ^ ((vz * 805459861) & M32)) & (T - 1)
        else:
            i = vx + vy * (N + 1) + vz * (N + 1) ** 2
        ww = 1.0
        for a in range(3):
            ww = ww * (f[:, a] if bit[a] else 1.0 - f[:, a])
        idx.append(i)
        w.append(ww)
    return torch.stack(idx, 1), torch.stack(w, 1)


def _encode(grid, p, levels):
    e = []
    for N, T, hashed, off in levels:
        idx, w = _corners(p, N, T, hashed)
        e.append((grid[off + idx] * w[:, :, None]).sum(1))
    return torch.cat(e, 1)


def _scatter(grad, p, levels, de):
    for l, (N, T, hashed, off) in enumerate(levels):
        idx, w = _corners(p, N, T, hashed)
        for b in range(8):
            grad.index_add_(0, off + idx[:, b], w[:, b:b + 1] * de[:, 2 * l:2 * l + 2])


def _split(case, params):
    n, out = params.numel() - _n_mlp(case), []
    at = n
    for o, i in _mats(case):
        out.append(params[at:at + o * i].view(o, i))
        at += o * i
    return params[:n].view(-1, 2), out


def _mlp(W, e):
    h = torch.relu(e @ W[0].T)
    for k in range(1, len(W) - 3):
        h = torch.relu(h @ W[k].T)
    y = h @ W[-3].T
    z = torch.relu(y[:, 1:] @ W[-2].T) @ W[-1].T
    return y[:, 0], torch.sigmoid(z)


def _sample_positions(o, d, tn, delta, half, N):
    """FP32, in the documented order: distances (R, N) and unit positions (R N, 3)."""
    i = torch.arange(N, device=o.device, dtype=torch.float32) + 0.5
    dist = tn[:, None] + i[None, :] * delta[:, None]
    x = o[:, None, :] + dist[:, :, None] * d[:, None, :]
    q = (x + half) / (half + half)
    return dist, q.clamp(0, 1).view(-1, 3)


def _live(occ, p):
    if occ is None:
        return None
    bits = torch.from_numpy(np.unpackbits(occ, bitorder="little")).to(p.device).bool()
    c = (p * 64.0).floor().long().clamp(0, 63)
    return bits[c[:, 0] + 64 * c[:, 1] + 4096 * c[:, 2]]


def _composite(y0, c, delta, dist, live):
    """Colour, depth, T_end and densities of rays whose samples are given."""
    R, N = dist.shape
    sig = torch.exp(torch.clamp(y0, max=15.0)).view(R, N)
    if live is not None:
        sig = torch.where(live.view(R, N), sig, torch.zeros_like(sig))
    tau = sig * delta.double()[:, None]
    before = torch.cumsum(tau, 1) - tau
    w = torch.exp(-before) * -torch.expm1(-tau)
    C = (w[:, :, None] * c.view(R, N, 3)).sum(1)
    return C, (w * dist.double()).sum(1), torch.exp(-tau.sum(1)), sig


def _field(case, params, o, d, tn, delta, half, occ, head, grad=None):
    """head(colour, depth, T_end, sigma) of hit rays; with `grad` (a 64-bit
    parameter vector) its backward pass is added there."""
    grid, W = _split(case, params)
    levels = _levels_of(case, grid.shape[0])
    dist, p = _sample_positions(o, d, tn, delta, half, case["samples"])
    live = _live(occ, p)
    with torch.no_grad():
        e = _encode(grid, p, levels)
    if grad is None:
        with torch.no_grad():
            y0, c = _mlp(W, e)
            return head(*_composite(y0, c, delta, dist, live))
    e.requires_grad_(True)
    W = [w.detach().clone().requires_grad_(True) for w in W]
    y0, c = _mlp(W, e)
    out = head(*_composite(y0, c, delta, dist, live))
    out.backward()
    ggrid, gW = _split(case, grad)
    _scatter(ggrid, p, levels, e.grad)
    for a, w in zip(gW, W):
        a += w.grad
    return out.detach()


def _levels_of(case, entries):
    for log2T in range(8, 25):
        lv, n = _levels(case, log2T)
        if n == entries:
            return lv
    raise ValueError("no table of %d entries" % entries)


def _user_rays(case, seed):
    R = _object_rays(case, seed)
    hit = R[:, 7] > R[:, 6]
    return R, hit, torch.where(hit, (R[:, 7] - R[:, 6]) / float(case["samples"]), torch.zeros_like(R[:, 0]))


def _render64(case, params, hit, o, d, tn, delta, half, occ):
    n = o.shape[0]
    rgb = torch.zeros(n, 3, dtype=torch.float64, device="cuda")
    depth = torch.zeros(n, dtype=torch.float64, device="cuda")
    tend = torch.ones(n, dtype=torch.float64, device="cuda")
    at = hit.nonzero()[:, 0]
    for k in at.split(8192):
        rgb[k], depth[k], tend[k] = _field(case, params, o[k], d[k], tn[k], delta[k], half, occ,
                                           lambda C, D, T, s: (C, D, T))
    return rgb, depth, tend


def _object_frame(T, t, yaw):
    c, s = math.cos(yaw), math.sin(yaw)
    R = np.array([[c, s, 0.0], [-s, c, 0.0], [0.0, 0.0, 1.0]])
    T = np.asarray(T, float).reshape(3, 4)
    return (R @ T[:, :3]).astype(np.float32), (R @ (T[:, 3] - np.asarray(t, float))).astype(np.float32)


def _pixel_rays(M, c, cam, u, v, half, N):
    """FP32 back-projection and slab clipping: o, d, t_near, delta, hit.  M (n, 3, 3), c (n, 3)."""
    f = [torch.tensor(cam[k], dtype=torch.float32, device="cuda") for k in ("cx", "cy", "fx", "fy")]
    x = ((u.float() + 0.5) - f[0]) / f[2]
    y = ((v.float() + 0.5) - f[1]) / f[3]
    dd = torch.stack([(M[:, k, 0] * x + M[:, k, 1] * y) + M[:, k, 2] for k in range(3)], 1)
    n = torch.sqrt((dd[:, 0] * dd[:, 0] + dd[:, 1] * dd[:, 1]) + dd[:, 2] * dd[:, 2])
    d = dd / n[:, None]
    inv = 1.0 / d
    t0, t1 = (-half - c) * inv, (half - c) * inv
    lo, hi = torch.fmin(t0, t1), torch.fmax(t0, t1)
    tmin = torch.fmax(torch.fmax(lo[:, 0], lo[:, 1]), lo[:, 2])
    tmax = torch.fmin(torch.fmin(hi[:, 0], hi[:, 1]), hi[:, 2])
    tn = torch.clamp(tmin, min=0.0)
    hit = tmax > tn
    return c, d, tn, torch.where(hit, (tmax - tn) / float(N), torch.zeros_like(tn)), hit


def _philox(c0, c1, key):
    """Philox4x32-10 of counters (c0, c1, 0, 0): four int64 tensors of 32-bit values."""
    c = [torch.full_like(c1, c0 & M32), c1, torch.zeros_like(c1), torch.zeros_like(c1)]
    k0, k1 = key
    for _ in range(10):
        a, b = c[0] * 0xD2511F53, c[2] * 0xCD9E8D57
        c = [((b >> 32) & M32) ^ c[1] ^ k0, b & M32, ((a >> 32) & M32) ^ c[3] ^ k1, a & M32]
        k0, k1 = (k0 + 0x9E3779B9) & M32, (k1 + 0xBB67AE85) & M32
    return c


def _train64(case, seed):
    spec, frames = _room(case, seed)
    N, cfg = case["samples"], _config(case, seed)
    key = int(cfg.seed)
    b1, b2, lr, eps = (np.float32(x) for x in (cfg.beta1, cfg.beta2, cfg.lr, cfg.eps))
    rgb = torch.from_numpy(np.stack([f[1] for f in frames])).cuda()
    mask = torch.from_numpy(np.stack([f[2] for f in frames])).cuda()
    depth = torch.from_numpy(np.stack([f[3] for f in frames])).cuda()
    H, W = mask.shape[1:]
    losses, weights = [], []
    for k, s in enumerate(spec):
        refs, base = [], 0
        for j, (cam, _, m, _) in enumerate(frames):
            vv, uu = np.nonzero(m == k + 1)
            if vv.size == 0:
                continue
            mx, my = (int(np.ptp(q) + 1) * 10 + 99 for q in (uu, vv))
            x0, y0 = max(0, uu.min() - mx // 100), max(0, vv.min() - my // 100)
            x1, y1 = min(W - 1, uu.max() + mx // 100), min(H - 1, vv.max() + my // 100)
            refs.append((j, x0, y0, x1 - x0 + 1, y1 - y0 + 1, base) + _object_frame(cam["T_wc"], s["t"], s["yaw"]))
            base += (x1 - x0 + 1) * (y1 - y0 + 1)
        if not refs:
            continue
        tab = torch.tensor([[int(q) for q in r[:6]] for r in refs], device="cuda")
        Ms = torch.from_numpy(np.stack([r[6] for r in refs])).cuda()
        cs = torch.from_numpy(np.stack([r[7] for r in refs])).cuda()
        half = torch.from_numpy(s["half"]).cuda()
        occ = _occupancy(case, seed, k)
        p32 = _params(case, seed, k, s["log2T"])
        p, (m, v) = p32.double(), (x.double() for x in _moments(case, seed, k, p32.numel()))
        B = s["rays"]
        for step in range(case["steps"]):
            x = _philox(step, torch.arange(B, device="cuda"), ((key & M32) ^ k, key >> 32))
            q = (x[0] * base) >> 32
            ref = torch.searchsorted(tab[:, 5].contiguous(), q, right=True) - 1
            r = tab[ref]
            lq = q - r[:, 5]
            u, w = r[:, 1] + lq % r[:, 3], r[:, 2] + lq // r[:, 3]
            cam = frames[0][0]
            o, d, tn, delta, hit = _pixel_rays(Ms[ref], cs[ref], cam, u, w, half, N)
            mk = mask[r[:, 0], w, u]
            bg, ob = mk == 0, mk == k + 1
            crand = torch.stack([(x[c] >> 8).double() / 16777216.0 for c in (1, 2, 3)], 1)
            img = (rgb[r[:, 0], w, u].float() / 255.0).double()
            tgt = torch.where(bg[:, None], crand, img)
            z = depth[r[:, 0], w, u]
            xn = ((u.float() + 0.5) - cam["cx"]) / np.float32(cam["fx"])
            yn = ((w.float() + 0.5) - cam["cy"]) / np.float32(cam["fy"])
            D = (z * torch.sqrt((xn * xn + yn * yn) + 1.0)).double()
            has = ob & (z > 0)
            on = (hit & (bg | ob)).nonzero()[:, 0]

            def head(C, Dh, T, sig):
                t, isbg = tgt[on], bg[on].double()
                Co = C + (T * isbg)[:, None] * t
                l = ((Co - t) ** 2).sum(1)
                l = l + float(cfg.lambda_depth) * has[on].double() * (Dh - D[on]).abs()
                l = l + float(cfg.lambda_density) * isbg * sig.sum(1)
                return l.sum() / B

            g = torch.zeros_like(p)
            losses.append(float(_field(case, p, o[on], d[on], tn[on], delta[on], half, occ, head, g))
                          if on.numel() else 0.0)
            m = float(b1) * m + float(np.float32(1) - b1) * g
            v = float(b2) * v + float(np.float32(1) - b2) * g * g
            bc1 = float(np.float32(1.0 - float(b1) ** (step + 1)))
            bc2 = float(np.float32(1.0 - float(b2) ** (step + 1)))
            p = p - float(lr) * (m / bc1) / (torch.sqrt(v / bc2) + float(eps))
        weights.append(p)
    return dict(loss=torch.tensor(np.mean(losses), dtype=torch.float64), weights=weights)


def exact(case, seed):
    op = case["op"]
    if op == "mesh":
        return None  # whether a corner is inside is a decision, not a number
    if op == "train":
        n = case["objects"] * case["rays"] * case["samples"] * case["steps"] * case["levels"]
        return _train64(case, seed) if n < 1.2e9 else None
    half = torch.from_numpy(_half(seed, 0)).cuda()
    params = _params(case, seed, 0, case["log2T"]).double()
    occ = _occupancy(case, seed, 0)
    if op == "query":
        grid, W = _split(case, params)
        p = ((_points(case, seed) + half) / (half + half)).clamp(0, 1)
        return torch.exp(torch.clamp(_mlp(W, _encode(grid, p, _levels_of(case, grid.shape[0])))[0], max=15.0))
    if op == "render":
        cam = _view(case, seed)
        W, H = cam["W"], cam["H"]
        M, c = _object_frame(cam["T_wc"], np.zeros(3), float(np.float32(0.3)))
        px = torch.arange(W * H, device="cuda")
        o, d, tn, delta, hit = _pixel_rays(torch.from_numpy(M).cuda().expand(W * H, 3, 3),
                                           torch.from_numpy(c).cuda().expand(W * H, 3), cam, px % W, px // W,
                                           half, case["samples"])
        rgb, depth, tend = _render64(case, params, hit, o, d, tn, delta, half, occ)
        return [x.cpu().numpy() for x in (rgb.view(H, W, 3), depth.view(H, W), 1.0 - tend.view(H, W))]
    R, hit, delta = _user_rays(case, seed)
    if op == "forward":
        return _render64(case, params, hit, R[:, :3], R[:, 3:6], R[:, 6], delta, half, occ)
    target = torch.rand(case["rays"], 3, generator=_gen(seed, 9), device="cuda").double()
    n = case["rays"]
    grad = torch.zeros_like(params)
    loss = torch.zeros((), dtype=torch.float64, device="cuda")
    rgb = torch.zeros(n, 3, dtype=torch.float64, device="cuda")
    for on in hit.nonzero()[:, 0].split(4096):
        def head(C, D, T, sig):
            rgb[on] = C.detach()
            return (((C - target[on]) ** 2).sum() + 0.1 * D.sum() + 0.05 * T.sum()) / n
        loss += _field(case, params, R[on, :3], R[on, 3:6], R[on, 6], delta[on], half, occ, head, grad)
    miss = (~hit).nonzero()[:, 0]
    loss += ((target[miss] ** 2).sum() + 0.05 * miss.numel()) / n
    return dict(loss=loss, rgb=rgb, grad=grad)
