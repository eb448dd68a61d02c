"""The work that a user of this library has it do, as timed cases.

Each kind of case is one public entry point, called the way a player, an
encoder or a training program calls it:

* ``play``     frames of a GOP one by one (Decoder.decode_viewport): a player
               that gets each frame when it is due;
* ``gop``      a whole GOP in one call (Decoder.decode_gop);
* ``set``      the frames of an inter-frame set (Decoder.decode_set);
* ``encode``   source planes to stored coefficients (Decoder.encode_intra);
* ``rebuild``  dense planes from the sparse storage format (fmt.rebuild);
* ``train``    forward, loss and backward pass of the restoration network;
* ``restore``  restoration of a decoded viewport with its guard.

A GOP starts with an intra frame, so a pass gives the same result every time
it is repeated on the same state.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2208_10859_amd import cnn, fmt, wv

GOP_LEN = 8
INTRA_STEP = {"5/3": 4, "9/7": 8}
SET_STEPS = (4, 2, 1, 1)


# ------------------------------------------------------------------- cases
def listed():
    return [
        # The smallest call: one grey 512 x 512 tile, three levels, one intra
        # frame.  Launch and latency are all there is.
        _decode("play_grey_tile", "play", 512, 512, 512, 3, "5/3", 1, grey=True),
        # Playback of an 8192 x 8192 top-bottom stereo stream, frame by frame,
        # one eye's 110 x 110 degree viewport: an intra frame, then residuals.
        _decode("play_53_8192", "play", 8192, 8192, 512, 5, "5/3", 4, fov=110.0, yaw=23.0, pitch=-7.0),
        # The same stream a GOP at a time, tuned first: the throughput form.
        _decode("gop_53_8192", "gop", 8192, 8192, 512, 5, "5/3", GOP_LEN, fov=110.0, yaw=-131.0, pitch=12.0,
                tuned=True),
        # Float wavelet, four levels, foveated at the gaze.
        _decode("gop_97_8192_foveated", "gop", 8192, 8192, 512, 4, "9/7", GOP_LEN, fov=110.0, yaw=64.0,
                pitch=5.0, foveate=True, tuned=True),
        # Keyframe-free random access: an inter-frame set of four.
        _decode("set_53_8192", "set", 8192, 8192, 512, 5, "5/3", 4, fov=110.0, yaw=23.0, pitch=-7.0),
        # Streams cut into smaller tiles (finer viewports): 256 and 64.
        _decode("play_53_tile256", "play", 3840, 3840, 256, 5, "5/3", 3, fov=110.0, yaw=-50.0, pitch=20.0),
        _decode("gop_53_tile64", "gop", 1920, 1920, 64, 4, "5/3", GOP_LEN, fov=110.0, yaw=101.0, pitch=-15.0),
        # Ingest: a full frame encoded, integer and float.
        _encode("encode_53_8192", 8192, 8192, 512, 5, "5/3"),
        _encode("encode_97_4096", 4096, 4096, 512, 5, "9/7"),
        # A viewport of a stream kept in the sparse storage format.
        _rebuild("rebuild_97_4096", 4096, 4096, 512, 5, "9/7", 0.1, fov=110.0, yaw=11.0, pitch=3.0),
        # The restoration network: a training batch, and a decoded viewport of
        # 4 x 4 tiles.
        _train("train_16x128x128", 16, 128, 128),
        _restore("restore_2048", 512, 4, 4),
    ]


def _decode(name, kind, width, height, tile, levels, wavelet, frames, fov=0.0, yaw=0.0, pitch=0.0,
            grey=False, foveate=False, tuned=False):
    return {"name": name, "kind": kind, "width": width, "height": height, "tile": tile, "levels": levels,
            "wavelet": wavelet, "frames": frames, "fov": fov, "yaw": yaw, "pitch": pitch, "grey": grey,
            "foveate": foveate, "tuned": tuned}


def _encode(name, width, height, tile, levels, wavelet, grey=False):
    return {"name": name, "kind": "encode", "width": width, "height": height, "tile": tile,
            "levels": levels, "wavelet": wavelet, "grey": grey}


def _rebuild(name, width, height, tile, levels, wavelet, alpha, fov=0.0, yaw=0.0, pitch=0.0, grey=False,
             foveate=False):
    return {"name": name, "kind": "rebuild", "width": width, "height": height, "tile": tile,
            "levels": levels, "wavelet": wavelet, "alpha": alpha, "fov": fov, "yaw": yaw, "pitch": pitch,
            "grey": grey, "foveate": foveate}


def _train(name, n, h, w):
    return {"name": name, "kind": "train", "n": n, "h": h, "w": w}


def _restore(name, tile, tiles_x, tiles_y):
    return {"name": name, "kind": "restore", "tile": tile, "tiles_x": tiles_x, "tiles_y": tiles_y}


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("play", "gop", "set", "encode", "rebuild", "train", "restore"))
    if kind == "train":
        while True:
            n, h, w = _log_int(rng, 1, 16), _log_int(rng, 17, 512), _log_int(rng, 17, 512)
            if n * h * w <= 16 * 128 * 128:
                break
        case = _train("", n, h, w)
    elif kind == "restore":
        while True:
            tile = rng.choice((64, 128, 256, 512))
            tx, ty = _log_int(rng, 1, 16), _log_int(rng, 1, 16)
            if tile * tile * tx * ty <= 2048 * 2048:
                break
        case = _restore("", tile, tx, ty)
    else:
        wavelet = rng.choice(("5/3", "9/7"))
        grey = rng.random() < 0.2
        # the largest frame of each kind of call
        cap = 4096 if kind == "rebuild" or (kind == "encode" and wavelet == "9/7") else 8192
        tile = 512 if kind == "set" else rng.choice((16, 32, 64, 128, 256, 512))
        most = min(cap // tile, 64)
        width, height = tile * _log_int(rng, 1, most), tile * _log_int(rng, 1, most)
        deepest = int(math.log2(tile)) - (0 if grey else 1)
        levels = rng.randint(3, 5) if tile == 512 else rng.randint(min(2, deepest), min(5, deepest))
        view = {"fov": rng.choice((0.0, 70.0, 110.0)), "yaw": rng.uniform(-180.0, 180.0),
                "pitch": rng.uniform(-30.0, 30.0), "grey": grey, "foveate": rng.random() < 0.3}
        if kind == "encode":
            case = _encode("", width, height, tile, levels, wavelet, grey)
        elif kind == "rebuild":
            case = _rebuild("", width, height, tile, levels, wavelet, rng.choice((0.02, 0.1, 0.25)), **view)
        else:
            frames = rng.choice((2, 4)) if kind == "set" else rng.randint(1, GOP_LEN)
            case = _decode("", kind, width, height, tile, levels, wavelet, frames,
                           tuned=rng.random() < 0.3, **view)
            # no drawn case decodes more than the largest listed one
            budget = 36 * 512 * 512 * GOP_LEN // (1 if wavelet == "5/3" else 2)
            while _visible_samples(case) > budget:
                if case["fov"] == 0.0:
                    case["fov"] = 110.0
                elif kind != "set" and case["frames"] > 1:
                    case["frames"] -= 1
                else:
                    case["width"] = max(tile, case["width"] // 2 // tile * tile)
                    case["height"] = max(tile, case["height"] // 2 // tile * tile)
    del case["name"]
    return case


# ---------------------------------------------------------------- geometry
def _mask(case):
    """Visible tiles (uint8 per tile): the top eye's viewport, or all."""
    n = (case["width"] // case["tile"]) * (case["height"] // case["tile"])
    if case["fov"] == 0.0:
        return np.ones(n, np.uint8)
    m = wv.viewport_mask(case["width"], case["height"], case["tile"], case["yaw"], case["pitch"],
                         case["fov"], case["fov"])
    return m if m.any() else np.ones(n, np.uint8)


def _level_count(case):
    if not case["foveate"]:
        return None
    return wv.foveation_levels(case["width"], case["height"], case["tile"], case["levels"], case["yaw"],
                               case["pitch"])


def _visible_samples(case):
    return int(np.count_nonzero(_mask(case))) * case["tile"] ** 2 * case["frames"]


def _plane_edges(case):
    return (case["tile"],) if case["grey"] else (case["tile"], case["tile"] // 2, case["tile"] // 2)


def _kept(case):
    """Visible coefficients that the level counts keep, all planes."""
    vis = np.nonzero(_mask(case))[0]
    lc = _level_count(case)
    drop = np.zeros(len(vis), int) if lc is None else case["levels"] - lc[vis].astype(int)
    return sum(int(((edge >> drop).astype(np.int64) ** 2).sum()) for edge in _plane_edges(case))


# ------------------------------------------------------------------ inputs
def _generator(seed, device="cuda"):
    g = torch.Generator(device=device)
    g.manual_seed(seed)
    return g


def _laplace(shape, scale, gen):
    e = torch.empty(shape, device="cuda").exponential_(generator=gen)
    e -= torch.empty(shape, device="cuda").exponential_(generator=gen)
    return e.mul_(scale)


def _band_scale(edge, levels):
    """Spread of the detail coefficients of an edge x edge tile: a natural
    picture's, growing towards the coarse levels; 0 in the approximation."""
    s = torch.zeros(edge, edge, device="cuda")
    for k in range(1, levels + 1):
        m = edge >> (k - 1)
        s[:m, :m] = 3.0 * 2.0 ** (0.7 * (k - 1))
        s[:m // 2, :m // 2] = 0.0
    return s


def _intra_planes(case, gen, step):
    """Coefficients of a picture, on the multiples of step, as float32."""
    n = (case["width"] // case["tile"]) * (case["height"] // case["tile"])
    out = []
    for edge in _plane_edges(case):
        c = _laplace((n, edge, edge), 1.0, gen).mul_(_band_scale(edge, case["levels"]))
        a = edge >> case["levels"]
        level = 40.0 + 170.0 * torch.rand((n, 1, 1), device="cuda", generator=gen)
        c[:, :a, :a] = level + 12.0 * torch.randn((n, a, a), device="cuda", generator=gen)
        out.append(c.div_(step).round_().mul_(step))
    return out


def _residual_planes(case, gen, scale=2.0):
    n = (case["width"] // case["tile"]) * (case["height"] // case["tile"])
    return [_laplace((n, edge, edge), scale, gen) for edge in _plane_edges(case)]


def _stored(case, planes, step):
    """Values as they are stored: int16 indices (5/3) or float32 (9/7)."""
    if case["wavelet"] == "9/7":
        return planes
    return [(p / step).round_().to(torch.int16) for p in planes]


def _frames(case, seed):
    """(values, stored planes, is_intra, step) of each frame."""
    gen = _generator(seed)
    step = INTRA_STEP[case["wavelet"]]
    for t in range(case["frames"]):
        if t == 0:
            yield _stored(case, _intra_planes(case, gen, step), step), True, step
        else:
            yield _stored(case, _residual_planes(case, gen), 1), False, 1


def _set_bands(case, seed):
    """Per plane the bands [n][n_tiles][P][P]: a picture, then details."""
    gen = _generator(seed)
    bands = []
    for b in range(case["frames"]):
        step = SET_STEPS[b]
        planes = _intra_planes(case, gen, step) if b == 0 else _residual_planes(case, gen)
        bands.append(_stored(case, planes, step))
    return [torch.stack([b[p] for b in bands]) for p in range(len(bands[0]))]


def _source(case, seed):
    """8-bit picture planes: a gradient, noise and flat patches."""
    gen = _generator(seed)
    n = (case["width"] // case["tile"]) * (case["height"] // case["tile"])
    out = []
    for edge in _plane_edges(case):
        ramp = torch.linspace(0.0, 1.0, edge, device="cuda")
        p = 60.0 * torch.rand((n, 1, 1), device="cuda", generator=gen) + 64.0 * (ramp[:, None] + ramp)
        p = p + 8.0 * torch.randn((n, edge, edge), device="cuda", generator=gen)
        cells = (n, -(-edge // 32), -(-edge // 32))
        flat = torch.randint(0, 256, cells, device="cuda", generator=gen).float()
        flat[torch.rand(cells, device="cuda", generator=gen) < 0.8] = -1.0
        flat = flat.repeat_interleave(32, 1).repeat_interleave(32, 2)[:, :edge, :edge]
        out.append(torch.where(flat >= 0.0, flat, p).round_().clamp_(0, 255).to(torch.uint8))
    return out


def _net_params(seed):
    """He-normal weights, small biases, a last layer near the identity."""
    rng = np.random.default_rng(seed)
    parts = []
    for i, (ci, co) in enumerate(cnn.LAYERS):
        w = rng.normal(0.0, math.sqrt(2.0 / (9 * ci)), (co, 3, 3, ci))
        parts += [w * (0.05 if i == len(cnn.LAYERS) - 1 else 1.0), rng.normal(0.0, 0.01, co)]
    return cnn.flatten(parts)


def _train_batch(case, seed):
    gen = _generator(seed)
    shape = (case["n"], case["h"], case["w"], 4)
    t = 0.5 + 0.2 * torch.randn((case["n"], 1, 1, 4), device="cuda", generator=gen)
    t = t + 0.1 * torch.randn(shape, device="cuda", generator=gen)
    t = (t.clamp_(0.0, 1.0) * 255.0).round_() / 255.0
    x = (t + torch.randn(shape, device="cuda", generator=gen) * 0.03).clamp_(0.0, 1.0)
    t[..., 3] = 0.0
    x[..., 3] = 0.0
    return x.to(torch.bfloat16), t


# ----------------------------------------------------------------- prepare
def _decoder(case):
    return wv.Decoder(case["width"], case["height"], case["tile"], case["levels"],
                      wv.W53 if case["wavelet"] == "5/3" else wv.W97,
                      wv.GRAY8 if case["grey"] else wv.YUV420)


def prepare(case, seed):
    kind = case["kind"]
    st = {"case": case}
    if kind == "train":
        st["net"] = cnn.Net(case["n"] * case["h"] * case["w"])
        st["net"].set_params(_net_params(seed))
        st["x"], st["t"] = _train_batch(case, seed)
        st["z"] = torch.zeros(st["t"].shape, device="cuda")
        st["grads"] = torch.zeros(cnn.param_count(), device="cuda")
        return st
    if kind == "restore":
        tiles = case["tiles_x"] * case["tiles_y"]
        st["net"] = cnn.Net(tiles * case["tile"] ** 2)
        st["net"].set_params(_net_params(seed))
        gen = _generator(seed)
        shape = (tiles, 3, case["tile"], case["tile"])
        p = 60.0 + 120.0 * torch.rand((tiles, 3, 1, 1), device="cuda", generator=gen)
        p = p + 10.0 * torch.randn(shape, device="cuda", generator=gen)
        st["decoded"] = p.round_().clamp_(0, 255).to(torch.uint8)
        st["out"] = torch.empty_like(st["decoded"])
        return st
    dec = st["dec"] = _decoder(case)
    if kind == "encode":
        st["src"] = _source(case, seed)
        st["coef"] = [torch.zeros(dec.plane_shape(p), dtype=dec.coef_dtype, device="cuda")
                      for p in range(dec.nplanes)]
        return st
    mask = st["mask"] = _mask(case)
    st["lc"] = _level_count(case)
    n_vis = int(np.count_nonzero(mask))
    if kind == "rebuild":
        planes = _intra_planes(case, _generator(seed), 1.0)
        desc = wv.make_desc(case["width"], case["height"], case["tile"], case["levels"], dec.wavelet, dec.fmt)
        st["records"] = [fmt.DevicePlane(fmt.encode_plane(desc, p, planes[p].cpu().numpy(), case["alpha"], True))
                         for p in range(dec.nplanes)]
        st["dense"] = [torch.zeros(dec.plane_shape(p), dtype=dec.coef_dtype, device="cuda")
                       for p in range(dec.nplanes)]
        return st
    st["outs"] = [torch.zeros(dec.out_shape(n_vis), dtype=dec.sample_dtype, device="cuda")
                  for _ in range(case["frames"])]
    if kind == "set":
        st["bands"] = _set_bands(case, seed)
    else:
        st["frames"] = list(_frames(case, seed))
        st["ref"] = wv.Reference(dec)
    if case["tuned"]:
        dec.autotune(n_vis)
    return st


# --------------------------------------------------------------------- run
def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "train":
        net = state["net"]
        net.forward(state["x"], state["z"])
        loss = net.loss_grad(state["t"])
        net.backward(state["grads"])
        return [state["z"], loss, state["grads"]]
    if kind == "restore":
        out, fell = state["net"].restore(state["decoded"], case["tile"], case["tiles_x"], case["tiles_y"], 0.05,
                                         state["out"])
        return [out, fell]
    dec = state["dec"]
    if kind == "encode":
        dec.encode_intra(state["src"], state["coef"], INTRA_STEP[case["wavelet"]])
        return state["coef"]
    if kind == "rebuild":
        fmt.rebuild(dec, state["records"], state["mask"], state["dense"], state["lc"])
        return state["dense"]
    if kind == "set":
        dec.decode_set(state["bands"], case["frames"], SET_STEPS[:case["frames"]], 0, state["mask"],
                       state["outs"], state["lc"])
        return state["outs"]
    ref = state["ref"]
    if kind == "gop":
        dec.decode_gop(state["frames"], 0, state["mask"], ref, state["outs"], state["lc"])
    else:
        for t, (planes, intra, step) in enumerate(state["frames"]):
            dec.decode_viewport(planes, t, intra, step, state["mask"], ref, state["outs"][t], state["lc"])
    return [*state["outs"], *ref.planes]


# -------------------------------------------------------------------- work
# Lifting operations per sample and level, both directions.
LIFT_OPS = {"5/3": 6.0, "9/7": 10.0}


def work(case):
    kind = case["kind"]
    if kind == "train":
        px = case["n"] * case["h"] * case["w"]
        macs = sum(9 * ci * co for ci, co in cnn.LAYERS)
        first = 9 * cnn.LAYERS[0][0] * cnn.LAYERS[0][1]
        # forward, weight gradients, data gradients of all but the first layer;
        # x, t and z once, the parameters and their gradients
        return {"bytes": px * (8 + 16 + 16) + 8 * cnn.param_count(), "flops": 2.0 * px * (3 * macs - first)}
    if kind == "restore":
        px = case["tile"] ** 2 * case["tiles_x"] * case["tiles_y"]
        return {"bytes": 6 * px + 4 * cnn.param_count(),
                "flops": 2.0 * px * sum(9 * ci * co for ci, co in cnn.LAYERS)}
    cb, sb = (2, 1) if case["wavelet"] == "5/3" else (4, 4)
    ops = LIFT_OPS[case["wavelet"]] * 4.0 / 3.0
    n = (case["width"] // case["tile"]) * (case["height"] // case["tile"])
    per_tile = sum(e * e for e in _plane_edges(case))
    if kind == "encode":
        return {"bytes": n * per_tile * (1 + cb), "flops": n * per_tile * ops}
    n_vis, kept = int(np.count_nonzero(_mask(case))), _kept(case)
    if kind == "rebuild":
        # the kept part of the visible planes; the records are a few percent
        return {"bytes": kept * cb, "flops": 2.0 * kept}
    rgb = case["tile"] ** 2 * (1 if case["grey"] else 3)
    frames = case["frames"]
    if kind == "set":
        bands, refs = frames, 0
    elif kind == "gop":
        bands, refs = frames, 1            # only the last frame's reference has to leave the chip
    else:
        bands, refs = frames, 2 * frames - 1
    return {"bytes": kept * cb * bands + n_vis * sb * (rgb * frames + per_tile * refs),
            "flops": n_vis * per_tile * ops * frames}


# ------------------------------------------------------------------- exact
ALPHA, BETA, GAMMA, DELTA = -1.586134342059924, -0.052980118572961, 0.882911075530934, 0.443506852043971
KAPPA = 1.230174104914001


def _next(e):
    return torch.cat([e[..., 1:], e[..., -1:]], -1)


def _prev(o):
    return torch.cat([o[..., :1], o[..., :-1]], -1)


def _synthesis(c):
    m = c.shape[-1] // 2
    e, o = c[..., :m] * KAPPA, c[..., m:] / KAPPA
    e = e - DELTA * (_prev(o) + o)
    o = o - GAMMA * (e + _next(e))
    e = e - BETA * (_prev(o) + o)
    o = o - ALPHA * (e + _next(e))
    return torch.stack([e, o], -1).flatten(-2)


def _analysis(x):
    e, o = x[..., 0::2], x[..., 1::2]
    o = o + ALPHA * (e + _next(e))
    e = e + BETA * (_prev(o) + o)
    o = o + GAMMA * (e + _next(e))
    e = e + DELTA * (_prev(o) + o)
    return torch.cat([e / KAPPA, o * KAPPA], -1)


def _inverse(c, levels, dropped):
    """9/7 inverse of tiles [n, P, P]; dropped: finest levels without detail."""
    c = c.double().clone()
    edge = c.shape[-1]
    for k in range(levels, 0, -1):
        m = edge >> (k - 1)
        r = c[:, :m, :m].clone()
        off = dropped >= k
        r[off, m // 2:, :] = 0.0
        r[off, :m // 2, m // 2:] = 0.0
        r = _synthesis(r)
        c[:, :m, :m] = _synthesis(r.transpose(1, 2)).transpose(1, 2)
    return c


def _rgb(rec):
    if len(rec) == 1:
        return rec[0][:, None].clone()
    cb, cr = ((p - 128.0).repeat_interleave(2, 1).repeat_interleave(2, 2) for p in rec[1:])
    y = rec[0]
    rgb = [y + 1.402 * cr, y - 0.344136 * cb - 0.714136 * cr, y + 1.772 * cb]
    return torch.stack(rgb, 1).clamp_(0.0, 255.0)


def _exact_decode(case, seed):
    vis = torch.from_numpy(np.nonzero(_mask(case))[0]).cuda()
    lc = _level_count(case)
    dropped = torch.zeros(len(vis), dtype=torch.int64, device="cuda")
    if lc is not None:
        dropped = case["levels"] - torch.from_numpy(lc.astype(np.int64)).cuda()[vis]
    outs, rec = [], None
    if case["kind"] == "set":
        bands = [b[:, vis].double() for b in _set_bands(case, seed)]
        n = case["frames"]
        for t in range(n):
            rec = []
            for b in bands:
                if n == 4:
                    c = b[0] + (-b[1] if t & 2 else b[1]) + (-b[2 + t // 2] if t & 1 else b[2 + t // 2])
                else:
                    c = b[0] + (-b[1] if t & 1 else b[1])
                rec.append(_inverse(c, case["levels"], dropped).clamp_(0.0, 255.0))
            outs.append(_rgb(rec))
        return outs
    for planes, intra, _ in _frames(case, seed):
        pix = [_inverse(p[vis], case["levels"], dropped) for p in planes]
        rec = [(p if intra else r + p).clamp_(0.0, 255.0) for p, r in zip(pix, rec or pix)]
        outs.append(_rgb(rec))
    n = (case["width"] // case["tile"]) * (case["height"] // case["tile"])
    for r in rec:
        full = torch.zeros((n, *r.shape[1:]), dtype=torch.float64, device="cuda")
        full[vis] = r
        outs.append(full)
    return outs


def _exact_encode(case, seed):
    step = INTRA_STEP[case["wavelet"]]
    out = []
    for src in _source(case, seed):
        c = src.double()
        for k in range(1, case["levels"] + 1):
            m = c.shape[-1] >> (k - 1)
            r = _analysis(c[:, :m, :m].transpose(1, 2)).transpose(1, 2)
            c[:, :m, :m] = _analysis(r)
        out.append(torch.sign(c) * torch.floor(c.abs() / step + 0.5) * step)
    return out


def _exact_train(case, seed):
    x, t = (v.double()[..., :3].permute(0, 3, 1, 2) for v in _train_batch(case, seed))
    parts = [torch.from_numpy(p).cuda().requires_grad_() for p in cnn.unflatten(_net_params(seed))]
    a = x
    for i, (ci, co) in enumerate(cnn.LAYERS):
        w = parts[2 * i].permute(0, 3, 1, 2).reshape(co, 9 * ci)
        a = w @ torch.nn.functional.unfold(a, 3, padding=1) + parts[2 * i + 1][:, None]
        a = (a.relu() if i + 1 < len(cnn.LAYERS) else a).reshape(case["n"], co, case["h"], case["w"])
    loss = ((x + a - t) ** 2).mean()
    loss.backward()
    z = torch.nn.functional.pad(a.detach().permute(0, 2, 3, 1), (0, 1))
    return [z, loss.detach().reshape(1), torch.cat([p.grad.reshape(-1) for p in parts])]


def exact(case, seed):
    """The float results in 64 bits.  The 5/3 results and restored pictures are
    whole numbers; a rebuilt plane is made of stored codes."""
    if case["kind"] == "train":
        return _exact_train(case, seed)
    if case["kind"] in ("restore", "rebuild") or case["wavelet"] == "5/3":
        return None
    return _exact_encode(case, seed) if case["kind"] == "encode" else _exact_decode(case, seed)
