"""What this framework is timed on: its public entry points over the range of batches they serve.

A codec built on the library runs three kinds of pass: the coder under a logistic law per subpixel
(small batches that are all launch latency, a few thousand long lanes, a lane per row, tiles of
video frames and of photographs whose sides divide by nothing), the paper's table-driven coder, and
the residual transform around it; the mixture coder is the heavy variant of the first.  `listed`
holds one case for each of these uses, `draw` takes further ones from the same ranges.

Everything is integer: a coded container and a decoded image are right or wrong, hence "exact".
"""
from __future__ import annotations

import math

import torch
import torch.nn.functional as F

from paper_2206_05279_amd import binding as pb
from paper_2206_05279_amd import synth_pieces

DEVICE = "cuda:0"

# The twelve parameters of the residual transform: the plane predictor for red, and for green and
# blue the value to the left corrected by what the channel before it did.  Q2.14.
_ONE = 1 << 14
TWAR_WEIGHTS = [[-_ONE, _ONE, _ONE], [_ONE, -_ONE, _ONE], [_ONE, -_ONE, _ONE]]
TWAR_BIAS = [0, 0, 0]


def _lanes(name, op, n, h, w, prec_bits, lane_mode, lane_a, lane_b, mean_error, scale_low, scale_high):
    """A batch for the coder under one logistic law per subpixel.  mean_error: standard deviation of
    the predicted mean around the pixel; the log-scales are uniform in [scale_low, scale_high]."""
    return {"name": name, "path": "lanes", "op": op, "n": n, "h": h, "w": w, "prec_bits": prec_bits,
            "lane_mode": lane_mode, "lane_a": lane_a, "lane_b": lane_b, "mean_error": mean_error,
            "scale_low": scale_low, "scale_high": scale_high}


def _mixture(name, op, n, h, w, prec_bits, lane_mode, lane_a, lane_b, components):
    c = _lanes(name, op, n, h, w, prec_bits, lane_mode, lane_a, lane_b, 3.0, -1.5, 2.5)
    c.update(path="mixture", components=components)
    return c


def _table(name, op, pieces, count, prec_bits, laws):
    return {"name": name, "path": "table", "op": op, "pieces": pieces, "count": count,
            "prec_bits": prec_bits, "laws": laws}


def _residual(name, op, n, h, w):
    return {"name": name, "path": "residual", "op": op, "n": n, "h": h, "w": w}


def listed():
    return [
        # a handful of thumbnails compressed and read back: nothing but launches and latency
        _lanes("small_round_trip", "round_trip", 64, 32, 32, 14, 0, 32, 0, 4.0, -1.0, 3.0),
        # a CIFAR-sized archive in 3125 long lanes (16 images each): the smallest overhead per lane
        _lanes("long_lanes_encode", "encode", 50000, 32, 32, 14, 0, 16384, 0, 4.0, -1.0, 3.0),
        _lanes("long_lanes_decode", "decode", 50000, 32, 32, 14, 0, 16384, 0, 4.0, -1.0, 3.0),
        # an ImageNet64-sized archive with a lane per row: as many lanes as the chip can use
        _lanes("row_lanes_encode", "encode", 16384, 64, 64, 15, 0, 64, 0, 3.0, -1.5, 2.5),
        # a second of 1080p30 video in 16 x 16 tiles (clipped at the bottom), on the playing side
        _lanes("video_tiles_decode", "decode", 30, 1080, 1920, 15, 1, 16, 16, 2.0, -2.0, 2.0),
        # photographs with odd sides in the same tiles: nothing is aligned, edge tiles are 5 x 15
        _lanes("photo_tiles_decode", "decode", 8, 1365, 2047, 12, 1, 16, 16, 3.0, -1.5, 2.5),
        # the table-driven coder on the paper's own measurement: 10^6 pieces of 1000 symbols, 8 laws
        _table("table_encode", "encode", 1000000, 1000, 12, 8),
        _table("table_decode", "decode", 1000000, 1000, 12, 8),
        # the residual transform: a second of video read back, and photographs with odd sides both ways
        _residual("video_residual_inverse", "inverse", 30, 1080, 1920),
        _residual("photo_residual_round_trip", "round_trip", 16, 1365, 2047),
        # ten laws per subpixel, as the learned codecs that the paper compares itself with have
        _mixture("mixture_encode", "encode", 2048, 64, 64, 15, 0, 64, 0, 10),
        _mixture("mixture_decode", "decode", 2048, 64, 64, 15, 0, 64, 0, 10),
    ]


def _log_uniform(rng, low, high):
    return int(round(math.exp(rng.uniform(math.log(low), math.log(high)))))


def _draw_image_batch(rng, pixels_low, pixels_high, h_high, w_high):
    pixels = _log_uniform(rng, pixels_low, pixels_high)
    h = min(_log_uniform(rng, 8, h_high), pixels // 8)
    w = max(1, min(_log_uniform(rng, 8, w_high), pixels // h))
    return max(1, pixels // (h * w)), h, w


def _draw_lanes(rng, h, w, most_pixels):
    """Rows, whole images or several of them, or tiles as lanes of at most `most_pixels` pixels."""
    pick = rng.random()
    if pick < 0.3 and w <= most_pixels:
        return 0, w, 0
    if pick < 0.5 and h * w <= most_pixels:
        return 0, h * w * rng.randint(1, max(1, min(64, most_pixels // (h * w)))), 0
    return 1, rng.choice((8, 16, rng.randint(4, 32))), rng.choice((8, 16, 32, rng.randint(4, 32)))


def draw(rng):
    path = rng.choice(("lanes", "lanes", "lanes", "table", "residual", "mixture"))
    if path == "lanes":
        op = rng.choice(("encode", "decode", "round_trip"))
        n, h, w = _draw_image_batch(rng, 1 << 14, 1 << (18 if op == "round_trip" else 26), 1365, 2047)
        mode, a, b = _draw_lanes(rng, h, w, 16384)
        low = rng.uniform(-2.0, -1.0)
        case = _lanes("", op, n, h, w, rng.randint(10, 16), mode, a, b, rng.uniform(2.0, 4.0), low, low + 4.0)
    elif path == "mixture":
        components = rng.choice((2, 3, 4, 5, 8, 10, 16))
        n, h, w = _draw_image_batch(rng, 1 << 14, (80 << 20) // components, 1365, 2047)
        mode, a, b = _draw_lanes(rng, h, w, 512)
        case = _mixture("", rng.choice(("encode", "decode")), n, h, w, rng.randint(10, 16), mode, a, b, components)
    elif path == "table":
        symbols = _log_uniform(rng, 1 << 18, 1000000000)
        count = _log_uniform(rng, 64, 4096)
        case = _table("", rng.choice(("encode", "decode")), max(1, symbols // count), count,
                      rng.choice((10, 11, 12, 13)), rng.choice((1, 2, 4, 8)))
    else:
        n, h, w = _draw_image_batch(rng, 1 << 14, 1 << 25, 1365, 2047)
        case = _residual("", rng.choice(("forward", "inverse", "round_trip")), n, h, w)
    del case["name"]
    return case


# ------------------------------------------------------------------------------------------ inputs
def _generator(seed):
    return torch.Generator(device=DEVICE).manual_seed(int(seed))


def _u16(values):
    """float values in 0 .. 65535 -> uint16 (through the 16 bits of an int16)."""
    return values.round_().to(torch.int32).to(torch.int16).view(torch.uint16)


def _images(g, n, h, w):
    """Smooth colour fields in two octaves and noise of a strength of each image's own, uint8 [n,h,w,3]."""
    out = torch.empty((n, h, w, 3), dtype=torch.uint8, device=DEVICE)
    step = max(1, (1 << 23) // (h * w))
    for i in range(0, n, step):
        b = min(step, n - i)
        x = torch.zeros((b, 3, h, w), device=DEVICE)
        for share, cell in ((0.75, 32), (0.25, 4)):
            field = torch.rand((b, 3, 2 + h // cell, 2 + w // cell), generator=g, device=DEVICE)
            x += 255.0 * share * F.interpolate(field, size=(h, w), mode="bilinear", align_corners=False)
        sigma = 2.0 + 6.0 * torch.rand((b, 1, 1, 1), generator=g, device=DEVICE)
        x += sigma * torch.randn((b, 3, h, w), generator=g, device=DEVICE)
        out[i:i + b] = x.clamp_(0, 255).round_().to(torch.uint8).permute(0, 2, 3, 1)
    return out


def _logistic_params(g, img, mean_error, low, high):
    """A predictor's output for `img`: means near the pixels, log-scales, channel coefficients."""
    mu = torch.randn(img.shape, generator=g, device=DEVICE).mul_(mean_error).add_(img).mul_(256.0)
    mu = _u16(mu.clamp_(0, 65535))
    ls = torch.rand(img.shape, generator=g, device=DEVICE).mul_((high - low) * 4096.0).add_(low * 4096.0)
    coef = torch.rand((img.shape[0], 3), generator=g, device=DEVICE).mul_(16384.0)
    return mu, ls.round_().to(torch.int16), coef.round_().to(torch.int16)


def _mixture_params(g, img, case):
    """Component 0 as above, the others wider and further off; weights that sum to 2^15 exactly."""
    k = case["components"]
    mu0, ls0, coef = _logistic_params(g, img, case["mean_error"], case["scale_low"], case["scale_high"])
    mu = torch.empty(img.shape + (k,), dtype=torch.uint16, device=DEVICE)
    ls = torch.empty(img.shape + (k,), dtype=torch.int16, device=DEVICE)
    weight = torch.empty(img.shape[:3] + (k,), dtype=torch.uint16, device=DEVICE)
    step = max(1, (1 << 22) // (img.shape[1] * img.shape[2]))
    for i in range(0, img.shape[0], step):
        part = img[i:i + step]
        m = torch.randn(part.shape + (k,), generator=g, device=DEVICE).mul_(24.0).add_(part[..., None])
        mu[i:i + step] = _u16(m.clamp_(0.0, 255.99).mul_(256.0))
        s = torch.rand(part.shape + (k,), generator=g, device=DEVICE).mul_(3.0 * 4096.0)
        ls[i:i + step] = s.round_().to(torch.int16)
        e = torch.rand(part.shape[:3] + (k,), generator=g, device=DEVICE).clamp_(min=1e-7).log_().neg_()
        e[..., 0] += 1.0
        q = (e / e.sum(-1, keepdim=True)).mul_(32768.0).floor_().to(torch.int32)
        rest = 32768 - q.sum(-1, keepdim=True, dtype=torch.int32)
        q.scatter_add_(-1, q.argmax(-1, keepdim=True), rest)
        weight[i:i + step] = q.to(torch.int16).view(torch.uint16)
    mu[..., 0] = mu0
    ls[..., 0] = ls0
    return mu, ls, weight, coef


def _pieces(g, case):
    """Symbols and law indices: for every symbol a law picked uniformly and the symbol drawn from it."""
    bits, laws = case["prec_bits"], case["laws"]
    mass = (synth_pieces.index_stream_masses(bits) if laws == 1 else synth_pieces.logistic_masses(bits, laws))
    d_mass = torch.from_numpy(mass).to(DEVICE)
    inverse = torch.repeat_interleave(torch.arange(256, dtype=torch.uint8).repeat(laws),
                                      torch.from_numpy(mass.astype("int64").reshape(-1))).to(DEVICE)
    shape = (case["pieces"], case["count"])
    sym = torch.empty(shape, dtype=torch.uint8, device=DEVICE)
    dist = torch.zeros(shape, dtype=torch.uint8, device=DEVICE)
    if laws > 1:
        torch.randint(0, laws, shape, generator=g, device=DEVICE, dtype=torch.uint8, out=dist)
    flat_s, flat_d = sym.view(-1), dist.view(-1)
    for i in range(0, flat_s.numel(), 1 << 26):
        d = flat_d[i:i + (1 << 26)]
        u = torch.randint(0, 1 << bits, d.shape, generator=g, device=DEVICE, dtype=torch.int32)
        flat_s[i:i + (1 << 26)] = inverse[u.add_(d.to(torch.int32) << bits)]
    return d_mass, sym, dist


def _bytes(count):
    return torch.empty(count, dtype=torch.uint8, device=DEVICE)


def _container(most_bytes):
    """The buffer an encoder writes its container to, given out whole: zeros after the container's end."""
    return torch.zeros(most_bytes, dtype=torch.uint8, device=DEVICE)


# ----------------------------------------------------------------------------------------- a state
class State:
    """What a program holds between calls: geometry, tables, workspace, buffers."""


def prepare(case, seed):
    g = _generator(seed)
    s = State()
    s.case = case
    if case["path"] == "table":
        s.shape = pb.make_ansai_shape(case["pieces"], case["count"], case["prec_bits"], case["laws"])
        mass, s.sym, s.dist = _pieces(g, case)
        s.tables = _bytes(pb.pilc_ansai_table_bytes(case["prec_bits"], case["laws"]))
        pb.pilc_ansai_build_tables(case["prec_bits"], case["laws"], 256, mass, s.tables)
        workspace, coded = pb.pilc_ansai_workspace_size(s.shape)
        s.workspace, s.coded = _bytes(workspace), _container(coded)
        if case["op"] == "decode":
            s.coded_bytes = _encode(s)
            s.coded = s.coded[:s.coded_bytes].clone()
            s.sym = torch.empty_like(s.sym)
        return s
    s.img = _images(g, case["n"], case["h"], case["w"])
    if case["path"] == "residual":
        s.params = pb.make_twar_params(TWAR_WEIGHTS, TWAR_BIAS)
        s.res = torch.empty_like(s.img)
        if case["op"] == "inverse":
            pb.pilc_twar_forward(s.params, s.img, s.res)
        if case["op"] == "round_trip":
            s.out = torch.empty_like(s.img)
        return s
    s.geom = pb.make_geom(case["n"], case["h"], case["w"], case["prec_bits"], case["lane_mode"],
                          case["lane_a"], case["lane_b"])
    if case["path"] == "mixture":
        s.mu, s.log_scale, s.weight, s.coef = _mixture_params(g, s.img, case)
    else:
        s.mu, s.log_scale, s.coef = _logistic_params(g, s.img, case["mean_error"], case["scale_low"],
                                                     case["scale_high"])
    workspace, coded = pb.pilc_workspace_size(s.geom)
    s.workspace, s.coded = _bytes(workspace), _container(coded)
    if case["op"] == "decode":
        s.coded_bytes = _encode(s)
        s.coded = s.coded[:s.coded_bytes].clone()
        s.img = torch.empty_like(s.img)
    if case["op"] == "round_trip":
        s.out = torch.empty_like(s.img)
    return s


# ------------------------------------------------------------------------------------------- a pass
def _encode(s):
    path = s.case["path"]
    if path == "table":
        return pb.pilc_ansai_encode(s.shape, s.sym, s.dist, s.tables, s.workspace, s.coded)[1]
    if path == "mixture":
        return pb.pilc_mix_encode(s.geom, s.case["components"], s.img, s.mu, s.log_scale, s.weight, s.coef,
                                  s.workspace, s.coded)[1]
    return pb.pilc_encode(s.geom, s.img, s.mu, s.log_scale, s.coef, s.workspace, s.coded)[1]


def _decode(s, coded_bytes, out):
    path = s.case["path"]
    if path == "table":
        pb.pilc_ansai_decode(s.shape, s.coded, coded_bytes, s.dist, s.tables, s.workspace, out)
    elif path == "mixture":
        pb.pilc_mix_decode(s.geom, s.case["components"], s.coded, coded_bytes, s.mu, s.log_scale, s.weight,
                           s.coef, s.workspace, out)
    else:
        pb.pilc_decode(s.geom, s.coded, coded_bytes, s.mu, s.log_scale, s.coef, s.workspace, out)


def run(s):
    op = s.case["op"]
    if s.case["path"] == "residual":
        if op == "inverse":
            pb.pilc_twar_inverse(s.params, s.res, s.img)
            return {"image": s.img}
        pb.pilc_twar_forward(s.params, s.img, s.res)
        if op == "forward":
            return {"residual": s.res}
        pb.pilc_twar_inverse(s.params, s.res, s.out)
        return {"residual": s.res, "image": s.out}
    if op == "decode":
        out = s.sym if s.case["path"] == "table" else s.img
        _decode(s, s.coded_bytes, out)
        return {"decoded": out}
    coded_bytes = _encode(s)
    outputs = {"coded": s.coded, "coded_bytes": coded_bytes}
    if op == "round_trip":
        _decode(s, coded_bytes, s.out)
        outputs["decoded"] = s.out
    return outputs


# ------------------------------------------------------------------------------------------- bounds
def _lane_count(case):
    if case["lane_mode"] == 0:
        return -(-case["n"] * case["h"] * case["w"] // case["lane_a"])
    return case["n"] * -(-case["h"] // case["lane_a"]) * -(-case["w"] // case["lane_b"])


def work(case):
    """Bytes: every input read once, every output written once (6 coded bits per symbol, near what
    these inputs take, and the per-lane record).  Operations: integer ones, counted the cheapest way
    the definitions allow: two evaluations of the law per symbol (about 12 operations each, per
    component), the coder's step (about 10), a table step (about 10), a prediction (about 8)."""
    passes = 2 if case["op"] == "round_trip" else 1
    if case["path"] == "table":
        symbols = case["pieces"] * case["count"]
        return {"bytes": 2 * symbols + symbols * 6 // 8 + 12 * case["pieces"], "flops": 10 * symbols}
    subpixels = 3 * case["n"] * case["h"] * case["w"]
    if case["path"] == "residual":
        return {"bytes": passes * 2 * subpixels, "flops": passes * 8 * subpixels}
    coded = subpixels * 6 // 8 + 8 * _lane_count(case)
    if case["path"] == "mixture":
        k = case["components"]
        params = 4 * k * subpixels + 2 * k * (subpixels // 3)
        return {"bytes": passes * (subpixels + params + coded), "flops": passes * subpixels * (24 * k + 10)}
    return {"bytes": passes * (5 * subpixels + coded), "flops": passes * 34 * subpixels}


def tolerance(case):
    return "exact"
