"""What a program asks of this library, as cases that can be timed and compared.

Every case is one pass through the public entry points on a T x H x W grid of video tokens plus text
tokens, with a seeded mix of local, cross-shaped and global heads.  The listed cases take the shapes
of the configurations, tests and benchmark of this repository, or generic ones between them; `draw`
fills in the ranges they span.

`op`, what is called:
  step     compact_attn_permute on q, k and v, compact_attn_forward, inverse compact_attn_permute: one
           attention call of a model that keeps its activations in natural token order
  forward  compact_attn_forward on tensors that already are in tile order
  natural  compact_attn_forward_natural
  dense    compact_attn_dense: the full-attention steps at the start of a sampling run, and the baseline
  static   compact_attn_forward_static: the entry point without allocations
  mass     compact_attn_tile_mass: the input of the mask search

Layouts (compact_attn_build_layout) are made and uploaded once and kept, as a program does that calls
the same layer at every denoising step.
"""
import math
import random

import numpy as np
import torch

import paper_2508_12969_amd as ca

ABSENT = (-1, -1)
DEVICE = "cuda:0"
DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}


def _case(name, op, grid, tile, n_text, heads, head_dim, dtype, reach, mask_seed, batch=1):
    case = dict(zip(("T", "H", "W"), grid)) | dict(zip(("tt", "th", "tw"), tile))
    case |= dict(op=op, n_text=n_text, heads=heads, head_dim=head_dim, dtype=dtype, reach=reach, mask_seed=mask_seed, batch=batch)
    return dict(name=name, **case) if name else case


def listed():
    return [
        # the smallest call: two heads on 256 tokens in fp32; latency and launches are all there is
        _case("step-f32-256tok", "step", (4, 8, 8), (1, 4, 4), 0, 2, 64, "f32", 0.3, 1),
        # fp32 on a ragged grid: checks of a model in full precision, and small models that run in it
        _case("forward-f32-7Ktok", "forward", (7, 30, 33), (1, 8, 8), 64, 8, 128, "f32", 0.4, 2),
        # small model: 64-token tiles, head dim 64, a few thousand tokens
        _case("step-d64-8Ktok", "step", (8, 32, 32), (1, 8, 8), 0, 12, 64, "bf16", 0.5, 3),
        # head dim 64 with 128-token tiles on a grid that no axis divides, two batch entries (guided and unguided)
        _case("forward-d64-b2-20Ktok", "forward", (13, 30, 52), (2, 8, 8), 128, 12, 64, "bf16", 0.4, 4, batch=2),
        # one rank's share of the heads of a short clip, in a loop that must not allocate
        _case("static-3heads-15Ktok", "static", (9, 30, 52), (2, 8, 8), 128, 3, 128, "bf16", 0.4, 5),
        # low-resolution clip, activations in natural order, gather and scatter in the kernel
        _case("natural-33Ktok", "natural", (21, 30, 52), (2, 8, 8), 256, 24, 128, "bf16", 0.3, 6),
        # full attention on the same kind of clip
        _case("dense-20Ktok", "dense", (13, 30, 52), (1, 8, 8), 0, 16, 128, "bf16", 1.0, 7),
        # 75K video tokens, 64-token tiles, 40 heads
        _case("step-75Ktok", "step", (21, 45, 80), (1, 8, 8), 0, 40, 128, "bf16", 0.6, 8),
        # 119K video tokens and text, 128-token tiles, 24 heads
        _case("step-119Ktok", "step", (33, 45, 80), (2, 8, 8), 256, 24, 128, "bf16", 0.45, 9),
        # long clip at high sparsity: the most tokens
        _case("forward-230Ktok", "forward", (64, 45, 80), (2, 8, 8), 0, 24, 128, "bf16", 0.08, 10),
        # tile masses of a small model for the mask search
        _case("mass-d64-12Ktok", "mass", (8, 30, 52), (1, 8, 8), 64, 12, 64, "bf16", 1.0, 11),
        # tile masses of half of the heads of the 119K-token layer
        _case("mass-119Ktok", "mass", (33, 45, 80), (2, 8, 8), 256, 12, 128, "bf16", 1.0, 12),
    ]


def draw(rng):
    limits = {}
    for c in listed():
        w = work(c)
        for key in ("flops", "bytes"):
            limits[_family(c), key] = max(limits.get((_family(c), key), 0), w[key])

    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    while True:
        dtype = "f32" if rng.random() < 0.2 else "bf16"
        if dtype == "f32":
            op = rng.choice(["step", "forward", "dense"])
            head_dim = rng.choice([32, 64, 128])
            tile = rng.choice([(1, 4, 4), (1, 8, 8), (2, 2, 4), (1, 6, 10), (2, 4, 8), (2, 8, 8)])
        else:
            op = rng.choice(["step", "step", "forward", "forward", "natural", "dense", "static", "mass"])
            head_dim = rng.choice([64, 128, 128])
            tile = rng.choice([(1, 8, 8), (2, 4, 8), (2, 8, 8), (2, 8, 8), (1, 8, 16), (4, 4, 8)])
        grid = (log_int(1, 64), log_int(8, 60), log_int(8, 104))
        n_text = rng.choice([0, 0, 1, 2, 3]) * tile[0] * tile[1] * tile[2]
        case = _case(None, op, grid, tile, n_text, log_int(1, 40), head_dim, dtype, round(rng.uniform(0.05, 1.0), 2),
                     rng.randrange(1 << 30), batch=rng.choice([1, 1, 1, 2]))
        w = work(case)
        if any(w[key] > limits[_family(case), key] for key in ("flops", "bytes")):
            continue
        if op == "static" and _tile_pairs(case) > 1_000_000:  # its tables must fit the fixed device array
            continue
        return case


def _family(case):
    return "mass" if case["op"] == "mass" else case["dtype"]


# ---- geometry and masks -----------------------------------------------------------------------------

def _tiles(case):
    return tuple(-(-case[n] // case[t]) for n, t in (("T", "tt"), ("H", "th"), ("W", "tw")))


def _head_groups(case):
    """Per head (max tile-frame distance, window, window) groups: a seeded mix of local, cross-shaped and global heads."""
    nT, nH, nW = _tiles(case)
    heads = []
    for h in range(case["heads"]):
        r = random.Random(f"{case['mask_seed']}/{h}")
        kind = r.choice(["L1", "L1", "L2", "L3", "C0", "C0", "C1", "C1", "G", "G"])
        far = r.randint(0, max(0, math.ceil(case["reach"] * (nT - 1))))
        if kind == "G":
            windows = (nH - 1, nW - 1), ABSENT
            if r.random() < case["reach"]:
                far = nT - 1
        elif kind[0] == "L":
            windows = (int(kind[1]),) * 2, ABSENT
        else:
            windows = (int(kind[1]), nW - 1), (nH - 1, int(kind[1]))
        groups = [(far, *windows)]
        extra = r.randint(0, 2)
        if extra and far + extra < nT:
            groups.append((far + extra, (1, 1), ABSENT))
        heads.append(groups)
    return heads


def _pairs_within(sizes, radius):
    """Sum of sizes[i] * sizes[j] over all i, j at most `radius` apart."""
    i = np.arange(len(sizes))
    near = np.abs(i[:, None] - i[None, :]) <= radius
    return int(sizes @ near @ sizes)


def _kept_pairs(case, sizes_t, sizes_h, sizes_w, text):
    """Kept (query, key) pairs over all heads, for units of the given sizes along each axis and `text` text units."""
    video = int(sizes_t.sum() * sizes_h.sum() * sizes_w.sum())
    if case["op"] in ("dense", "mass"):
        return case["heads"] * (video + text) ** 2
    total = 0
    for groups in _head_groups(case):
        seen = 0
        for max_dt, a, b in groups:
            at_distance = _pairs_within(sizes_t, max_dt) - seen
            seen += at_distance
            area = sum(_pairs_within(sizes_h, w[0]) * _pairs_within(sizes_w, w[1]) for w in (a, b) if w != ABSENT)
            if b != ABSENT:
                area -= _pairs_within(sizes_h, min(a[0], b[0])) * _pairs_within(sizes_w, min(a[1], b[1]))
            total += at_distance * area
        total += 2 * video * text + text * text
    return total


def _axis_sizes(length, tile):
    return np.array([min(tile, length - i) for i in range(0, length, tile)], dtype=np.int64)


def _tile_pairs(case):
    nT, nH, nW = _tiles(case)
    one = lambda n: np.ones(n, dtype=np.int64)
    return _kept_pairs(case, one(nT), one(nH), one(nW), case["n_text"] // (case["tt"] * case["th"] * case["tw"]))


def work(case):
    """Products over pairs of real tokens, softmax not counted; every tensor once."""
    nT, nH, nW = _tiles(case)
    B = case["tt"] * case["th"] * case["tw"]
    real = case["T"] * case["H"] * case["W"] + case["n_text"]
    padded = nT * nH * nW * B + case["n_text"]
    pairs = _kept_pairs(case, _axis_sizes(case["T"], case["tt"]), _axis_sizes(case["H"], case["th"]),
                        _axis_sizes(case["W"], case["tw"]), case["n_text"])
    rows = case["batch"] * case["heads"]
    token_bytes = case["head_dim"] * (2 if case["dtype"] == "bf16" else 4)
    if case["op"] == "mass":
        n = padded // B
        return {"bytes": rows * (2 * real * token_bytes + 4 * n * n), "flops": 2 * case["batch"] * pairs * case["head_dim"]}
    out = real if case["op"] in ("step", "natural") else padded
    return {"bytes": rows * (3 * real + out) * token_bytes, "flops": 4 * case["batch"] * pairs * case["head_dim"]}


# ---- inputs -----------------------------------------------------------------------------------------

def _position_code(case):
    """A smooth code of (t, y, x) in sines and cosines, zero for text tokens; [tokens, head_dim]."""
    axes = [torch.arange(case[n], device=DEVICE, dtype=torch.float32) / case[n] for n in ("T", "H", "W")]
    coords = torch.stack(torch.meshgrid(*axes, indexing="ij"), dim=-1).reshape(-1, 3)
    channel = torch.arange(case["head_dim"], device=DEVICE)
    pair = channel // 3
    phase = math.pi * coords[:, channel % 3] * (pair // 2 + 1)
    code = torch.where(pair % 2 == 0, torch.sin(phase), torch.cos(phase))
    return torch.cat([code, torch.zeros(case["n_text"], case["head_dim"], device=DEVICE)])


def _natural_qkv(case, seed):
    """q, k, v [batch, heads, tokens, head_dim]: half the position code plus unit noise."""
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(seed)
    code = 0.5 * _position_code(case)
    out = []
    for _ in range(2 if case["op"] == "mass" else 3):
        x = torch.empty(case["batch"], case["heads"], *code.shape, dtype=DTYPES[case["dtype"]], device=DEVICE)
        for b in range(case["batch"]):
            for h in range(case["heads"]):
                x[b, h] = torch.randn(code.shape, generator=gen, device=DEVICE) + code
        out.append(x)
    return out


def prepare(case, seed):
    layout = ca.compact_attn_build_layout(case["T"], case["H"], case["W"], (case["tt"], case["th"], case["tw"]), case["n_text"],
                                          case["batch"], case["heads"], case["head_dim"], case["dtype"], _head_groups(case))
    ca.compact_attn_layout_upload(layout)
    inputs = _natural_qkv(case, seed)
    if case["op"] not in ("step", "natural"):
        inputs = [ca.compact_attn_permute(x, layout) for x in inputs]
    return {"op": case["op"], "layout": layout, "inputs": inputs}


def run(state):
    op, layout, inputs = state["op"], state["layout"], state["inputs"]
    if op == "step":
        q, k, v = (ca.compact_attn_permute(x, layout) for x in inputs)
        return ca.compact_attn_permute(ca.compact_attn_forward(q, k, v, layout), layout, inverse=True)
    entry = {"forward": ca.compact_attn_forward, "natural": ca.compact_attn_forward_natural, "dense": ca.compact_attn_dense,
             "static": ca.compact_attn_forward_static, "mass": ca.compact_attn_tile_mass}[op]
    return entry(*inputs, layout)


# ---- expected results -------------------------------------------------------------------------------

def tolerance(case):
    # About four times what is measured against `exact`: 1.6e-3 .. 1.9e-3 for bf16 attention (probabilities
    # and results are rounded to bf16), 4e-7 .. 1.2e-6 for fp32 attention and 5e-8 .. 7e-8 for tile masses,
    # whose few hundred fp32 sums another order of summation moves more than the present one.
    if case["op"] == "mass":
        return {"rel": 1e-6}
    return {"rel": 7e-3} if case["dtype"] == "bf16" else {"rel": 5e-6}


def _token_places(case):
    """Position in tile order of every natural-order token."""
    nT, nH, nW = _tiles(case)
    t, y, x = np.meshgrid(np.arange(case["T"]), np.arange(case["H"]), np.arange(case["W"]), indexing="ij")
    tile = ((t // case["tt"]) * nH + y // case["th"]) * nW + x // case["tw"]
    slot = ((t % case["tt"]) * case["th"] + y % case["th"]) * case["tw"] + x % case["tw"]
    B = case["tt"] * case["th"] * case["tw"]
    places = np.concatenate([(tile * B + slot).reshape(-1), nT * nH * nW * B + np.arange(case["n_text"])])
    return torch.from_numpy(places).to(DEVICE)


def _keep_matrix(case, groups):
    """bool [n, n]: key tiles that each query tile of a head keeps."""
    nT, nH, nW = _tiles(case)
    n_vid = nT * nH * nW
    n = n_vid + case["n_text"] // (case["tt"] * case["th"] * case["tw"])
    keep = np.ones((n, n), dtype=bool)
    if case["op"] in ("dense", "mass"):
        return keep
    ids = np.arange(n_vid)
    dist = [np.abs(c[:, None] - c[None, :]) for c in (ids // (nH * nW), ids // nW % nH, ids % nW)]
    video, last = np.zeros((n_vid, n_vid), dtype=bool), -1
    for max_dt, a, b in groups:
        inside = ((dist[1] <= a[0]) & (dist[2] <= a[1])) | ((dist[1] <= b[0]) & (dist[2] <= b[1]))
        video |= inside & (dist[0] > last) & (dist[0] <= max_dt)
        last = max_dt
    keep[:n_vid, :n_vid] = video
    return keep


def exact(case, seed):
    nT, nH, nW = _tiles(case)
    B = case["tt"] * case["th"] * case["tw"]
    padded = nT * nH * nW * B + case["n_text"]
    n, D = padded // B, case["head_dim"]
    if case["batch"] * case["heads"] * 4 * padded * padded * D > 2.5e14:
        return None
    inputs = _natural_qkv(case, seed)
    places = _token_places(case)
    real = torch.zeros(padded, dtype=torch.bool, device=DEVICE)
    real[places] = True
    mass = case["op"] == "mass"
    shape = (case["batch"], case["heads"], n, n) if mass else (case["batch"], case["heads"], padded, D)
    result = torch.zeros(shape, dtype=torch.float64, device=DEVICE)
    tiles_at_once = max(1, (1 << 27) // (padded * B))
    for h, groups in enumerate(_head_groups(case)):
        keep = torch.from_numpy(_keep_matrix(case, groups)).to(DEVICE)
        for b in range(case["batch"]):
            planes = []
            for x in inputs:
                plane = torch.zeros(padded, D, dtype=torch.float64, device=DEVICE)
                plane[places] = x[b, h].double()
                planes.append(plane)
            q = planes[0] / math.sqrt(D)
            k_t = planes[1].t().contiguous()
            for lo in range(0, n, tiles_at_once):
                hi = min(n, lo + tiles_at_once)
                p = (q[lo * B:hi * B] @ k_t).view(hi - lo, B, n, B)
                p.masked_fill_(~(keep[lo:hi, None, :, None] & real.view(1, 1, n, B)), -math.inf)
                p = p.view((hi - lo) * B, padded)
                p -= p.amax(dim=1, keepdim=True).clamp_(min=-1e300)
                p.exp_()
                total = p.sum(dim=1, keepdim=True)
                weight = torch.where(real[lo * B:hi * B, None] & (total > 0), 1 / total, torch.zeros_like(total))
                if mass:
                    per_tile = p.view(-1, n, B).sum(dim=2) * weight
                    result[b, h, lo:hi] = per_tile.view(hi - lo, B, n).sum(dim=1)
                else:
                    result[b, h, lo * B:hi * B] = (p @ planes[2]) * weight
                del p
    return result[:, :, places] if case["op"] in ("step", "natural") else result
