"""Parity of the HIP path (through the C ABI) with the fp64 oracle, on a real MI355X.

Layouts and permutations are compared bit for bit; attention outputs within
max-abs 2e-2 / mean-abs 2e-3 for bf16 and 1e-4 / 1e-5 for fp32.
"""
import math

import numpy as np
import pytest
import torch

import paper_2508_12969_amd as ca
from oracle import attention as OA
from oracle import layout as OL
from oracle import permute as OP
from workloads import get_workload, make_qkv

from helpers import (build_layout, compare, geometry_of, gpu_attention, layout_for_kernel, make_workload,
                     sample_query_tiles, to_f64, tolerances, workload_for_kernel)

pytestmark = pytest.mark.gpu
ABSENT = (-1, -1)
DEV = "cuda:0"


def _say(*a):
    print(*a, flush=True)


def _full_parity(wl, q_gain=1.0, dense=False, scale=0.0):
    g = geometry_of(wl)
    lay = build_layout(ca, wl, scale)
    q, k, v = make_qkv(wl, DEV, q_gain=q_gain)
    out, _ = gpu_attention(ca, wl, lay, q, k, v, dense=dense)
    torch.cuda.synchronize()
    heads = wl.heads
    if dense:
        heads = [[(g.nT - 1, (g.nH - 1, g.nW - 1), ABSENT)]] * wl.num_heads
    want = OA.masked_attention(g, heads, to_f64(q[0]), to_f64(k[0]), to_f64(v[0]), scale if scale > 0 else None)
    return compare(to_f64(out[0]), want, *tolerances(wl.dtype), what=wl.name)


# ---------------------------------------------------------------- permutation (bit-exact)

@pytest.mark.parametrize("case", [
    ("f32", 64, (4, 8, 8), (1, 4, 4), 0),
    ("bf16", 128, (5, 13, 20), (2, 8, 8), 128),      # padded T and H, text tokens
    ("bf16", 64, (3, 9, 17), (1, 8, 8), 64),          # padded H and W
    ("f32", 32, (3, 5, 7), (2, 2, 4), 0),
])
def test_permute_bit_exact_and_roundtrip(case):
    dtype, D, (T, H, W), tile, n_text = case
    _say("permute", case)
    wl = make_workload("perm", T, H, W, tile, n_text, 3, D, dtype, [[(0, (0, 0), ABSENT)]] * 3)
    g = geometry_of(wl)
    lay = build_layout(ca, wl)
    q, _, _ = make_qkv(wl, DEV)
    qp = ca.compact_attn_permute(q, lay)
    back = ca.compact_attn_permute(qp, lay, inverse=True)
    torch.cuda.synchronize()
    view = torch.int16 if dtype == "bf16" else torch.int32
    want = OP.permute(g, q.cpu().view(view).numpy())
    assert np.array_equal(qp.cpu().view(view).numpy(), want)
    assert torch.equal(back, q)


def test_permute_full_size_sampled_planes():
    wl = get_workload("cfg4-S65")
    _say("permute full size", wl.name)
    g = geometry_of(wl)
    lay = build_layout(ca, wl)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(5)
    x = torch.randn(1, wl.num_heads, g.N_real, wl.head_dim, device=DEV, generator=gen).to(torch.bfloat16)
    xp = ca.compact_attn_permute(x, lay)
    back = ca.compact_attn_permute(xp, lay, inverse=True)
    torch.cuda.synchronize()
    assert torch.equal(back, x)
    for h in (0, 11, 23):
        want = OP.permute(g, x[0, h].cpu().view(torch.int16).numpy())
        assert np.array_equal(xp[0, h].cpu().view(torch.int16).numpy(), want)


# ---------------------------------------------------------------- attention, small configs in full

def test_config1_fp32_full_parity():
    _say("cfg1 fp32")
    wl = get_workload("cfg1")
    _say(_full_parity(wl))
    _say(_full_parity(wl, dense=True))


def test_config2_bf16_full_parity():
    _say("cfg2 bf16")
    wl = get_workload("cfg2")
    _say(_full_parity(wl))


def test_config2_dense_equals_dense_softmax():
    _say("cfg2 dense")
    wl = get_workload("cfg2")
    g = geometry_of(wl)
    lay = build_layout(ca, wl)
    q, k, v = make_qkv(wl, DEV)
    out, _ = gpu_attention(ca, wl, lay, q, k, v, dense=True)
    want = OA.dense_attention(to_f64(q[0]), to_f64(k[0]), to_f64(v[0]))
    _say(compare(to_f64(out[0]), want, *tolerances("bf16"), what="cfg2 dense"))


_EDGE_HEADS = [
    [(0, (1, 1), ABSENT), (1, (0, 0), ABSENT)],
    [(2, (0, 2), (1, 0))],
    [(0, ABSENT, ABSENT), (2, (1, 1), ABSENT)],          # skips its own frame
    [],                                                    # keeps text tiles only
]


@pytest.mark.parametrize("shape", [
    ("bf16", 128, (5, 13, 20), (2, 8, 8), 128),           # B=128 D=128, T and H padded, one text tile
    ("bf16", 64, (5, 13, 20), (2, 8, 8), 128),            # B=128 D=64
    ("bf16", 128, (3, 13, 20), (1, 8, 8), 64),            # B=64 D=128
    ("bf16", 64, (3, 13, 20), (1, 8, 8), 64),             # B=64 D=64
    ("f32", 32, (3, 5, 7), (2, 2, 4), 16),                # fp32 kernel, B=16
    ("f32", 128, (2, 9, 9), (1, 8, 8), 0),                # fp32 kernel, B=64, D=128
])
def test_padded_grids_text_and_odd_heads(shape):
    dtype, D, (T, H, W), tile, n_text = shape
    _say("edge grid", shape)
    wl = make_workload("edge", T, H, W, tile, n_text, len(_EDGE_HEADS), D, dtype, _EDGE_HEADS)
    _say(_full_parity(wl))
    _say(_full_parity(wl, q_gain=4.0))                    # peaky softmax: a dropped tile would show
    _say(_full_parity(wl, dense=True))
    _say(_full_parity(wl, scale=0.05))


def test_windows_that_keep_their_size_at_the_border():
    """Heads with clamp_centre set: the layout moves windows inward at the border (checked bit for
    bit on the host); here the kernels run such a layout and match the oracle's rule."""
    from oracle import layout as OLay
    _say("clamped windows")
    heads = [[(0, (1, 1), ABSENT), (1, (0, 0), ABSENT)], [(2, (0, 2), (1, 0))]]
    wl = make_workload("clamped", 5, 29, 40, (2, 8, 8), 128, len(heads), 128, "bf16", heads)
    g = geometry_of(wl)
    lay = ca.compact_attn_build_layout(wl.T, wl.H, wl.W, wl.tile, wl.n_text, 1, len(heads), 128, "bf16", heads,
                                       clamp_centre=[True, True])
    plain = build_layout(ca, wl)
    assert lay.nnz_total > plain.nnz_total                  # border rows gained tiles
    q, k, v = make_qkv(wl, DEV, q_gain=2.0)
    out, _ = gpu_attention(ca, wl, lay, q, k, v)
    torch.cuda.synchronize()
    moved = [OLay.ClampedHead(h) for h in heads]
    want = OA.masked_attention(g, moved, to_f64(q[0]), to_f64(k[0]), to_f64(v[0]))
    _say(compare(to_f64(out[0]), want, *tolerances("bf16"), what="clamped windows"))


def test_no_text_and_empty_rows_give_zeros():
    _say("empty rows")
    heads = [[(0, ABSENT, ABSENT)], [(0, (0, 0), ABSENT)]]
    wl = make_workload("empty", 2, 8, 16, (1, 8, 8), 0, 2, 64, "bf16", heads)
    lay = build_layout(ca, wl)
    q, k, v = make_qkv(wl, DEV)
    out, out_tiled = gpu_attention(ca, wl, lay, q, k, v)
    torch.cuda.synchronize()
    assert torch.all(out[0, 0] == 0)
    assert torch.any(out[0, 1] != 0)


# ---------------------------------------------------------------- mask probes (closed forms)

@pytest.mark.parametrize("shape", [("bf16", 128, (2, 8, 8)), ("bf16", 64, (1, 8, 8)), ("f32", 64, (1, 4, 4))])
def test_zero_query_tile_indicator_probe(shape):
    """Q = 0 makes the softmax uniform, so the output is the share of allowed real keys per
    value class; with V = indicator of (tile mod D) this pins the tile list the kernel walked
    and its handling of padding keys, free of any tolerance on the scores."""
    dtype, D, tile = shape
    _say("probe", shape)
    T, H, W = 5, 13, 20
    B = tile[0] * tile[1] * tile[2]
    heads = [[(0, (1, 1), ABSENT), (2, (0, 0), ABSENT)], [(1, (0, 2), (1, 0))], [(4, (1, 2), ABSENT)]]
    wl = make_workload("probe", T, H, W, tile, B, len(heads), D, dtype, heads)
    g = geometry_of(wl)
    lay = build_layout(ca, wl)
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    tok_tile, _ = g.token_tile_and_slot()
    q = torch.zeros(1, len(heads), g.N_real, D, dtype=tdt, device=DEV)
    k = torch.randn(1, len(heads), g.N_real, D, device=DEV).to(tdt)
    v_np = np.zeros((g.N_real, D), dtype=np.float32)
    v_np[np.arange(g.N_real), tok_tile % D] = 1.0
    v = torch.from_numpy(v_np).to(DEV).to(tdt)[None, None].expand(1, len(heads), -1, -1).contiguous()
    out, _ = gpu_attention(ca, wl, lay, q, k, v)
    got = to_f64(out[0])
    real_per_tile = np.bincount(tok_tile, minlength=g.n).astype(float)
    for h, head in enumerate(heads):
        for q_tile in range(g.n):
            kept = OL.kept_tiles(g, head, q_tile)
            want = np.zeros(D)
            np.add.at(want, kept % D, real_per_tile[kept])
            want /= real_per_tile[kept].sum()
            idx = np.nonzero(tok_tile == q_tile)[0]
            err = np.abs(got[h, idx] - want[None]).max()
            assert err < (6e-3 if dtype == "bf16" else 1e-5), (h, q_tile, err)


# ---------------------------------------------------------------- full-size configs, sampled rows

def _sampled_parity(name, heads_to_check, dense=False):
    wl = get_workload(name)
    g = geometry_of(wl)
    lay = build_layout(ca, wl)
    q, k, v = make_qkv(wl, DEV)
    out, _ = gpu_attention(ca, wl, lay, q, k, v, dense=dense)
    torch.cuda.synchronize()
    if not dense:       # the same at full size with the gather / scatter inside the kernel: every bit equal
        fused = ca.compact_attn_forward_natural(q, k, v, lay)
        torch.cuda.synchronize()
        assert torch.equal(fused, out), f"{name}: natural-order forward differs from the permuted path"
        del fused
    counts = OL.row_counts(g, wl.heads)
    tok_tile, _ = g.token_tile_and_slot()
    rng = np.random.default_rng(2508)
    worst = (0.0, 0.0)
    full = [(g.nT - 1, (g.nH - 1, g.nW - 1), ABSENT)]
    for h in heads_to_check:
        qh, kh, vh = to_f64(q[0, h]), to_f64(k[0, h]), to_f64(v[0, h])
        oh = to_f64(out[0, h])
        tiles = sample_query_tiles(g, counts[h], rng, extra=2)
        for q_tile in tiles:
            idx, want = OA.attention_tile(g, full if dense else wl.heads[h], q_tile, qh, kh, vh, token_tile=tok_tile)
            mx, mean = compare(oh[idx], want, *tolerances(wl.dtype), what=f"{name} head {h} tile {q_tile}")
            worst = (max(worst[0], mx), max(worst[1], mean))
        _say(name, "head", h, "tiles", tiles, "worst", worst)
    return worst


def test_config3_sampled_rows():
    _say("cfg3 sampled")
    _sampled_parity("cfg3", [0, 4, 6, 15, 29])


def test_config4_sampled_rows():
    _say("cfg4-S65 sampled")
    _sampled_parity("cfg4-S65", [0, 1, 4, 15, 18])


def test_config4_dense_sampled_rows():
    _say("cfg4 dense sampled (heads restricted to keep the run short)")
    wl = get_workload("cfg4-S80")
    small = make_workload("cfg4-dense", wl.T, wl.H, wl.W, wl.tile, wl.n_text, 2, wl.head_dim, wl.dtype, wl.heads[:2], cfg=4)
    g = geometry_of(small)
    lay = build_layout(ca, small)
    q, k, v = make_qkv(small, DEV)
    out, _ = gpu_attention(ca, small, lay, q, k, v, dense=True)
    tok_tile, _ = g.token_tile_and_slot()
    full = [(g.nT - 1, (g.nH - 1, g.nW - 1), ABSENT)]
    qh, kh, vh, oh = (to_f64(t[0, 1]) for t in (q, k, v, out))
    for q_tile in (0, 511, g.n_vid - 1, g.n - 1):
        idx, want = OA.attention_tile(g, full, q_tile, qh, kh, vh, token_tile=tok_tile)
        _say(q_tile, compare(oh[idx], want, *tolerances("bf16"), what=f"dense tile {q_tile}"))


def test_config5_sampled_rows():
    _say("cfg5 sampled")
    _sampled_parity("cfg5", [4, 6, 13, 17])


def test_config4_sparsity50_sampled_rows():
    _say("cfg4-S50 sampled")
    _sampled_parity("cfg4-S50", [0, 4, 9, 15, 21])          # cross, local, global + local tail, wide local, thick cross


def test_config4_sparsity80_sampled_rows():
    _say("cfg4-S80 sampled")
    _sampled_parity("cfg4-S80", [6, 11, 13, 17, 19])        # G/4/6, G/0/2, C0/0/2, full, L2/2/3


# ---------------------------------------------------------------- full-size configs, every row (closed form)

@pytest.mark.parametrize("name", ["cfg3", "cfg4-S50", "cfg4-S65", "cfg4-S80", "cfg5"])
def test_every_row_at_full_size_zero_query_probe(name):
    """Every real query row of every head at the benchmark sizes, sparse and dense, in the launch
    configuration the benchmark times.  Q = 0 makes the softmax uniform over exactly the kept real
    keys (Appendix D: softmax over the kept blocks; Sec. 4.1: the keep rule), so with V = indicator of
    (key tile mod D) the output row is the kept real-token count per class over the total: a closed
    form from the oracle's tile mask alone, which pins the walked tile list, the padding-key
    masking, the launch-order remapping and its remainder, and the paired walk at scale."""
    wl = get_workload(name)
    _say("all rows", name)
    g = geometry_of(wl)
    D = wl.head_dim
    lay = build_layout(ca, wl)
    tok_tile = g.token_slots() // g.B                       # natural order -> tile id
    real_per_tile = np.bincount(tok_tile, minlength=g.n).astype(np.float64)
    onehot = np.zeros((g.n, D))
    onehot[np.arange(g.n), np.arange(g.n) % D] = real_per_tile
    tile_dev = torch.from_numpy(tok_tile).to(DEV)
    q = torch.zeros(1, wl.num_heads, g.N_real, D, dtype=torch.bfloat16, device=DEV)
    gen = torch.Generator(device=DEV)
    gen.manual_seed(11)
    k = torch.randn(1, wl.num_heads, g.N_real, D, device=DEV, generator=gen).to(torch.bfloat16)
    v1 = torch.zeros(g.N_real, D, dtype=torch.bfloat16, device=DEV)
    v1[torch.arange(g.N_real, device=DEV), tile_dev % D] = 1.0
    v = v1[None, None].expand(1, wl.num_heads, -1, -1).contiguous()
    del v1
    out, _ = gpu_attention(ca, wl, lay, q, k, v)
    dense, _ = gpu_attention(ca, wl, lay, q, k, v, dense=True)
    torch.cuda.synchronize()
    del q, k, v
    want_dense = torch.from_numpy(onehot.sum(axis=0) / real_per_tile.sum()).to(DEV).float()
    worst = 0.0
    for h in range(wl.num_heads):
        mask = OL.keep_mask(g, wl.heads[h]).astype(np.float64)
        want = (mask @ onehot) / (mask @ real_per_tile)[:, None]            # [n, D] per query tile
        want_rows = torch.from_numpy(want).to(DEV).float()[tile_dev]         # [N_real, D]
        err = (out[0, h].float() - want_rows).abs().max().item()
        err_d = (dense[0, h].float() - want_dense[None]).abs().max().item()
        worst = max(worst, err, err_d)
        assert err < 6e-3 and err_d < 6e-3, (name, h, err, err_d)
    _say(name, "worst abs err over all rows", worst)


# ---------------------------------------------------------------- dynamically drawn tail of a launch

@pytest.mark.parametrize("D,tile,T,Hd,batch", [(64, (1, 8, 8), 8, 8, 1), (128, (1, 8, 8), 6, 24, 1), (128, (2, 8, 8), 6, 22, 2)])
def test_dynamic_tail_of_the_launch_order(D, tile, T, Hd, batch):
    """Launches of 4096 entries and more hand the cheapest entries out by ticket instead of by
    workgroup id (rows here; pairs of rows for 64-token tiles with head dim 128).  Every row must
    still be computed exactly once per launch: checked against the closed form of the Q = 0 probe on
    every row, on 70 launches in a row (more than the layout has ticket counters, and every launch
    must leave its counter at zero), on the dense walk, on the natural-order variant and on replays
    of a captured graph."""
    import dataclasses
    _say("dynamic tail", D, tile, T, Hd, batch)
    H = W = 64
    rng = np.random.default_rng(3)
    heads = [[(int(rng.integers(0, 3)), (int(rng.integers(0, 4)), int(rng.integers(0, 4))), ABSENT)] for _ in range(Hd)]
    heads[1] = [(T, (99, 99), ABSENT)]                                       # one global head: long rows first
    wl = dataclasses.replace(make_workload("tail", T, H, W, tile, 0, Hd, D, "bf16", heads), batch=batch)
    g = geometry_of(wl)
    assert Hd * g.n >= 4096
    lay = build_layout(ca, wl)
    tok_tile = g.token_slots() // g.B
    per_tile = np.bincount(tok_tile, minlength=g.n).astype(np.float64)
    onehot = np.zeros((g.n, D))
    onehot[np.arange(g.n), np.arange(g.n) % D] = per_tile
    tile_dev = torch.from_numpy(tok_tile).to(DEV)
    q = torch.zeros(batch, Hd, g.N_real, D, dtype=torch.bfloat16, device=DEV)
    k = torch.randn(batch, Hd, g.N_real, D, device=DEV).to(torch.bfloat16)
    v1 = torch.zeros(g.N_real, D, dtype=torch.bfloat16, device=DEV)
    v1[torch.arange(g.N_real, device=DEV), tile_dev % D] = 1.0
    v = v1[None, None].expand(batch, Hd, -1, -1).contiguous()
    qp, kp, vp = (ca.compact_attn_permute(t, lay) for t in (q, k, v))
    first = ca.compact_attn_forward(qp, kp, vp, lay)
    out = ca.compact_attn_permute(first, lay, inverse=True)
    dense = ca.compact_attn_permute(ca.compact_attn_dense(qp, kp, vp, lay), lay, inverse=True)
    torch.cuda.synchronize()
    want_dense = torch.from_numpy(onehot.sum(axis=0) / per_tile.sum()).to(DEV).float()
    for h in range(Hd):
        mask = OL.keep_mask(g, wl.heads[h]).astype(np.float64)
        want = torch.from_numpy((mask @ onehot) / (mask @ per_tile)[:, None]).to(DEV).float()[tile_dev]
        for b in range(batch):
            assert (out[b, h].float() - want).abs().max().item() < 6e-3, (h, b)
            assert (dense[b, h].float() - want_dense[None]).abs().max().item() < 6e-3, (h, b)
    if tile[2] % (4 if D == 128 else 8) == 0:
        assert torch.equal(ca.compact_attn_forward_natural(q, k, v, lay), out)
    again = torch.empty_like(first)
    for rep in range(70):
        again.fill_(float("nan"))
        ca.compact_attn_forward(qp, kp, vp, lay, out=again)
        assert torch.equal(again, first), f"launch {rep}"
    for rep in range(3):                                                    # the allocation-free entry point keeps
        again.fill_(float("nan"))                                          # its one ticket counter in the fixed array
        try:
            ca.compact_attn_forward_static(qp, kp, vp, lay, out=again)
        except ca.CompactAttnError as exc:
            assert exc.status == -2                                         # tables beyond the array: refused, fine
            break
        assert torch.equal(again, first), f"static launch {rep}"
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        ca.compact_attn_forward(qp, kp, vp, lay, out=again)
    for rep in range(3):
        again.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(again, first), f"replay {rep}"
        ca.compact_attn_forward(qp, kp, vp, lay)                           # eager launches between replays


# ---------------------------------------------------------------- exponent reference moves

@pytest.mark.parametrize("shape", [("bf16", 128, (2, 8, 8)), ("bf16", 128, (1, 8, 8)), ("bf16", 64, (2, 8, 8))])
def test_rising_and_huge_scores(shape):
    """Scores that keep rising along the key-tile walk force the kernel to move its exponent
    reference again and again (rescaling the output tile each time); scores hundreds of units
    apart must neither overflow nor lose the small terms' normalisation.  The oracle's softmax
    subtracts the exact row maximum, so it is immune to both."""
    dtype, D, tile = shape
    _say("rising scores", shape)
    T, H, W = 6, 16, 16
    B = tile[0] * tile[1] * tile[2]
    heads = [[(T, (1, 1), ABSENT)], [(T, (9, 9), ABSENT)]]
    wl = make_workload("rising", T, H, W, tile, B, len(heads), D, dtype, heads)
    g = geometry_of(wl)
    lay = build_layout(ca, wl)
    q, k, v = make_qkv(wl, DEV)
    # keys grow with their position in tile order, so later tiles of every row score higher
    tok_tile, _ = g.token_tile_and_slot()
    ramp = torch.tensor(np.asarray(tok_tile), device=DEV, dtype=torch.float32) / g.n
    for gain, what in ((1.0, "rising"), (40.0, "huge")):
        kk = (k.float() * (1.0 + 3.0 * gain * ramp[None, None, :, None])).to(k.dtype)
        qq = (q.float() * (2.0 if gain == 1.0 else 6.0)).to(q.dtype)
        out, _ = gpu_attention(ca, wl, lay, qq, kk, v)
        torch.cuda.synchronize()
        want = OA.masked_attention(g, heads, to_f64(qq[0]), to_f64(kk[0]), to_f64(v[0]), None)
        _say(what, compare(to_f64(out[0]), want, *tolerances(dtype), what=what))


# ---------------------------------------------------------------- imported and merged masks

@pytest.mark.parametrize("shape", [("bf16", 128, (2, 8, 8)), ("bf16", 128, (1, 8, 8)), ("f32", 64, (1, 4, 4))])
def test_imported_random_mask_and_union(shape):
    """An arbitrary tile mask given as CSR, and the union of two layouts, run through the same
    kernels and match the oracle's definition evaluated on the boolean masks."""
    dtype, D, tile = shape
    _say("imported mask", shape)
    T, H, W = 5, 13, 20
    B = tile[0] * tile[1] * tile[2]
    Hd = 3
    wl = make_workload("import", T, H, W, tile, B, Hd, D, dtype, [[]] * Hd)
    g = geometry_of(wl)
    rng = np.random.default_rng(5)
    masks = rng.random((Hd, g.n, g.n)) < 0.25
    masks[0, 3] = False                                   # an empty row gives zeros
    masks[1, :, g.n - 1] = True
    masks[2, :6] = False                                  # whole pairs of neighbouring rows empty,
    masks[2, 7] = True                                    # a full row next to sparse ones
    lay = ca.compact_attn_layout_from_csr(T, H, W, tile, B, 1, Hd, D, dtype, [OL.csr_of_mask(m) for m in masks])
    q, k, v = make_qkv(wl, DEV)
    out, _ = gpu_attention(ca, wl, lay, q, k, v)
    torch.cuda.synchronize()
    want = OA.tile_mask_attention(g, masks, to_f64(q[0]), to_f64(k[0]), to_f64(v[0]))
    _say(compare(to_f64(out[0]), want, *tolerances(dtype), what="imported mask"))
    other = rng.random((Hd, g.n, g.n)) < 0.1
    lay_b = ca.compact_attn_layout_from_csr(T, H, W, tile, B, 1, Hd, D, dtype, [OL.csr_of_mask(m) for m in other])
    merged = ca.compact_attn_layout_union(lay, lay_b)
    out, _ = gpu_attention(ca, wl, merged, q, k, v)
    torch.cuda.synchronize()
    want = OA.tile_mask_attention(g, OL.union_masks(masks, other), to_f64(q[0]), to_f64(k[0]), to_f64(v[0]))
    _say(compare(to_f64(out[0]), want, *tolerances(dtype), what="merged mask"))


@pytest.mark.parametrize("tile,D,dtype", [((1, 4, 4), 32, "f32"), ((1, 8, 8), 64, "f32"), ((2, 8, 8), 64, "bf16")])
@pytest.mark.parametrize("heads", [127, 128, 129, 255, 1023, 1024])
def test_launches_of_few_rounds(heads, tile, D, dtype):
    """Launches around 512 and 4096 rows, where the order of the fp32 kernels' workgroups changes: every row of every head.  The bf16 ones
    run the one-tile kernel, whose order does not, all but those of 129 heads; ways-4x4 has a test of its own."""
    _say("few rounds", heads, tile, D, dtype)
    wl = make_workload("rounds", tile[0], 2 * tile[1], 2 * tile[2] - 1, tile, 0, heads, D, dtype, [[]] * heads)
    lay = build_layout(ca, wl)
    q, k, v = make_qkv(wl, DEV)
    out = ca.compact_attn_permute(ca.compact_attn_dense(*(ca.compact_attn_permute(x, lay) for x in (q, k, v)), lay), lay, inverse=True)
    s = q[0].double().cpu() @ k[0].double().cpu().transpose(1, 2) * D ** -0.5
    err = (out[0].double().cpu() - torch.softmax(s, dim=2) @ v[0].double().cpu()).abs().max().item()
    assert err <= (1e-4 if dtype == "f32" else 2e-2)      # the bounds of the other forward tests


@pytest.mark.parametrize("rows,D,tile,grid,heads", [
    (508, 128, (2, 8, 8), (7, 4, 4), 127),
    (512, 128, (4, 4, 8), (4, 5, 9), 128),
    (513, 64, (2, 8, 8), (6, 8, 1), 171),
    (4095, 64, (2, 8, 8), (1, 4, 20), 1365),
    (4096, 128, (4, 4, 8), (14, 1, 8), 1024),
    (4100, 128, (4, 4, 8), (5, 5, 1), 1025),
])
def test_launches_of_few_rounds_of_the_four_wave_kernel(rows, D, tile, grid, heads):
    """ways-4x4 on both sides of 512 and 4096 workgroups, sparse, where rows differ in length and are taken from the order table, and dense:
    every row of every head."""
    _say("few rounds of ways-4x4", rows, D, tile, grid, heads)
    cycle = [_GLOBAL, [(0, (0, 1), ABSENT)], [(1, (1, 0), ABSENT)], _GLOBAL]
    wl = make_workload("rounds", *grid, tile, 0, heads, D, "bf16", [cycle[h % 4] for h in range(heads)])
    lay = build_layout(ca, wl)
    assert lay.n_tiles * heads == rows
    q, k, v = make_qkv(wl, DEV)
    tile_of = torch.from_numpy(np.asarray(geometry_of(wl).token_tile_and_slot()[0]))
    keep = torch.zeros(4, lay.n_tiles, lay.n_tiles, dtype=torch.bool)
    for h in range(4):                                        # the table itself is compared with the oracle elsewhere
        row_ptr, col_idx = ca.compact_attn_layout_csr(lay, h)
        for r in range(lay.n_tiles):
            keep[h, r, torch.from_numpy(np.asarray(col_idx[row_ptr[r]:row_ptr[r + 1]]).astype(np.int64))] = True
    seen = keep[:, tile_of][:, :, tile_of].to(DEV)
    s = (q[0].double() @ k[0].double().transpose(1, 2).contiguous()) * D ** -0.5
    x = [ca.compact_attn_permute(t, lay) for t in (q, k, v)]
    for dense in (False, True):
        assert ca.compact_attn_layout_kernel(lay, dense=dense) == "ways-4x4" and ca.compact_attn_layout_split(lay, dense=dense) == (0, None)
        out = ca.compact_attn_permute((ca.compact_attn_dense if dense else ca.compact_attn_forward)(*x, lay), lay, inverse=True)
        masked = s if dense else s.masked_fill(~seen[torch.arange(heads, device=DEV) % 4], -math.inf)
        err = (out[0].double() - torch.softmax(masked, dim=2) @ v[0].double()).abs().max().item()
        assert err <= 2e-2, dense                             # the bound of the other forward tests


# ---------------------------------------------------------------- attention mass per tile pair

MASS_ABS = 2e-4      # per tile pair, in units of "query tokens": a pair sums up to 128*128 probabilities in
                     # fp32 from fp32 scores of the same bf16 inputs; exp2 and the sums carry ~1e-6 relative
                     # error on masses of O(10), measured 1e-6 .. 1.2e-5


@pytest.mark.parametrize("shape", [(128, (2, 8, 8), 5, 13, 20, 128), (64, (2, 8, 8), 4, 16, 16, 0),
                                   (128, (1, 8, 8), 3, 13, 20, 64), (64, (1, 8, 8), 2, 16, 24, 0)])
def test_tile_mass_matches_the_definition(shape):
    from oracle import search as OS
    D, tile, T, H, W, n_text = shape
    _say("tile mass", shape)
    Hd = 2
    wl = make_workload("mass", T, H, W, tile, n_text, Hd, D, "bf16", [[]] * Hd)
    g = geometry_of(wl)
    lay = build_layout(ca, wl)
    for gain in (1.0, 3.0):
        q, k, _ = make_qkv(wl, DEV, q_gain=gain)
        qp, kp = ca.compact_attn_permute(q, lay), ca.compact_attn_permute(k, lay)
        mass = ca.compact_attn_tile_mass(qp, kp, lay)
        again = ca.compact_attn_tile_mass(qp, kp, lay)
        torch.cuda.synchronize()
        assert torch.equal(mass, again)                              # fixed summation order
        got = mass[0].double().cpu().numpy()
        tok_tile, _ = g.token_tile_and_slot()
        pop = np.bincount(tok_tile, minlength=g.n)
        assert np.allclose(got.sum(axis=2), pop[None, :].repeat(Hd, 0), atol=1e-2)   # rows sum to tile populations
        for h in range(Hd):
            want = OS.tile_mass(g, to_f64(q[0, h]), to_f64(k[0, h]))
            err = np.abs(got[h] - want)
            _say("head", h, "gain", gain, "max err", err.max(), "max mass", want.max())
            assert err.max() <= MASS_ABS


@pytest.mark.parametrize("shape", [(128, (2, 8, 8)), (64, (1, 8, 8))])
def test_tile_mass_with_a_moving_exponent_reference(shape):
    """Scores that keep rising along the key-tile walk move the kernel's exponent reference again
    and again after sums have been stored against earlier references; scores hundreds of units apart
    push the early sums below fp32 range relative to the final reference.  The definition subtracts
    the exact row maximum and knows neither."""
    from oracle import search as OS
    D, tile = shape
    _say("tile mass, rising scores", shape)
    T, H, W = 6, 16, 16
    B = tile[0] * tile[1] * tile[2]
    wl = make_workload("massrise", T, H, W, tile, B, 2, D, "bf16", [[]] * 2)
    g = geometry_of(wl)
    lay = build_layout(ca, wl)
    q, k, _ = make_qkv(wl, DEV)
    tok_tile, _ = g.token_tile_and_slot()
    pop = np.bincount(tok_tile, minlength=g.n)
    ramp = torch.tensor(np.asarray(tok_tile), device=DEV, dtype=torch.float32) / g.n
    for gain, what in ((1.0, "rising"), (40.0, "huge")):
        kk = (k.float() * (1.0 + 3.0 * gain * ramp[None, None, :, None])).to(k.dtype)
        qq = (q.float() * (2.0 if gain == 1.0 else 6.0)).to(q.dtype)
        mass = ca.compact_attn_tile_mass(ca.compact_attn_permute(qq, lay), ca.compact_attn_permute(kk, lay), lay)
        torch.cuda.synchronize()
        got = mass[0].double().cpu().numpy()
        assert np.isfinite(got).all()
        assert np.allclose(got.sum(axis=2), pop[None, :].repeat(2, 0), atol=1e-2)
        for h in range(2):
            want = OS.tile_mass(g, to_f64(qq[0, h]), to_f64(kk[0, h]))
            err = np.abs(got[h] - want)
            _say(what, "head", h, "max err", err.max(), "max mass", want.max())
            assert err.max() <= MASS_ABS


@pytest.mark.parametrize("D,tile", [(128, (2, 8, 8)), (64, (2, 8, 8)), (128, (1, 8, 8)), (64, (1, 8, 8))])
def test_tile_mass_of_scores_far_below_zero(D, tile):
    """A constant added to all scores of a query changes no mass: with every score near -150 (scaled) the masses are
    those of the definition, as they are near zero.  The products carry the rounding of sums of that size, 2^11 in raw
    units: D / 16 roundings to 2^-13 at most, below 1e-3 in raw units, 1e-4 relative in a probability."""
    from oracle import search as OS
    _say("far below zero", D, tile)
    B = tile[0] * tile[1] * tile[2]
    wl = make_workload("mass-low", 3, 13, 20, tile, B, 2, D, "bf16", [[]] * 2)
    g = geometry_of(wl)
    lay = build_layout(ca, wl)
    q, k, _ = make_qkv(wl, DEV)
    q[..., 0] = 32.0
    k[..., 0] = -150.0 * D ** 0.5 / 32.0
    mass = ca.compact_attn_tile_mass(ca.compact_attn_permute(q, lay), ca.compact_attn_permute(k, lay), lay)
    for h in range(2):
        want = OS.tile_mass(g, to_f64(q[0, h]), to_f64(k[0, h]))
        assert np.abs(mass[0, h].double().cpu().numpy() - want).max() <= MASS_ABS + 1e-4 * want.max()


@pytest.mark.parametrize("T,Hd", [(5, 2), (60, 24)])
@pytest.mark.parametrize("tokens", [1, 15, 16, 17, 31, 32, 33, 63, 64, 65, 95, 96, 97, 127])
@pytest.mark.parametrize("D", [64, 128])
def test_tile_mass_of_padded_tiles(D, tokens, T, Hd):
    """Every second tile of 128 holds `tokens` tokens: up to 96 its tokens are brought to the front and whole blocks of 32 keys left
    out.  Few rows, whose key tiles are shared by workgroups, and enough for one workgroup each; padding rows of K hold NaN."""
    from oracle import search as OS
    _say("tile mass, padded tiles", D, tokens, T, Hd)
    wl = make_workload("masspad", T, 1, 128 + tokens, (1, 1, 128), 0, Hd, D, "bf16", [[]] * Hd)
    g = geometry_of(wl)
    lay = build_layout(ca, wl)
    q, k, _ = make_qkv(wl, DEV, q_gain=2.0)
    qp, kp = ca.compact_attn_permute(q, lay), ca.compact_attn_permute(k, lay)
    tok_tile, tok_slot = (np.asarray(x) for x in g.token_tile_and_slot())
    padding = torch.ones(g.n * 128, dtype=torch.bool, device=DEV)
    padding[torch.from_numpy(tok_tile * 128 + tok_slot).to(DEV)] = False
    kp[:, :, padding] = float("nan")
    mass = ca.compact_attn_tile_mass(qp, kp, lay)
    assert torch.equal(mass, ca.compact_attn_tile_mass(qp, kp, lay))
    got = mass[0].double().cpu().numpy()
    assert np.allclose(got.sum(axis=2), np.bincount(tok_tile, minlength=g.n)[None, :].repeat(Hd, 0), atol=1e-2)
    for h in (0, Hd - 1):
        want = OS.tile_mass(g, to_f64(q[0, h]), to_f64(k[0, h]))
        assert np.abs(got[h] - want).max() <= MASS_ABS


@pytest.mark.parametrize("D,tile", [(64, (1, 8, 8)), (128, (1, 8, 8)), (64, (2, 8, 8)), (128, (2, 8, 8))])
def test_tile_mass_with_more_rows_than_workgroups(D, tile):
    """More groups of 128 queries than the launch has workgroups (two or three per compute unit), so
    workgroups take a second group by ticket and reuse their block of the workspace and their tables in
    LDS: heads of both batch entries are compared with the definition, among them one that only second
    and later tickets can reach, and all rows with their closed-form sums."""
    import dataclasses
    from oracle import search as OS
    _say("tile mass, more rows than workgroups", D, tile)
    T, H, W, Hd, batch = 6, 32, 32, 12, 2
    B = tile[0] * tile[1] * tile[2]
    wl = dataclasses.replace(make_workload("masslaunch", T, H, W, tile, 0, Hd, D, "bf16", [[]] * Hd), batch=batch)
    g = geometry_of(wl)
    groups = -(-g.n * B // 128)                                        # per head
    workgroups = torch.cuda.get_device_properties(0).multi_processor_count * (2 if (B, D) == (128, 128) else 3)
    late = -(-workgroups // groups)                                    # (batch, head) whose groups all come after the first round
    assert late + 1 < batch * Hd
    lay = build_layout(ca, wl)
    q, k, _ = make_qkv(wl, DEV, q_gain=2.0)
    mass = ca.compact_attn_tile_mass(ca.compact_attn_permute(q, lay), ca.compact_attn_permute(k, lay), lay)
    torch.cuda.synchronize()
    got = mass.double().cpu().numpy()
    assert np.allclose(got.sum(axis=3), float(B), atol=1e-2)           # every slot holds a token
    for b, h in ((0, 0), divmod(late, Hd), (batch - 1, Hd - 1)):
        want = OS.tile_mass(g, to_f64(q[b, h]), to_f64(k[b, h]))
        err = np.abs(got[b, h] - want)
        _say("batch", b, "head", h, "max err", err.max())
        assert err.max() <= MASS_ABS


@pytest.mark.parametrize("D,tile,T,H,W,n_text,Hd,batch,shares", [
    (64, (1, 8, 8), 5, 30, 52, 64, 1, 1, 4),      # 141 tiles in 71 steps, the last of one tile
    (64, (1, 8, 8), 2, 25, 40, 0, 3, 2, 1),       # 40 tiles, 20 steps and 120 groups: not split
    (64, (1, 8, 8), 4, 8, 64, 0, 2, 1, 4),        # 32 tiles, 16 steps: the shortest walk that is split
    (128, (1, 8, 8), 3, 20, 27, 0, 2, 1, 4),      # steps of one 64-token tile
    (64, (2, 8, 8), 11, 13, 20, 128, 2, 2, 4),
    (128, (2, 8, 8), 9, 26, 20, 0, 6, 2, 4),      # 720 groups, more than run at a time
])
def test_tile_mass_of_few_rows(D, tile, T, H, W, n_text, Hd, batch, shares):
    """Launches that leave compute units without work split the key tiles of a row group over several workgroups:
    the masses are the definition's, the same on every call, and keys whose scores are minus infinity or far below all others
    (more of them than a share has) change nothing but their own masses."""
    import dataclasses
    from oracle import search as OS
    _say("tile mass, few rows", D, tile, T, H, W, n_text, Hd, batch)
    B = tile[0] * tile[1] * tile[2]
    wl = dataclasses.replace(make_workload("massfew", T, H, W, tile, n_text, Hd, D, "bf16", [[]] * Hd), batch=batch)
    g = geometry_of(wl)
    lay = build_layout(ca, wl)
    q, k, _ = make_qkv(wl, DEV, q_gain=2.0)
    for hidden in (False, True):
        if hidden:
            q[..., 0] = 1.0
            tile_of = torch.from_numpy(np.asarray(g.token_tile_and_slot()[0])).to(DEV)
            gone = tile_of < g.n // 2 + 1
            # padding queries are zero, and zero times an infinity is not: the infinity where there are none
            k[:, :, gone, 0] = float("-inf") if g.n * B == g.N_real else -4096.0
        qp, kp = ca.compact_attn_permute(q, lay), ca.compact_attn_permute(k, lay)
        mass = ca.compact_attn_tile_mass(qp, kp, lay)
        assert ca.compact_attn_layout_mass_shares(lay) == shares
        for _ in range(3):
            assert torch.equal(mass, ca.compact_attn_tile_mass(qp, kp, lay))
        replayed = torch.empty_like(mass)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            ca.compact_attn_tile_mass(qp, kp, lay, out=replayed)
        for _ in range(3):
            replayed.zero_()
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(mass, replayed)
        got = mass.double().cpu().numpy()
        for b in range(batch):
            for h in range(Hd):
                if not hidden:
                    want = OS.tile_mass(g, to_f64(q[b, h]), to_f64(k[b, h]))
                else:
                    p = torch.softmax(q[b, h].double() @ k[b, h].double().t() / D ** 0.5, dim=1)
                    want = torch.zeros(g.n, g.n, dtype=torch.float64, device=DEV)
                    cols = torch.zeros(p.shape[0], g.n, dtype=torch.float64, device=DEV).index_add_(1, tile_of, p)
                    want = want.index_add_(0, tile_of, cols).cpu().numpy()
                    assert (got[b, h][:, :g.n // 2 + 1] == 0).all()
                err = np.abs(got[b, h] - want)
                _say("hidden", hidden, "batch", b, "head", h, "max err", err.max())
                assert err.max() <= MASS_ABS


# grids without padding: a padding query is zero, and zero times an infinity is not
_MASS_WITHOUT_PADDING = [
    (64, (1, 8, 8), 5, 32, 56, 64, 1, 1, 4),
    (64, (1, 8, 8), 4, 8, 64, 0, 2, 1, 4),
    (128, (1, 8, 8), 3, 24, 32, 0, 2, 1, 4),
    (64, (2, 8, 8), 12, 16, 24, 128, 2, 2, 4),
    (128, (2, 8, 8), 10, 24, 24, 0, 6, 2, 4),
    # a workgroup takes all key tiles of a group of queries
    (64, (1, 8, 8), 2, 24, 40, 0, 3, 2, 1),
    (128, (1, 8, 8), 2, 16, 24, 0, 2, 1, 1),
    (64, (2, 8, 8), 4, 16, 24, 128, 2, 1, 1),
    (128, (2, 8, 8), 6, 16, 24, 0, 2, 1, 1),
]


@pytest.mark.parametrize("hidden", ["a half of the tiles", "two of three tiles"])
@pytest.mark.parametrize("D,tile,T,H,W,n_text,Hd,batch,shares", _MASS_WITHOUT_PADDING)
def test_tile_mass_beside_minus_infinite_scores(D, tile, T, H, W, n_text, Hd, batch, shares, hidden):
    """Keys whose scores are minus infinity have no mass, and those beside them keep theirs however far below zero they lie (-512
    scaled here: exp2 of such a score against a reference of zero is zero), whether such keys fill the first tiles of a walk, all
    that a workgroup walks, or only its first tiles.  Rounding: as for scores far below zero, with sums of 2^13 in raw units at head
    dim 128, in the tiles that are multiplied before there is a reference: 4e-4 relative in a probability."""
    import dataclasses
    _say("tile mass beside minus infinity", D, tile, T, H, W, n_text, Hd, batch, hidden)
    wl = dataclasses.replace(make_workload("massinf", T, H, W, tile, n_text, Hd, D, "bf16", [[]] * Hd), batch=batch)
    g = geometry_of(wl)
    assert g.n * tile[0] * tile[1] * tile[2] == g.N_real
    lay = build_layout(ca, wl)
    q, k, _ = make_qkv(wl, DEV)
    tile_of = torch.from_numpy(np.asarray(g.token_tile_and_slot()[0])).to(DEV)
    gone = torch.arange(g.n, device=DEV) < g.n // 2 + 1 if hidden == "a half of the tiles" else torch.arange(g.n, device=DEV) % 3 != 2
    q[..., 0] = 16.0
    k[..., 0] = -32.0 * D ** 0.5
    k[:, :, gone[tile_of], 0] = float("-inf")
    mass = ca.compact_attn_tile_mass(ca.compact_attn_permute(q, lay), ca.compact_attn_permute(k, lay), lay)
    assert ca.compact_attn_layout_mass_shares(lay) == shares
    for b in range(batch):
        for h in range(Hd):
            p = torch.softmax(q[b, h].double() @ k[b, h].double().t() / D ** 0.5, dim=1)
            cols = torch.zeros(p.shape[0], g.n, dtype=torch.float64, device=DEV).index_add_(1, tile_of, p)
            want = torch.zeros(g.n, g.n, dtype=torch.float64, device=DEV).index_add_(0, tile_of, cols)
            assert (mass[b, h][:, gone] == 0).all()
            err = (mass[b, h].double() - want).abs().max().item()
            _say("batch", b, "head", h, "max err", err, "max mass", want.max().item())
            assert err <= MASS_ABS + 4e-4 * want.max().item()


@pytest.mark.parametrize("D,tile,T,H,W,n_text,Hd,batch,shares", _MASS_WITHOUT_PADDING)
def test_tile_mass_of_scores_without_a_softmax(D, tile, T, H, W, n_text, Hd, batch, shares):
    """A score of infinity and a NaN leave a query no softmax.  Where the kernel shows it does not depend on how the key tiles are
    dealt out: infinity from its key tile on, with zeros before, a tile of NaN everywhere, a single NaN in its own tile.
    The masses of other queries stay as they are, bit for bit."""
    import dataclasses
    _say("tile mass without a softmax", D, tile, T, H, W, n_text, Hd, batch)
    wl = dataclasses.replace(make_workload("massnan", T, H, W, tile, n_text, Hd, D, "bf16", [[]] * Hd), batch=batch)
    g = geometry_of(wl)
    assert g.n * tile[0] * tile[1] * tile[2] == g.N_real
    lay = build_layout(ca, wl)
    q, k, _ = make_qkv(wl, DEV)
    tile_of = torch.from_numpy(np.asarray(g.token_tile_and_slot()[0])).to(DEV)
    row, col = g.n // 2, 2 * g.n // 3            # tile of the infinite score's query, and of its key
    q[..., 0] = -1.0
    key = int(torch.nonzero(tile_of == col)[3])
    k[:, :, key, 0] = float("inf")               # minus infinity for every query but one
    def masses():
        return ca.compact_attn_tile_mass(ca.compact_attn_permute(q, lay), ca.compact_attn_permute(k, lay), lay)
    plain = masses()
    assert torch.isfinite(plain).all() and ca.compact_attn_layout_mass_shares(lay) == shares
    others = torch.arange(g.n, device=DEV) != row
    q[:, :, tile_of == row, 0] = 1.0
    mass = masses()
    assert torch.equal(mass[:, :, others], plain[:, :, others])
    assert torch.isnan(mass[:, :, row, col:]).all() and (mass[:, :, row, :col] == 0).all()
    k[:, :, key, 0] = float("nan")
    mass = masses()
    assert torch.isnan(mass[..., col]).all() and (mass[..., :col] == 0).all() and (mass[..., col + 1:] == 0).all()
    k[:, :, tile_of == col] = float("nan")
    assert torch.isnan(masses()).all()


@pytest.mark.parametrize("name", ["cfg3", "cfg4-S65"])
def test_tile_mass_every_pair_at_full_size_two_level_probe(name):
    """Every tile pair of every head at the benchmark sizes (24 and 50 launches per call).  Queries
    are one constant vector and a key's only non-zero component says whether its tile id is odd, so
    the softmax of every query has two levels, p_j = w^[tile(j) odd] / Z with w = exp(scale * 32)
    and Z = (real keys in even tiles) + w * (real keys in odd tiles), and the mass of a pair is
    pop[a] * pop[b] * w^[b odd] / Z: a closed form from the tile populations alone.  With q = 0 it
    is the uniform pop[a] * pop[b] / N."""
    wl = get_workload(name)
    _say("tile mass, all pairs", name)
    g = geometry_of(wl)
    D, Hd = wl.head_dim, wl.num_heads
    lay = build_layout(ca, wl)
    tok_tile = g.token_slots() // g.B
    pop = np.bincount(tok_tile, minlength=g.n).astype(np.float64)
    odd = (np.arange(g.n) % 2).astype(np.float64)
    q = torch.zeros(1, Hd, g.N_real, D, dtype=torch.bfloat16, device=DEV)
    k = torch.zeros(1, Hd, g.N_real, D, dtype=torch.bfloat16, device=DEV)
    k[..., 0] = torch.from_numpy(odd[tok_tile]).to(DEV).to(torch.bfloat16)
    kp = ca.compact_attn_permute(k, lay)
    del k
    scale = 1.0 / np.sqrt(D)
    for q0 in (0.0, 32.0):
        q[..., 0] = q0
        mass = ca.compact_attn_tile_mass(ca.compact_attn_permute(q, lay), kp, lay)
        torch.cuda.synchronize()
        w = np.exp(scale * q0 * odd)                                   # per key tile
        want = np.outer(pop, pop * w) / float((pop * w).sum())        # [n, n], the same for every head
        want_dev = torch.from_numpy(want).to(DEV).float()
        worst = max((mass[0, h] - want_dev).abs().max().item() for h in range(Hd))
        _say(name, "q0", q0, "worst abs err over all pairs", worst, "largest mass", want.max())
        assert worst <= MASS_ABS
        del mass


def test_tile_mass_in_a_captured_graph():
    """The first call for a layout allocates the kernel's workspace and is refused on a stream under
    capture; after one eager call the same call enqueues kernels only, and replays of the captured
    graph reproduce the eager masses (the workspace is reused by every replay)."""
    _say("tile mass, graph capture")
    wl = make_workload("massgraph", 4, 16, 16, (2, 8, 8), 128, 2, 128, "bf16", [[]] * 2)
    lay, fresh = build_layout(ca, wl), build_layout(ca, wl)
    q, k, _ = make_qkv(wl, DEV, q_gain=2.0)
    qp, kp = ca.compact_attn_permute(q, lay), ca.compact_attn_permute(k, lay)
    want = ca.compact_attn_tile_mass(qp, kp, lay)
    ca.compact_attn_layout_upload(fresh)                                # tables there, workspace not
    torch.cuda.synchronize()
    out, other = torch.zeros_like(want), torch.zeros_like(want)
    graph = torch.cuda.CUDAGraph()
    refused = None
    with torch.cuda.graph(graph):
        ca.compact_attn_tile_mass(qp, kp, lay, out=out)
        try:
            ca.compact_attn_tile_mass(qp, kp, fresh, out=other)
        except ca.CompactAttnError as exc:
            refused = exc
    assert refused is not None and refused.status == -1 and "workspace" in str(refused)
    for rep in range(3):
        out.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want), f"replay {rep}"
        _ = (qp.float() * 1.0001).sum().item()                          # eager work between replays


def test_tile_mass_rejects_fp32():
    wl = make_workload("massf", 2, 8, 8, (1, 4, 4), 0, 1, 64, "f32", [[]])
    lay = build_layout(ca, wl)
    q, k, _ = make_qkv(wl, DEV)
    qp, kp = ca.compact_attn_permute(q, lay), ca.compact_attn_permute(k, lay)
    with pytest.raises(ca.CompactAttnError) as e:
        ca.compact_attn_tile_mass(qp, kp, lay)
    assert e.value.status == -2


def test_search_pipeline_end_to_end():
    """Mass on the GPU -> window search on the host -> layout -> sparse forward, against the same
    chain in the oracle: identical windows, recall as reported, outputs within tolerance."""
    from oracle import search as OS
    _say("search pipeline")
    T, H, W, tile, D, Hd = 6, 32, 32, (2, 8, 8), 128, 3
    wl = make_workload("search", T, H, W, tile, 0, Hd, D, "bf16", [[]] * Hd)
    g = geometry_of(wl)
    probe = build_layout(ca, wl)
    q, k, v = make_qkv(wl, DEV, q_gain=3.0)
    qp, kp = ca.compact_attn_permute(q, probe), ca.compact_attn_permute(k, probe)
    mass = ca.compact_attn_tile_mass(qp, kp, probe)
    torch.cuda.synchronize()
    mass = mass[0].cpu().numpy()
    dts, tau, lam = [0, 1, g.nT - 1], 0.9, 0.6
    heads = []
    for h in range(Hd):
        groups, recall, kept = ca.compact_attn_search_head(probe, mass[h], dts, tau, lam)
        want_mass = OS.tile_mass(g, to_f64(q[0, h]), to_f64(k[0, h]))
        want_groups, want_recall, _ = OS.search_head(g, want_mass, dts, tau, lam)
        _say("head", h, groups, "recall", recall, "kept", kept)
        assert groups == want_groups and abs(recall - want_recall) < 1e-4 and recall >= tau
        assert kept < 1.0                                   # the position code gives it something to cut
        heads.append(groups)
    found = make_workload("found", T, H, W, tile, 0, Hd, D, "bf16", heads)
    lay = build_layout(ca, found)
    out, _ = gpu_attention(ca, found, lay, q, k, v)
    torch.cuda.synchronize()
    want = OA.masked_attention(g, heads, to_f64(q[0]), to_f64(k[0]), to_f64(v[0]))
    _say(compare(to_f64(out[0]), want, *tolerances("bf16"), what="searched layout"))


def test_pattern_families_end_to_end():
    """The three pattern families of Table 3 searched from GPU tile mass on structured heads (local,
    cross, global): the library finds what the oracle's search finds on the oracle's mass, the
    narrower families never return a second window, and the layout built from each answer runs
    through the sparse kernel within tolerance."""
    from oracle import search as OS
    _say("pattern families")
    T, H, W, tile, D = 6, 32, 32, (2, 8, 8), 128
    gains = [(2.5, 2.5, 2.5), (1.0, 3.0, 3.0), (0.0, 0.0, 0.0)]
    wl = make_workload("patterns", T, H, W, tile, 0, len(gains), D, "bf16", [[]] * len(gains))
    g = geometry_of(wl)
    probe = build_layout(ca, wl)
    q, k, v = make_qkv(wl, DEV, axis_gain=gains)
    mass = ca.compact_attn_tile_mass(ca.compact_attn_permute(q, probe), ca.compact_attn_permute(k, probe), probe)
    torch.cuda.synchronize()
    mass = mass[0].cpu().numpy()
    want_mass = [OS.tile_mass(g, to_f64(q[0, h]), to_f64(k[0, h])) for h in range(len(gains))]
    dts, tau, lam = [0, 1, 2], 0.9, 0.6
    sparsity = {}
    for pattern in ("cubic", "frame_groups", "dual"):
        heads = []
        for h in range(len(gains)):
            groups, recall, kept = ca.compact_attn_search_head(probe, mass[h], dts, tau, lam, pattern)
            want_groups, want_recall, want_kept = OS.search_head(g, want_mass[h], dts, tau, lam, pattern)
            _say(pattern, "head", h, groups, "recall", round(recall, 4), "sparsity", round(1 - kept, 4))
            assert groups == want_groups and abs(recall - want_recall) < 1e-4 and kept == pytest.approx(want_kept, abs=1e-12)
            assert recall >= tau
            if pattern != "dual":
                assert all(b == ABSENT for _, _, b in groups)
            heads.append(groups)
            sparsity[pattern, h] = 1 - kept
        found = make_workload("found", T, H, W, tile, 0, len(gains), D, "bf16", heads)
        lay = build_layout(ca, found)
        out, _ = gpu_attention(ca, found, lay, q, k, v)
        torch.cuda.synchronize()
        want = OA.masked_attention(g, heads, to_f64(q[0]), to_f64(k[0]), to_f64(v[0]))
        _say(compare(to_f64(out[0]), want, *tolerances("bf16"), what=f"{pattern} layout"))
    # the structure of Table 3 on these heads: the cross gains from the second window, the
    # time-variant local head from per-group windows, the structureless head from nothing
    assert sparsity["dual", 1] > sparsity["frame_groups", 1] + 0.1
    assert sparsity["frame_groups", 0] > sparsity["cubic", 0] + 0.1
    assert sparsity["dual", 2] == 0.0


# ---------------------------------------------------------------- gather / scatter inside the attention kernel

@pytest.mark.parametrize("shape", [
    (128, (5, 13, 20), (2, 8, 8), 128),       # B=128 D=128: T and H padded, text after the video
    (128, (5, 13, 18), (2, 8, 8), 0),         # no text: the padding slots of the last tiles lie past the last token;
                                              # W = 18 cuts a 4-token block in two
    (64, (5, 13, 20), (2, 8, 8), 128),        # B=128 D=64 (8-token blocks)
    (128, (3, 13, 20), (1, 8, 8), 64),        # B=64 D=128 (paired kernel)
    (64, (3, 9, 16), (1, 8, 8), 0),           # B=64 D=64
    (128, (4, 7, 12), (4, 8, 4), 0),          # tile width 4 = one block per run
    (128, (3, 9, 40), (1, 4, 16), 64),        # wide tiles: four blocks per run, B=64
    (64, (3, 5, 40), (2, 4, 16), 0),          # B=128 D=64, two 8-token blocks per run
])
def test_forward_natural_order(shape):
    """compact_attn_forward_natural reads q, k, v in natural order and writes natural order: same
    result as permute -> forward -> inverse permute, bit for bit, and within tolerance of the oracle."""
    D, (T, H, W), tile, n_text = shape
    _say("natural", shape)
    wl = make_workload("natural", T, H, W, tile, n_text, len(_EDGE_HEADS), D, "bf16", _EDGE_HEADS)
    g = geometry_of(wl)
    lay = build_layout(ca, wl)
    q, k, v = make_qkv(wl, DEV)
    out = torch.full_like(q, float("nan"))                 # every row must be written
    ca.compact_attn_forward_natural(q, k, v, lay, out=out)
    ref, _ = gpu_attention(ca, wl, lay, q, k, v)
    torch.cuda.synchronize()
    assert not torch.isnan(out.float()).any()
    assert torch.equal(out, ref)
    want = OA.masked_attention(g, wl.heads, to_f64(q[0]), to_f64(k[0]), to_f64(v[0]))
    _say(compare(to_f64(out[0]), want, *tolerances("bf16"), what="natural order"))


def test_forward_natural_rejects_what_it_does_not_cover():
    heads = [[(0, (1, 1), ABSENT)]]
    wl = make_workload("nat-f32", 2, 8, 8, (1, 4, 4), 0, 1, 64, "f32", heads)
    lay = build_layout(ca, wl)
    q, k, v = make_qkv(wl, DEV)
    with pytest.raises(ca.CompactAttnError):
        ca.compact_attn_forward_natural(q, k, v, lay)
    wl = make_workload("nat-tw", 2, 16, 16, (2, 8, 4), 0, 1, 64, "bf16", heads)   # D=64 needs tw % 8 == 0
    lay = build_layout(ca, wl)
    q, k, v = make_qkv(wl, DEV)
    with pytest.raises(ca.CompactAttnError):
        ca.compact_attn_forward_natural(q, k, v, lay)


# ---------------------------------------------------------------- random problems

_TILE_SHAPES = {64: [(1, 8, 8), (2, 4, 8), (1, 4, 16), (4, 4, 4), (1, 16, 4), (2, 8, 4)],
                128: [(2, 8, 8), (1, 8, 16), (1, 16, 8), (4, 4, 8), (2, 4, 16), (8, 4, 4)]}


def _random_problem(seed):
    """A seeded random problem: tile shape, ragged grid, text tiles, 1-3 heads with up to three frame
    groups of clipped or clamped windows (absent windows and empty heads included), batch 1-2."""
    rng = np.random.default_rng(seed)
    B, D = int(rng.choice([64, 128])), int(rng.choice([64, 128]))
    tile = _TILE_SHAPES[B][int(rng.integers(len(_TILE_SHAPES[B])))]
    T, H, W = int(rng.integers(1, 4 * tile[0] + 2)), int(rng.integers(3, 4 * tile[1] + 3)), int(rng.integers(3, 3 * tile[2] + 5))
    while T * H * W > 9000:
        H, W = max(3, H - 3), max(3, W - 3)
    n_text = int(rng.choice([0, 0, B, 2 * B]))
    Hd, batch = int(rng.integers(1, 4)), int(rng.choice([1, 1, 2]))
    heads = []
    for _ in range(Hd):
        if rng.integers(4) == 0:
            heads.append([])
            continue
        groups = []
        for dt in sorted(set(int(x) for x in rng.integers(0, 6, int(rng.integers(1, 4))))):
            a = (int(rng.integers(-1, 4)), int(rng.integers(-1, 4)))
            b = (int(rng.integers(-1, 4)), int(rng.integers(-1, 4)))
            groups.append((dt, a if min(a) >= 0 else ABSENT, b if min(b) >= 0 else ABSENT))
        heads.append(groups)
    clamp = [bool(rng.integers(2)) for _ in range(Hd)]
    return B, D, tile, (T, H, W), n_text, batch, heads, clamp, float(rng.choice([1.0, 2.0, 3.0]))


@pytest.mark.parametrize("first_seed", [0, 8, 16])
def test_random_problems_through_every_entry_point(first_seed):
    """Eight seeded random problems per case through permute, sparse forward, dense, the natural-order
    forward, the allocation-free forward and the tile mass, each against the oracle (the last two
    forwards bit for bit against the first)."""
    import dataclasses
    from oracle import search as OS
    for seed in range(first_seed, first_seed + 8):
        B, D, tile, (T, H, W), n_text, batch, heads, clamp, gain = _random_problem(seed)
        _say("random problem", seed, B, D, tile, (T, H, W), n_text, batch, heads, clamp)
        Hd = len(heads)
        wl = dataclasses.replace(make_workload("random", T, H, W, tile, n_text, Hd, D, "bf16", heads), batch=batch)
        g = geometry_of(wl)
        lay = ca.compact_attn_build_layout(T, H, W, tile, n_text, batch, Hd, D, "bf16", heads, clamp_centre=clamp)
        oracle_heads = [OL.ClampedHead(h) if c else h for h, c in zip(heads, clamp)]
        q, k, v = make_qkv(wl, DEV, q_gain=gain)
        out, out_tiled = gpu_attention(ca, wl, lay, q, k, v)
        dense, _ = gpu_attention(ca, wl, lay, q, k, v, dense=True)
        qp, kp, vp = (ca.compact_attn_permute(t, lay) for t in (q, k, v))
        mass = ca.compact_attn_tile_mass(qp, kp, lay)
        if tile[2] % (4 if D == 128 else 8) == 0:
            assert torch.equal(ca.compact_attn_forward_natural(q, k, v, lay), out)
        assert torch.equal(ca.compact_attn_forward_static(qp, kp, vp, lay), out_tiled)
        torch.cuda.synchronize()
        for b in range(batch):
            want = OA.masked_attention(g, oracle_heads, to_f64(q[b]), to_f64(k[b]), to_f64(v[b]))
            compare(to_f64(out[b]), want, *tolerances("bf16"), what=f"seed {seed} forward")
            want = OA.dense_attention(to_f64(q[b]), to_f64(k[b]), to_f64(v[b]))
            compare(to_f64(dense[b]), want, *tolerances("bf16"), what=f"seed {seed} dense")
            for h in range(Hd):
                want = OS.tile_mass(g, to_f64(q[b, h]), to_f64(k[b, h]))
                assert np.abs(mass[b, h].double().cpu().numpy() - want).max() <= MASS_ABS, f"seed {seed} mass"
        lay.free()


# ---------------------------------------------------------------- batch > 1

@pytest.mark.parametrize("dtype,D,tile", [("bf16", 128, (2, 8, 8)), ("bf16", 64, (1, 8, 8)), ("f32", 64, (1, 4, 4))])
def test_batch_of_three(dtype, D, tile):
    """Every batch entry is an independent problem with the same layout (rows * batch work items,
    enough of them here to exercise the XCD-aware remapping of workgroup ids and its remainder)."""
    import dataclasses
    _say("batch", dtype, D, tile)
    B = tile[0] * tile[1] * tile[2]
    heads = [[(1, (1, 1), ABSENT), (3, (0, 0), ABSENT)], [(5, (0, 3), (2, 0))], []]
    wl = make_workload("batch", 6, 24, 40, tile, B, len(heads), D, dtype, heads)
    wl = dataclasses.replace(wl, batch=3)
    g = geometry_of(wl)
    lay = build_layout(ca, wl)
    q, k, v = make_qkv(wl, DEV)
    out, _ = gpu_attention(ca, wl, lay, q, k, v)
    dense, _ = gpu_attention(ca, wl, lay, q, k, v, dense=True)
    torch.cuda.synchronize()
    assert not torch.equal(out[0], out[1])
    if dtype == "bf16":
        assert torch.equal(ca.compact_attn_forward_natural(q, k, v, lay), out)
    full = [[(g.nT - 1, (g.nH - 1, g.nW - 1), ABSENT)]] * len(heads)
    for b in range(3):
        want = OA.masked_attention(g, heads, to_f64(q[b]), to_f64(k[b]), to_f64(v[b]))
        _say(b, compare(to_f64(out[b]), want, *tolerances(dtype), what=f"batch {b}"))
    want = OA.masked_attention(g, full, to_f64(q[2]), to_f64(k[2]), to_f64(v[2]))
    _say("dense", compare(to_f64(dense[2]), want, *tolerances(dtype), what="dense batch 2"))


# ---------------------------------------------------------------- streams and graph replay

def test_forward_on_a_side_stream_and_in_a_replayed_graph():
    """The entry points enqueue on the caller's stream and allocate nothing once the layout is
    uploaded, so the whole path can be captured in a HIP graph; every replay (with eager work and
    synchronisation in between) must reproduce the eager result bit for bit."""
    _say("graph replay")
    wl = get_workload("cfg2")
    lay = build_layout(ca, wl)
    ca.compact_attn_layout_upload(lay)
    q, k, v = make_qkv(wl, DEV)
    eager, _ = gpu_attention(ca, wl, lay, q, k, v)
    torch.cuda.synchronize()
    shape_p = lay.shape(True)
    qp, kp, vp, op = (torch.empty(shape_p, dtype=q.dtype, device=DEV) for _ in range(4))
    out = torch.empty_like(q)

    def path():
        ca.compact_attn_permute(q, lay, out=qp)
        ca.compact_attn_permute(k, lay, out=kp)
        ca.compact_attn_permute(v, lay, out=vp)
        ca.compact_attn_forward(qp, kp, vp, lay, out=op)
        ca.compact_attn_permute(op, lay, inverse=True, out=out)

    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        path()
    side.synchronize()
    assert torch.equal(out, eager)

    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        path()
    for rep in range(3):
        out.zero_()
        op.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, eager), f"replay {rep}"
        _ = (q.float() * 1.0001).sum().item()             # eager work between replays


# ---------------------------------------------------------------- determinism

def test_run_to_run_bitwise_identical():
    _say("determinism")
    wl = get_workload("cfg2")
    lay = build_layout(ca, wl)
    q, k, v = make_qkv(wl, DEV)
    a, _ = gpu_attention(ca, wl, lay, q, k, v)
    b, _ = gpu_attention(ca, wl, lay, q, k, v)
    torch.cuda.synchronize()
    assert torch.equal(a, b)


def test_layout_on_device_matches_oracle_after_upload():
    """The CSR the kernels read is the host CSR: upload, then run a probe whose answer
    depends on every column index (covered by the probes above); here the C-ABI views are
    compared once more on the GPU machine so that the run records the library as loaded."""
    _say("layout on GPU box")
    wl = get_workload("cfg2")
    g = geometry_of(wl)
    lay = build_layout(ca, wl)
    ca.compact_attn_layout_upload(lay)
    want = OL.build_csr(g, wl.heads)
    for h in range(wl.num_heads):
        rp, ci = ca.compact_attn_layout_csr(lay, h)
        assert np.array_equal(rp, want[h][0]) and np.array_equal(ci, want[h][1])


# ---------------------------------------------------------------- fp32: every split of a tile over waves

@pytest.mark.parametrize("D,grid,tile,text_tiles,num_heads", [
    (64, (2, 3, 5), (1, 1, 1), 1, 2),         # one-token tiles: every block of 16 keys holds one
    (32, (5, 7, 9), (1, 3, 7), 1, 3),         # 21 slots: two query groups, the second with five
    (64, (2, 9, 11), (1, 6, 10), 1, 3),       # 60 slots, padded along H and W
    (128, (3, 17, 20), (2, 6, 8), 0, 2),      # 96 slots, padded along all axes
    (128, (3, 9, 9), (2, 8, 8), 1, 2),        # 128 slots, tiles down to one token, parts without any
    (32, (2, 32, 29), (1, 8, 8), 0, 20),      # 640 rows of 64: two groups side by side
    (64, (2, 32, 29), (1, 8, 8), 0, 40),      # 1280 rows of 64: four
])
def test_fp32_splits_of_a_tile(D, grid, tile, text_tiles, num_heads):
    """The fp32 kernel at the edges of its query groups and key blocks; what the padding slots of K and V hold does not matter."""
    _say("fp32 split", D, grid, tile, num_heads)
    B = tile[0] * tile[1] * tile[2]
    heads = (_EDGE_HEADS[:3] * num_heads)[:num_heads]
    wl = make_workload("f32-split", *grid, tile, text_tiles * B, num_heads, D, "f32", heads)
    g = geometry_of(wl)
    lay = build_layout(ca, wl)
    q, k, v = make_qkv(wl, DEV, q_gain=2.0)
    qp, kp, vp = (ca.compact_attn_permute(x, lay) for x in (q, k, v))
    held = ca.compact_attn_permute(torch.ones_like(q), lay) != 0
    kp[~held] = float("nan")
    vp[~held] = float("nan")
    out = ca.compact_attn_forward(qp, kp, vp, lay, out=torch.full_like(qp, float("nan")))
    assert torch.all(out[~held] == 0)
    got = ca.compact_attn_permute(out, lay, inverse=True)
    want = OA.masked_attention(g, heads, to_f64(q[0]), to_f64(k[0]), to_f64(v[0]))
    _say(compare(to_f64(got[0]), want, *tolerances("f32"), what="fp32 split"))


# ---------------------------------------------------------------- infinite values

# kernel, head dim and tile, and video grids on which the kernel serves some launch size
_EVERY_BF16_KERNEL = [("ways-8x2", 128, (2, 8, 8)), ("ways-8x2", 64, (2, 8, 8)), ("ways-8x2", 128, (1, 8, 8)), ("ways-8x2", 64, (1, 8, 8)),
                      ("ways-8x4", 128, (2, 8, 8)), ("ways-4x4", 128, (2, 8, 8)), ("ways-4x4", 64, (2, 8, 8)),
                      ("packed-faces", 128, (2, 8, 8)), ("paired", 128, (1, 8, 8)), ("one-tile", 64, (2, 8, 8)),
                      ("one-tile", 64, (1, 8, 8)), ("one-tile-3", 64, (1, 8, 8))]


@pytest.mark.parametrize("kernel,D,tile", [("f32", 128, (2, 8, 8)), ("f32", 64, (1, 6, 10)), ("f32", 32, (1, 3, 7)), *_EVERY_BF16_KERNEL])
def test_infinite_value_in_the_last_token_of_a_tile(kernel, D, tile):
    """Every query keeps every key, so an infinite channel of one V token makes that channel infinite in every row
    and leaves the others alone, also when the token is the last of a tile whose other slots are padding, or the last
    of the walk."""
    T, H, W = grid = (5, 13, 21)
    dtype = "f32" if kernel == "f32" else "bf16"
    for text_tiles in (0, 1):
        _say("infinite V", kernel, D, tile, text_tiles)
        wl, lay = workload_for_kernel(ca, kernel, grid, tile, text_tiles * tile[0] * tile[1] * tile[2], D, dtype, [[(T, (H, W), ABSENT)]])
        q, k, v = make_qkv(wl, DEV)
        corner = T * H * W - 1                             # of the last video tile
        tokens = {3: corner, 5: corner - (W - 1) % tile[2] - 1, 9: v.shape[2] - 1, 11: tile[2] - 1}   # by channel
        v_inf = v.clone()
        for channel, token in tokens.items():
            v_inf[:, :, token, channel] = float("inf")
        for dense in (False, True):
            want, _ = gpu_attention(ca, wl, lay, q, k, v, dense=dense)
            want[..., list(tokens)] = float("inf")
            got, _ = gpu_attention(ca, wl, lay, q, k, v_inf, dense=dense)
            assert torch.equal(got, want), (dense, torch.isnan(got).sum().item())
        if kernel.startswith("ways"):                      # the others copy whole tiles, and in natural order rows of neighbouring tiles
            got = ca.compact_attn_forward_natural(q, k, v_inf, lay)
            assert torch.equal(got, want)


# ---------------------------------------------------------------- tile mass: row groups and steps

@pytest.mark.parametrize("D,grid,tile,text_tiles", [
    (64, (1, 8, 8), (1, 8, 8), 0),            # one tile: half a row group, half a step of two key tiles
    (64, (1, 7, 15), (1, 8, 8), 0),           # two tiles, the second with 49 slots of 64
    (64, (1, 16, 20), (1, 8, 8), 1),          # seven tiles: the last group has one row, the last step one tile
    (128, (1, 8, 8), (1, 8, 8), 0),           # 64-token tiles, head dim 128: one key tile a step
    (128, (3, 8, 5), (1, 8, 8), 0),
    (64, (1, 8, 8), (2, 8, 8), 0),            # 128-token tile with an empty upper half
    (128, (3, 8, 9), (2, 8, 8), 1),
])
def test_tile_mass_short_walks(D, grid, tile, text_tiles):
    """Layouts of a few tiles: row groups and steps that are not full, with quiet and with peaked rows."""
    from oracle import search as OS
    _say("tile mass, short", D, grid, tile)
    B = tile[0] * tile[1] * tile[2]
    wl = make_workload("mass-short", *grid, tile, text_tiles * B, 3, D, "bf16", [[]] * 3)
    g = geometry_of(wl)
    lay = build_layout(ca, wl)
    for gain in (1.0, 8.0):
        q, k, _ = make_qkv(wl, DEV, q_gain=gain)
        mass = torch.full((1, 3, g.n, g.n), float("nan"), device=DEV)
        ca.compact_attn_tile_mass(ca.compact_attn_permute(q, lay), ca.compact_attn_permute(k, lay), lay, out=mass)
        got = mass[0].double().cpu().numpy()
        for h in range(3):
            err = np.abs(got[h] - OS.tile_mass(g, to_f64(q[0, h]), to_f64(k[0, h])))
            assert err.max() <= MASS_ABS, (h, gain, err.max())


# ---------------------------------------------------------------- every bf16 kernel at small sizes

@pytest.mark.parametrize("D,grid,tile,text_tiles,copies,batch", [
    # padded along all axes, empty rows, tiles of a few tokens
    (128, (5, 13, 20), (2, 8, 8), 0, 1, 2),
    (64, (5, 13, 20), (2, 8, 8), 0, 1, 2),
    (128, (3, 13, 20), (1, 8, 8), 1, 1, 1),
    (64, (3, 13, 20), (1, 8, 8), 1, 1, 1),
    (128, (1, 9, 17), (2, 8, 8), 1, 1, 1),
    (64, (5, 9, 9), (4, 4, 8), 0, 1, 1),
    # rows enough to fill the card
    (128, (7, 17, 17), (2, 8, 8), 0, 12, 1),
    (64, (7, 17, 17), (2, 8, 8), 0, 12, 1),
    (128, (7, 17, 17), (2, 8, 8), 1, 3, 2),
    (64, (4, 16, 24), (2, 8, 8), 0, 60, 2),
    (128, (5, 13, 20), (2, 8, 8), 1, 40, 2),
    (128, (9, 20, 20), (2, 8, 8), 1, 8, 1),
    (64, (5, 13, 20), (2, 8, 8), 1, 4, 1),
    (128, (3, 13, 20), (1, 8, 8), 1, 16, 2),
    (64, (3, 13, 20), (1, 8, 8), 1, 40, 2),
])
def test_bf16_kernels_by_launch_size(D, grid, tile, text_tiles, copies, batch):
    """The same four heads in launches of many sizes, tiles and grids, whichever kernel they take: sparse and dense
    walk against the oracle with peaked rows, natural order and the static entry point bit for bit."""
    import dataclasses
    _say("bf16 by launch size", D, grid, tile, copies, batch)
    B = tile[0] * tile[1] * tile[2]
    heads = list(_EDGE_HEADS) * copies
    wl = dataclasses.replace(make_workload("by-size", *grid, tile, text_tiles * B, len(heads), D, "bf16", heads), batch=batch)
    g = geometry_of(wl)
    lay = build_layout(ca, wl)
    q, k, v = make_qkv(wl, DEV, q_gain=3.0)
    out, out_tiled = gpu_attention(ca, wl, lay, q, k, v)
    dense, _ = gpu_attention(ca, wl, lay, q, k, v, dense=True)
    assert torch.equal(ca.compact_attn_forward_natural(q, k, v, lay, out=torch.full_like(q, float("nan"))), out)
    qp, kp, vp = (ca.compact_attn_permute(x, lay) for x in (q, k, v))
    assert torch.equal(ca.compact_attn_forward_static(qp, kp, vp, lay, out=torch.full_like(qp, float("nan"))), out_tiled)
    held = ca.compact_attn_permute(torch.ones_like(q), lay) != 0
    assert torch.all(out_tiled[~held] == 0)
    full = [[(g.nT - 1, (g.nH - 1, g.nW - 1), ABSENT)]]
    h0 = len(heads) - 4                                     # the last four heads of the last batch entry
    for h in range(4):
        qkv = [to_f64(x[batch - 1, h0 + h])[None] for x in (q, k, v)]
        _say(h, compare(to_f64(out[batch - 1, h0 + h])[None], OA.masked_attention(g, [heads[h]], *qkv), *tolerances("bf16"), what="sparse"))
        _say(h, compare(to_f64(dense[batch - 1, h0 + h])[None], OA.masked_attention(g, full, *qkv), *tolerances("bf16"), what="dense"))


@pytest.mark.parametrize("kernel,D,tile", _EVERY_BF16_KERNEL)
def test_every_bf16_kernel(kernel, D, tile):
    """The sparse walk of every kernel of the bf16 dispatch against the oracle, with peaked rows on a grid padded along
    all axes; natural order, the static entry point and a replayed graph bit for bit; the padding slots of K and V are
    not read by the kernels that say so."""
    _say("every kernel", kernel, D, tile)
    wl, lay = workload_for_kernel(ca, kernel, (5, 13, 20), tile, tile[0] * tile[1] * tile[2], D, "bf16", _EDGE_HEADS, batch=2)
    g = geometry_of(wl)
    q, k, v = make_qkv(wl, DEV, q_gain=3.0)
    out, out_tiled = gpu_attention(ca, wl, lay, q, k, v)
    for h in range(wl.num_heads - 4, wl.num_heads):
        qkv = [to_f64(x[1, h])[None] for x in (q, k, v)]
        _say(h, compare(to_f64(out[1, h])[None], OA.masked_attention(g, [wl.heads[h]], *qkv), *tolerances("bf16"), what=kernel))
    assert torch.equal(ca.compact_attn_forward_natural(q, k, v, lay, out=torch.full_like(q, float("nan"))), out)
    qp, kp, vp = (ca.compact_attn_permute(x, lay) for x in (q, k, v))
    again = torch.full_like(qp, float("nan"))
    assert torch.equal(ca.compact_attn_forward_static(qp, kp, vp, lay, out=again), out_tiled)
    held = ca.compact_attn_permute(torch.ones_like(q), lay) != 0
    assert torch.all(out_tiled[~held] == 0)
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        ca.compact_attn_forward(qp, kp, vp, lay, out=again)
    for rep in range(3):
        again.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(again, out_tiled), f"replay {rep}"
        assert torch.equal(ca.compact_attn_forward(qp, kp, vp, lay), out_tiled)   # an eager launch between replays
    if kernel.startswith("ways"):
        kp[~held] = float("nan")
        vp[~held] = float("nan")
        assert torch.equal(ca.compact_attn_forward(qp, kp, vp, lay), out_tiled)


@pytest.mark.parametrize("kernel,D,tile", _EVERY_BF16_KERNEL)
def test_rising_and_huge_scores_on_every_bf16_kernel(kernel, D, tile):
    """As test_rising_and_huge_scores: the exponent reference of every way moves along the walk, and the ways of a query
    end with references far apart."""
    T, H, W = grid = (5, 14, 18)
    _say("rising scores", kernel, D, tile)
    heads = [[(T, (1, 1), ABSENT)], [(T, (9, 9), ABSENT)]]
    wl, lay = workload_for_kernel(ca, kernel, grid, tile, tile[0] * tile[1] * tile[2], D, "bf16", heads)
    g = geometry_of(wl)
    q, k, v = make_qkv(wl, DEV)
    tok_tile, _ = g.token_tile_and_slot()
    ramp = torch.tensor(np.asarray(tok_tile), device=DEV, dtype=torch.float32) / g.n
    last = slice(wl.num_heads - 2, wl.num_heads)
    for gain, q_gain in ((1.0, 2.0), (40.0, 6.0)):
        kk = (k.float() * (1.0 + 3.0 * gain * ramp[None, None, :, None])).to(k.dtype)
        qq = (q.float() * q_gain).to(q.dtype)
        out, _ = gpu_attention(ca, wl, lay, qq, kk, v)
        want = OA.masked_attention(g, heads, *(to_f64(x[0, last]) for x in (qq, kk, v)))
        _say(gain, compare(to_f64(out[0, last]), want, *tolerances("bf16"), what=f"gain {gain}"))


@pytest.mark.parametrize("kernel,D,tile", [*_EVERY_BF16_KERNEL, ("one-tile", 128, (2, 8, 8))])
def test_imported_random_mask_on_every_bf16_kernel(kernel, D, tile):
    """Arbitrary tile masks given as CSR (an empty row, a full one, whole runs of empty rows) on every kernel, and their
    union with a second set."""
    T, H, W = 5, 13, 20
    B = tile[0] * tile[1] * tile[2]
    _say("imported masks", kernel, D, tile)
    g = geometry_of(make_workload("import", T, H, W, tile, B, 3, D, "bf16", [[]] * 3))
    rng = np.random.default_rng(5)
    masks = rng.random((3, g.n, g.n)) < 0.25
    masks[0, 3] = False
    masks[1, :, g.n - 1] = True
    masks[2, :6] = False
    masks[2, 7] = True
    if kernel == "packed-faces":                           # worth it where neighbours along w share their lists
        masks[:, :g.n_vid] = masks[:, np.arange(g.n_vid) // g.nW * g.nW]
    other = rng.random((3, g.n, g.n)) < 0.1

    def layout(ms, copies):
        return ca.compact_attn_layout_from_csr(T, H, W, tile, B, 1, 3 * copies, D, "bf16", [OL.csr_of_mask(m) for m in ms] * copies)

    copies, lay = layout_for_kernel(ca, kernel, lambda n: layout(masks, n))
    wl = make_workload("import", T, H, W, tile, B, 3 * copies, D, "bf16", [[]] * 3 * copies)
    q, k, v = make_qkv(wl, DEV)
    last = slice(3 * copies - 3, 3 * copies)
    for lay, ms in ((lay, masks), (ca.compact_attn_layout_union(lay, layout(other, copies)), OL.union_masks(masks, other))):
        out, _ = gpu_attention(ca, wl, lay, q, k, v)
        want = OA.tile_mask_attention(g, ms, *(to_f64(x[0, last]) for x in (q, k, v)))
        _say(ca.compact_attn_layout_kernel(lay), compare(to_f64(out[0, last]), want, *tolerances("bf16"), what="imported masks"))


@pytest.mark.parametrize("kernel,D,B", [("ways-8x2", 128, 128), ("ways-8x2", 64, 64), ("ways-8x4", 128, 128), ("ways-4x4", 128, 128), ("ways-4x4", 64, 128),
                                        ("packed-faces", 128, 128), ("paired", 128, 64), ("one-tile", 64, 128), ("one-tile-3", 64, 64)])
def test_random_problems_on_every_bf16_kernel(kernel, D, B):
    """Four seeded random problems (tile shapes, ragged grids, text tiles, windows, batch) per kernel, with as many copies
    of their heads as it takes to reach it: sparse walk of the last heads against the oracle, natural order and the
    static entry point bit for bit."""
    import dataclasses
    done = 0
    for seed in range(100, 220):
        seed_B, seed_D, tile, (T, H, W), n_text, batch, heads, clamp, gain = _random_problem(seed)
        if (seed_B, seed_D) != (B, D) or T * H * W > 5000:
            continue
        found = layout_for_kernel(ca, kernel, lambda n: ca.compact_attn_build_layout(T, H, W, tile, n_text, batch, n * len(heads), D, "bf16",
                                                                                     heads * n, clamp_centre=clamp * n))
        if not found:
            continue
        copies, lay = found
        Hd = copies * len(heads)
        _say("random problem", seed, kernel, B, D, tile, (T, H, W), n_text, batch, Hd)
        wl = dataclasses.replace(make_workload("random", T, H, W, tile, n_text, Hd, D, "bf16", heads * copies), batch=batch)
        g = geometry_of(wl)
        q, k, v = make_qkv(wl, DEV, q_gain=gain)
        out, out_tiled = gpu_attention(ca, wl, lay, q, k, v)
        if tile[2] % (4 if D == 128 else 8) == 0:
            assert torch.equal(ca.compact_attn_forward_natural(q, k, v, lay), out)
        qp, kp, vp = (ca.compact_attn_permute(t, lay) for t in (q, k, v))
        assert torch.equal(ca.compact_attn_forward_static(qp, kp, vp, lay), out_tiled)
        last = slice(Hd - len(heads), Hd)
        want = OA.masked_attention(g, [OL.ClampedHead(h) if c else h for h, c in zip(heads, clamp)], *(to_f64(x[batch - 1, last]) for x in (q, k, v)))
        compare(to_f64(out[batch - 1, last]), want, *tolerances("bf16"), what=f"seed {seed}")
        lay.free()
        done += 1
        if done == 4:
            return
    assert False, f"only {done} random problems reach the {kernel} kernel"


# ---------------------------------------------------------------- rows split along the keys

_GLOBAL, _LOCAL, _NEAR = [(99, (99, 99), ABSENT)], [(1, (1, 1), ABSENT)], [(0, (0, 1), ABSENT)]
_MIXED = [_GLOBAL, [], _NEAR]


_SPLIT_LAUNCHES = [
    # few tiles and one head: shares of one or two tiles, tiles of a few tokens
    ("one-tile", 64, (2, 8, 29), (1, 8, 8), 0, [_GLOBAL], 1),
    ("one-tile", 64, (2, 8, 40), (2, 8, 8), 0, [_GLOBAL], 1),
    ("one-tile", 128, (1, 21, 8), (2, 8, 8), 1, [_GLOBAL], 1),
    ("packed-faces", 128, (1, 8, 20), (2, 8, 8), 1, [_GLOBAL], 1),
    ("paired", 128, (1, 8, 29), (1, 8, 8), 1, [_GLOBAL], 1),
    ("ways-4x4", 128, (5, 21, 8), (2, 8, 8), 1, [_GLOBAL], 1),
    ("ways-8x2", 64, (3, 16, 12), (2, 8, 8), 1, [_GLOBAL], 1),
    ("ways-8x2", 64, (2, 21, 20), (1, 8, 8), 0, [_GLOBAL], 1),
    ("ways-8x2", 128, (5, 8, 20), (2, 8, 8), 1, [_GLOBAL], 1),
    # split and whole rows, empty rows
    ("one-tile", 64, (7, 8, 8), (1, 8, 8), 1, _MIXED, 2),
    ("one-tile-3", 64, (24, 8, 20), (1, 8, 8), 1, [_GLOBAL, _GLOBAL, _GLOBAL, _GLOBAL, _LOCAL, _LOCAL, [], _NEAR] * 2, 2),
    ("one-tile", 128, (2, 30, 8), (2, 8, 8), 1, _MIXED, 2),
    ("packed-faces", 128, (2, 13, 20), (2, 8, 8), 1, _MIXED, 2),
    ("paired", 128, (2, 21, 8), (1, 8, 8), 1, _MIXED, 2),
    ("ways-4x4", 64, (9, 21, 8), (2, 8, 8), 1, _MIXED, 2),
    ("ways-4x4", 128, (5, 30, 8), (2, 8, 8), 1, _MIXED, 2),
    ("ways-8x4", 128, (5, 8, 40), (2, 8, 8), 1, _MIXED, 2),
    ("ways-8x2", 64, (9, 13, 8), (2, 8, 8), 1, _MIXED, 2),
    ("ways-8x2", 128, (16, 30, 8), (1, 8, 8), 1, _MIXED, 2),
]


@pytest.mark.parametrize("kernel,D,grid,tile,text_tiles,heads,batch", _SPLIT_LAUNCHES)
def test_rows_split_along_the_keys(kernel, D, grid, tile, text_tiles, heads, batch):
    """Launches whose rows are shared by several workgroups: against the oracle with peaked rows, whatever the workspace holds
    before the call; natural order, the static entry point, a second stream and a replayed graph bit for bit; the C call without a
    workspace to within the rounding of bf16 probabilities."""
    import ctypes
    import dataclasses
    _say("split rows", kernel, D, grid, tile, batch)
    B = tile[0] * tile[1] * tile[2]
    wl = dataclasses.replace(make_workload("split", *grid, tile, text_tiles * B, len(heads), D, "bf16", heads), batch=batch)
    g = geometry_of(wl)
    lay = build_layout(ca, wl)
    nbytes, name = ca.compact_attn_layout_split(lay)
    assert name == kernel and nbytes > 0
    q, k, v = make_qkv(wl, DEV, q_gain=3.0)
    del_me = torch.full((nbytes // 2,), float("nan"), dtype=torch.bfloat16, device=DEV)  # the allocator's next block of that size
    del del_me
    out, out_tiled = gpu_attention(ca, wl, lay, q, k, v)
    for h in range(len(heads)):
        qkv = [to_f64(x[batch - 1, h])[None] for x in (q, k, v)]
        _say(h, compare(to_f64(out[batch - 1, h])[None], OA.masked_attention(g, [heads[h]], *qkv), *tolerances("bf16"), what=kernel))
    held = ca.compact_attn_permute(torch.ones_like(q), lay) != 0
    assert torch.all(out_tiled[~held] == 0)
    assert torch.equal(ca.compact_attn_forward_natural(q, k, v, lay, out=torch.full_like(q, float("nan"))), out)
    qp, kp, vp = (ca.compact_attn_permute(x, lay) for x in (q, k, v))
    again = torch.full_like(qp, float("nan"))
    assert torch.equal(ca.compact_attn_forward_static(qp, kp, vp, lay, out=again), out_tiled)
    side = torch.cuda.Stream()
    on_side = [torch.full_like(qp, float("nan")) for _ in range(2)]
    side.wait_stream(torch.cuda.current_stream())
    for x in on_side:
        ca.compact_attn_forward(qp, kp, vp, lay, out=x, stream=side)
    with_main = ca.compact_attn_forward(qp, kp, vp, lay)            # may overlap with them
    torch.cuda.synchronize()
    assert all(torch.equal(x, out_tiled) for x in (*on_side, with_main))
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        ca.compact_attn_forward(qp, kp, vp, lay, out=again)
    for rep in range(3):
        again.fill_(float("nan"))
        graph.replay()
        assert torch.equal(ca.compact_attn_forward(qp, kp, vp, lay), out_tiled)
        torch.cuda.synchronize()
        assert torch.equal(again, out_tiled), f"replay {rep}"
    # the C calls: without a workspace, and with one that will not do
    lib, stream = ca.load_library(), ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    ptrs = [ctypes.c_void_p(x.data_ptr()) for x in (qp, kp, vp)]
    assert lib.compact_attn_forward(*ptrs, lay.handle, ctypes.c_void_p(again.data_ptr()), stream) == 0
    compare(to_f64(again), to_f64(out_tiled), *tolerances("bf16"), what="without a workspace")
    work = torch.empty(nbytes + 16, dtype=torch.uint8, device=DEV)
    before = again.clone()
    for at, size in ((None, nbytes), (work.data_ptr(), nbytes - 1), (work.data_ptr() + 1, nbytes), (qp.data_ptr(), nbytes)):
        status = lib.compact_attn_forward_with_workspace(*ptrs, lay.handle, ctypes.c_void_p(again.data_ptr()), 0, ctypes.c_void_p(at), size, stream)
        assert status == -1, (at, size)
    torch.cuda.synchronize()
    assert torch.equal(again, before)


@pytest.mark.parametrize("kernel,D,grid,tile,text_tiles,heads,batch", _SPLIT_LAUNCHES)
@pytest.mark.parametrize("hidden", ["whole shares", "first tiles of a share"])
def test_minus_infinite_scores_in_split_rows(kernel, D, grid, tile, text_tiles, heads, batch, hidden):
    """Keys whose scores are minus infinity have no weight, and those beside them keep theirs however far below zero they lie
    (-512 scaled here: exp2 of such a score against a reference of zero is zero), whether such keys fill a share or only its first
    tiles.  The same for whole rows, which the C call without a workspace walks."""
    import ctypes
    import dataclasses
    _say("minus infinity", kernel, D, grid, tile, batch, hidden)
    B = tile[0] * tile[1] * tile[2]
    wl = dataclasses.replace(make_workload("split", *grid, tile, text_tiles * B, len(heads), D, "bf16", heads), batch=batch)
    g = geometry_of(wl)
    lay = build_layout(ca, wl)
    assert ca.compact_attn_layout_split(lay)[1] == kernel
    q, k, v = make_qkv(wl, DEV)
    tile_of = torch.from_numpy(np.asarray(g.token_tile_and_slot()[0])).to(DEV)
    q[..., 0] = 16.0
    k[..., 0] = -32.0 * D ** 0.5
    k[:, :, tile_of < g.n // 2 + 1 if hidden == "whole shares" else tile_of % 3 != 2, 0] = float("-inf")
    qp, kp, vp = (ca.compact_attn_permute(x, lay) for x in (q, k, v))
    split = ca.compact_attn_forward(qp, kp, vp, lay)
    whole = torch.empty_like(split)
    status = ca.load_library().compact_attn_forward(*(ctypes.c_void_p(x.data_ptr()) for x in (qp, kp, vp)), lay.handle, ctypes.c_void_p(whole.data_ptr()),
                                                    ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert status == 0
    for what, x in (("split", split), ("whole", whole)):
        out = ca.compact_attn_permute(x, lay, inverse=True)
        for h in range(len(heads)):
            with np.errstate(invalid="ignore"):
                want = OA.masked_attention(g, [heads[h]], *(to_f64(t[batch - 1, h])[None] for t in (q, k, v)))
            want = np.nan_to_num(want, nan=0.0)   # a query all of whose keys are hidden has no softmax, and gets zeros
            _say(what, h, compare(to_f64(out[batch - 1, h])[None], want, *tolerances("bf16"), what=what))


@pytest.mark.parametrize("which", ["side", "default"])
def test_split_rows_on_a_stream_known_by_its_handle(which):
    """`stream` is anything with a `cuda_stream`, also where the binding takes a workspace from that stream's memory."""
    class Handle:
        pass
    wl = make_workload("handle", 3, 16, 12, (2, 8, 8), 128, 1, 64, "bf16", [_GLOBAL])
    lay = build_layout(ca, wl)
    assert ca.compact_attn_layout_split(lay)[0] > 0
    q, k, v = make_qkv(wl, DEV)
    qp, kp, vp = (ca.compact_attn_permute(x, lay) for x in (q, k, v))
    want = ca.compact_attn_forward(qp, kp, vp, lay)
    out = torch.full_like(qp, float("nan"))
    stream = torch.cuda.Stream() if which == "side" else torch.cuda.default_stream()
    stream.wait_stream(torch.cuda.current_stream())
    handle = Handle()
    handle.cuda_stream = stream.cuda_stream
    ca.compact_attn_forward(qp, kp, vp, lay, out=out, stream=handle)
    nat = ca.compact_attn_forward_natural(q, k, v, lay, stream=handle)
    torch.cuda.synchronize()
    assert torch.equal(out, want)
    assert torch.equal(nat, ca.compact_attn_permute(want, lay, inverse=True))


def _whole_rows(qp, kp, vp, lay):
    """The C call without a workspace."""
    import ctypes
    out = torch.empty_like(qp)
    status = ca.load_library().compact_attn_forward(*(ctypes.c_void_p(x.data_ptr()) for x in (qp, kp, vp)), lay.handle, ctypes.c_void_p(out.data_ptr()),
                                                    ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert status == 0
    return out


def _split_layout_and_inputs():
    wl = make_workload("lend", 5, 32, 40, (2, 8, 8), 0, 2, 128, "bf16", [_GLOBAL] * 2)
    lay = build_layout(ca, wl)
    assert ca.compact_attn_layout_split(lay)[0] > 1 << 20
    qp, kp, vp = (ca.compact_attn_permute(x, lay) for x in make_qkv(wl, DEV))
    return lay, qp, kp, vp, ca.compact_attn_layout_split(lay)[0]


def test_split_rows_without_memory_for_a_workspace():
    """A call that has its output in hand is served also where the allocator has nothing left: with whole rows."""
    lay, qp, kp, vp, need = _split_layout_and_inputs()
    split, whole, out = ca.compact_attn_forward(qp, kp, vp, lay), _whole_rows(qp, kp, vp, lay), torch.empty_like(qp)
    assert not torch.equal(split, whole)
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    hogs = []
    torch.cuda.set_per_process_memory_fraction(0.0)
    try:
        for size in (need, need // 2, need // 4):         # what is left of the segments in use
            try:
                while True:
                    hogs.append(torch.empty(size, dtype=torch.uint8, device=DEV))
            except torch.cuda.OutOfMemoryError:
                pass
        ca.compact_attn_forward(qp, kp, vp, lay, out=out)
        torch.cuda.synchronize()
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)
    assert torch.equal(out, whole)
    del hogs
    assert torch.equal(ca.compact_attn_forward(qp, kp, vp, lay), whole)   # and the layout asks no more


def test_split_rows_in_a_capture_that_torch_does_not_run():
    """Memory lent by torch belongs to somebody else when such a graph is replayed: the call leaves its rows whole, and a replay
    writes nothing but the output."""
    import ctypes
    lay, qp, kp, vp, need = _split_layout_and_inputs()
    whole, out = _whole_rows(qp, kp, vp, lay), torch.full_like(qp, float("nan"))
    lib = ca.load_library()                               # the HIP runtime is among what it links
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        ca.compact_attn_forward(qp, kp, vp, lay)          # leaves a free block of the workspace's size
    torch.cuda.synchronize()
    handle, graph, launch = ctypes.c_void_p(stream.cuda_stream), ctypes.c_void_p(), ctypes.c_void_p()
    assert lib.hipStreamBeginCapture(handle, 0) == 0
    try:
        ca.compact_attn_forward(qp, kp, vp, lay, out=out, stream=stream)
    finally:
        assert lib.hipStreamEndCapture(handle, ctypes.byref(graph)) == 0
    assert lib.hipGraphInstantiate(ctypes.byref(launch), graph, None, None, ctypes.c_size_t(0)) == 0
    with torch.cuda.stream(stream):
        owned = [torch.full((need // 4,), 7.0, device=DEV) for _ in range(4)]   # one of them where the workspace would be
        for _ in range(3):
            out.fill_(float("nan"))
            assert lib.hipGraphLaunch(launch, handle) == 0
            assert torch.equal(out, whole)
    torch.cuda.synchronize()
    assert all(bool((x == 7.0).all()) for x in owned)
    assert lib.hipGraphExecDestroy(launch) == 0 and lib.hipGraphDestroy(graph) == 0


# ---------------------------------------------------------------- fp32 on the bf16 matrix instructions

_PLANE_LAUNCHES = [
    # tiles of 60, 64 and 128 tokens, padded down to a few tokens, and of 36 (units of 16, 16 and 4 tokens)
    ("2x2", 128, (9, 30, 25), (1, 8, 8), 0, 1),
    ("2x4", 128, (3, 17, 29), (1, 6, 10), 0, 2),
    ("1x4", 128, (3, 17, 29), (3, 3, 4), 0, 1),
    ("1x4", 128, (5, 13, 21), (2, 8, 8), 0, 1),
    ("2x2", 64, (7, 20, 33), (3, 3, 4), 0, 2),
    ("2x4", 64, (3, 17, 29), (1, 6, 10), 1, 4),
    ("2x2", 64, (9, 30, 25), (2, 8, 8), 0, 1),
    ("2x2", 32, (9, 30, 25), (1, 6, 10), 0, 4),
    ("2x4", 32, (7, 20, 33), (3, 3, 4), 0, 2),
    ("1x4", 32, (9, 30, 25), (1, 8, 8), 0, 1),
]


def _plane_problem(kernel, D, grid, tile, text_tiles, copies, batch=1):
    import dataclasses
    heads = [[(99, (99, 99), ABSENT)], *_EDGE_HEADS[1:]] * copies
    wl = dataclasses.replace(make_workload("planes", *grid, tile, text_tiles * tile[0] * tile[1] * tile[2], len(heads), D, "f32", heads), batch=batch)
    lay = build_layout(ca, wl)
    assert ca.compact_attn_layout_split(lay)[1] == "f32-planes-" + kernel
    return wl, lay


@pytest.mark.parametrize("kernel,D,grid,tile,text_tiles,copies", _PLANE_LAUNCHES)
def test_fp32_in_three_planes(kernel, D, grid, tile, text_tiles, copies):
    """fp32 operands as three bf16 values: against the oracle with peaked rows, whatever the padding slots and the workspace hold,
    and no further from it than the kernel on the fp32 matrix instructions (the C call without a workspace); the static
    entry point, a second stream and a replayed graph bit for bit."""
    import ctypes
    _say("fp32 planes", kernel, D, grid, tile)
    wl, lay = _plane_problem(kernel, D, grid, tile, text_tiles, copies)
    g, heads = geometry_of(wl), wl.heads
    q, k, v = make_qkv(wl, DEV, q_gain=2.0)
    qp, kp, vp = (ca.compact_attn_permute(x, lay) for x in (q, k, v))
    held = ca.compact_attn_permute(torch.ones_like(q), lay) != 0
    kp[~held] = float("nan")
    vp[~held] = float("nan")
    nbytes = ca.compact_attn_layout_split(lay)[0]
    del_me = torch.full((nbytes // 4,), float("nan"), device=DEV)  # the allocator's next block of that size
    del del_me
    out = ca.compact_attn_forward(qp, kp, vp, lay, out=torch.full_like(qp, float("nan")))
    assert torch.all(out[~held] == 0)
    got = ca.compact_attn_permute(out, lay, inverse=True)
    lib, stream = ca.load_library(), ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    other = torch.full_like(qp, float("nan"))
    assert lib.compact_attn_forward(*(ctypes.c_void_p(x.data_ptr()) for x in (qp, kp, vp)), lay.handle, ctypes.c_void_p(other.data_ptr()), stream) == 0
    before = ca.compact_attn_permute(other, lay, inverse=True)
    for h in range(4):
        want = OA.masked_attention(g, [heads[h]], *(to_f64(x[0, h])[None] for x in (q, k, v)))
        err = [np.linalg.norm(to_f64(x[0, h])[None] - want) for x in (got, before)]
        _say(h, compare(to_f64(got[0, h])[None], want, *tolerances("f32"), what=kernel), [e / max(np.linalg.norm(want), 1e-30) for e in err])
        assert err[0] <= err[1]
    again = torch.full_like(qp, float("nan"))
    assert nbytes <= 64 << 20 and torch.equal(ca.compact_attn_forward_static(qp, kp, vp, lay, out=again), out)
    side = torch.cuda.Stream()
    on_side = torch.full_like(qp, float("nan"))
    side.wait_stream(torch.cuda.current_stream())
    ca.compact_attn_forward(qp, kp, vp, lay, out=on_side, stream=side)
    with_main = ca.compact_attn_forward(qp, kp, vp, lay)            # may overlap with it
    torch.cuda.synchronize()
    assert torch.equal(on_side, out) and torch.equal(with_main, out)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        ca.compact_attn_forward(qp, kp, vp, lay, out=again)
    for rep in range(3):
        again.fill_(float("nan"))
        graph.replay()
        assert torch.equal(ca.compact_attn_forward(qp, kp, vp, lay), out)
        torch.cuda.synchronize()
        assert torch.equal(again, out), f"replay {rep}"


@pytest.mark.parametrize("kernel,D,grid,tile,text_tiles,copies", [_PLANE_LAUNCHES[i] for i in (0, 3, 5, 8, 9)])
@pytest.mark.parametrize("short", [False, True])
def test_fp32_in_three_planes_infinities(kernel, D, grid, tile, text_tiles, copies, short):
    """Infinities and NaN in q, k and v appear where the fp32 matrix instructions have them, also where the finite
    values are bf16 numbers (`short`), whose second and third parts hold nothing."""
    import ctypes
    wl, lay = _plane_problem(kernel, D, grid, tile, text_tiles, copies)
    q, k, v = make_qkv(wl, DEV)
    if short:
        q, k, v = (x.bfloat16().float() for x in (q, k, v))
    q, k, v = (ca.compact_attn_permute(x, lay) for x in (q, k, v))
    held = (ca.compact_attn_permute(torch.ones(q.shape[:2] + (wl.T * wl.H * wl.W + wl.n_text, D), device=DEV), lay) != 0)[0, 0, :, 0].nonzero().flatten()
    inf, nan = float("inf"), float("nan")
    some = held[torch.linspace(0, len(held) - 1, 7, device=DEV).long()]
    v[:, :, some[1], 3], v[:, :, some[2], 5], v[:, :, some[3], 5], v[:, :, some[4], 7] = inf, inf, -inf, nan
    v[:, :, held[-1], 9] = -inf
    v[:, :, some[1], 11] = torch.tensor(0x7f800001, dtype=torch.int32, device=DEV).view(torch.float32)  # a NaN with its payload in the lower half
    k[:, 0, some[5], 2] = -inf        # scores of both signs of infinity
    q[:, 0, some[0], 4] = inf
    q[:, 0, some[6], 4] = nan
    v[:, :, some[2], 6] = 0.0
    lib, stream = ca.load_library(), ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    want = torch.empty_like(q)
    assert lib.compact_attn_forward(*(ctypes.c_void_p(x.data_ptr()) for x in (q, k, v)), lay.handle, ctypes.c_void_p(want.data_ptr()), stream) == 0
    got = ca.compact_attn_forward(q, k, v, lay)
    padding = torch.ones(q.shape[2], dtype=torch.bool, device=DEV)
    padding[held] = False
    assert torch.all(got[:, :, padding] == 0)
    got, want = got[:, :, held], want[:, :, held]
    assert torch.equal(torch.isnan(got), torch.isnan(want)) and torch.isnan(want).any()
    assert torch.equal(torch.isinf(got), torch.isinf(want)) and torch.isinf(want).any()
    finite = ~torch.isnan(want)
    assert finite.any() and torch.allclose(got[finite], want[finite], rtol=1e-5, atol=1e-5)


@pytest.mark.parametrize("kernel,dense_kernel,D,grid,tile,copies", [
    ("2x4", "2x4", 128, (5, 13, 21), (1, 8, 8), 1),
    ("2x4", "2x2", 128, (3, 17, 29), (2, 8, 8), 1),
    ("2x2", "2x2", 128, (9, 30, 25), (3, 3, 4), 1),
    ("2x4", "2x4", 64, (5, 13, 21), (1, 8, 8), 1),
    ("1x4", "1x4", 32, (3, 17, 29), (1, 6, 10), 1),
    ("2x2", "2x2", 32, (5, 13, 21), (3, 3, 4), 2),
    ("2x4", "1x4", 32, (9, 30, 25), (1, 6, 10), 2),
])
def test_fp32_in_three_planes_with_two_batch_entries_and_dense(kernel, dense_kernel, D, grid, tile, copies):
    """Two batch entries of different values, on the sparse and the dense walk: against the oracle."""
    _say("fp32 planes, batch", kernel, dense_kernel, D, grid, tile)
    wl, lay = _plane_problem(kernel, D, grid, tile, 1, copies, batch=2)
    assert ca.compact_attn_layout_split(lay, dense=True)[1] == "f32-planes-" + dense_kernel
    g = geometry_of(wl)
    q, k, v = make_qkv(wl, DEV, q_gain=2.0)
    assert not torch.equal(k[0], k[1])
    x = [ca.compact_attn_permute(t, lay) for t in (q, k, v)]
    got, dense = (ca.compact_attn_permute(fn(*x, lay), lay, inverse=True) for fn in (ca.compact_attn_forward, ca.compact_attn_dense))
    for b in range(2):
        for h in range(4):
            one = [to_f64(t[b, h])[None] for t in (q, k, v)]
            compare(to_f64(got[b, h])[None], OA.masked_attention(g, [wl.heads[h]], *one), *tolerances("f32"), what=kernel)
            compare(to_f64(dense[b, h])[None], OA.dense_attention(*one), *tolerances("f32"), what=dense_kernel)


def _without_workspace(q, k, v, lay, call="forward"):
    """The C call without a workspace: the kernel on the fp32 matrix instructions."""
    import ctypes
    lib, out = ca.load_library(), torch.full_like(q, float("nan"))
    stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    assert getattr(lib, "compact_attn_" + call)(*(ctypes.c_void_p(x.data_ptr()) for x in (q, k, v)), lay.handle, ctypes.c_void_p(out.data_ptr()), stream) == 0
    return out


@pytest.mark.parametrize("kernel,D,grid,tile,text_tiles,copies", _PLANE_LAUNCHES)
@pytest.mark.parametrize("what", ["huge values", "infinite value of a small weight", "infinite query of small keys", "values near the smallest",
                                  "weights near the smallest", "large values"])
def test_fp32_in_three_planes_at_the_ends_of_the_range(kernel, D, grid, tile, text_tiles, copies, what):
    """Values that fp32 products take and three bf16 parts or a lagging exponent reference do not: as the fp32 matrix instructions give them."""
    _say("ends of the range", kernel, D, grid, tile, what)
    wl, lay = _plane_problem(kernel, D, grid, tile, text_tiles, copies)
    q, k, v = make_qkv(wl, DEV)
    tokens = q.shape[2]
    if what == "huge values":
        # scores rise from 0 to 7 bits over the walk, so that a reference of its beginning makes weights of up to 2^7; with weights of up to 1 the
        # sums stay below tokens * 2e38 / tokens
        q, k = 1e-3 * q, 1e-3 * k
        q[..., 0] = 1.0
        k[..., 0] = torch.linspace(0, 7 * math.log(2) * D ** 0.5, tokens, device=DEV)
        v = (v.abs().clamp(0.1, 1.0) * (2e38 / tokens)).contiguous()
    elif what == "infinite value of a small weight":
        # e^-70 of the largest weight of a row: 2^-101, whose second and third parts are below what a bf16 value can be
        q, k = 0.1 * q, 0.1 * k
        q[..., 0], k[..., 0] = 1.0, 0.0
        k[:, :, tokens // 2, 0] = -70.0 * D ** 0.5
        v[:, :, tokens // 2, 3] = float("inf")
    elif what == "infinite query of small keys":
        q[:, :, ::3, 4] = float("-inf")
        k[..., 4] = 2.0 ** -100
    elif what == "values near the smallest":
        # all rows of a head and channel alike: whatever their parts lose, the sums lose too
        v = ((1 + torch.rand(v.shape[0], v.shape[1], 1, D, device=DEV)) * 2.0 ** -122).expand(v.shape).contiguous()
    elif what == "large values":
        v = v.abs().clamp(0.1, 1.0) * 2.0 ** 95
    else:
        # one key has values, and e^-86 of the largest weight, 2^-124
        q, k, v = torch.zeros_like(q), torch.zeros_like(k), torch.zeros_like(v)
        q[..., 0] = 1.0
        k[:, :, tokens // 2, 0] = -86.0 * D ** 0.5
        v[:, :, tokens // 2] = 1e10 * (1 + torch.rand(v.shape[0], v.shape[1], D, device=DEV))
    q, k, v = (ca.compact_attn_permute(x, lay) for x in (q, k, v))
    want, got = (ca.compact_attn_permute(x, lay, inverse=True) for x in (_without_workspace(q, k, v, lay), ca.compact_attn_forward(q, k, v, lay)))
    if what == "huge values":
        assert torch.isfinite(want).all() and want.max() > 1e37 / tokens
    else:
        assert torch.isinf(want).any() == (what == "infinite value of a small weight") and not torch.isnan(want).any(), what
    assert torch.equal(torch.isnan(got), torch.isnan(want)) and torch.equal(torch.isinf(got), torch.isinf(want))
    finite = torch.isfinite(want)
    got, want = got[finite].double(), want[finite].double()
    assert want.abs().max() > 0 and (got - want).abs().max() <= 1e-5 * want.abs().max()


@pytest.mark.parametrize("kernel,D,grid,tile,text_tiles,copies", _PLANE_LAUNCHES)
def test_fp32_in_three_planes_of_the_least_favourable_values(kernel, D, grid, tile, text_tiles, copies):
    """Operands of 1 + 2^-7 - 2^-23: cut off after 8 and 16 bits they leave as much as there can be, and always to one side.  No further from
    the oracle than the kernel on the fp32 matrix instructions."""
    _say("least favourable values", kernel, D, grid, tile)
    wl, lay = _plane_problem(kernel, D, grid, tile, text_tiles, copies)
    g, heads = geometry_of(wl), wl.heads
    worst = 1 + 2.0 ** -7 - 2.0 ** -23
    q, k, v = (torch.where(x < 0, -worst, worst).float() for x in make_qkv(wl, DEV))
    q *= 8.0                                                           # scores of 8 on average
    p = [ca.compact_attn_permute(x, lay) for x in (q, k, v)]
    got, plain = (ca.compact_attn_permute(x, lay, inverse=True) for x in (ca.compact_attn_forward(*p, lay), _without_workspace(*p, lay)))
    for h in range(4):
        want = OA.masked_attention(g, [heads[h]], *(to_f64(x[0, h])[None] for x in (q, k, v)))
        err = [np.linalg.norm(to_f64(x[0, h])[None] - want) / max(np.linalg.norm(want), 1e-30) for x in (got, plain)]
        _say(h, err)
        assert err[0] <= err[1]


# ---------------------------------------------------------------- dense calls without the padding

@pytest.mark.parametrize("kernel,D,grid,tile,text_tiles,num_heads,batch", [
    # on copies: with and without rows split along the keys; the last: no tile is padded, but they do not pair up
    ("closed-one-tile", 128, (1, 45, 49), (2, 8, 8), 0, 4, 2),
    ("closed-one-tile", 128, (1, 45, 49), (1, 8, 8), 1, 1, 1),
    ("closed-one-tile", 64, (5, 17, 27), (1, 8, 8), 0, 12, 1),
    ("closed-one-tile", 64, (5, 17, 27), (2, 8, 8), 1, 1, 2),
    ("closed-ways-4x4", 64, (7, 20, 33), (2, 4, 8), 0, 1, 2),
    ("closed-ways-8x2", 128, (7, 20, 33), (2, 4, 8), 0, 3, 1),
    ("closed-ways-8x4", 128, (4, 32, 32), (1, 8, 8), 1, 1, 1),
    # in place: tiles of 64 tokens two by two
    ("one-tile", 128, (4, 32, 32), (1, 8, 8), 0, 3, 2),
    ("ways-4x4", 128, (4, 32, 32), (1, 8, 8), 0, 3, 1),
    ("ways-4x4", 64, (4, 32, 32), (1, 8, 8), 0, 3, 1),
])
def test_dense_calls_without_the_padding(kernel, D, grid, tile, text_tiles, num_heads, batch):
    """Dense calls on the tokens alone: against the oracle with peaked rows, whatever the padding slots and the workspace hold; a
    second stream and a replayed graph bit for bit; the C call without a workspace to within the rounding of bf16."""
    import ctypes
    import dataclasses
    _say("closed-up dense", kernel, D, grid, tile, num_heads, batch)
    n_text = text_tiles * tile[0] * tile[1] * tile[2]
    wl = dataclasses.replace(make_workload("closed", *grid, tile, n_text, num_heads, D, "bf16", [[]] * num_heads), batch=batch)
    lay = build_layout(ca, wl)
    nbytes, name = ca.compact_attn_layout_split(lay, dense=True)
    assert kernel in (name, ca.compact_attn_layout_kernel(lay, dense=True)) and (not kernel.startswith("closed") or name == kernel)
    q, k, v = make_qkv(wl, DEV, q_gain=3.0)
    qp, kp, vp = (ca.compact_attn_permute(x, lay) for x in (q, k, v))
    held = ca.compact_attn_permute(torch.ones_like(q), lay) != 0
    lib, stream = ca.load_library(), ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    again = torch.full_like(qp, float("nan"))
    assert lib.compact_attn_dense(*(ctypes.c_void_p(x.data_ptr()) for x in (qp, kp, vp)), lay.handle, ctypes.c_void_p(again.data_ptr()), stream) == 0
    for x in (qp, kp, vp):
        x[~held] = float("nan")                                      # on copies they are never read
    del_me = torch.full((nbytes // 2,), float("nan"), dtype=torch.bfloat16, device=DEV)
    del del_me
    out = ca.compact_attn_dense(qp, kp, vp, lay, out=torch.full_like(qp, float("nan")))
    assert torch.all(out[~held] == 0)
    compare(to_f64(again), to_f64(out), *tolerances("bf16"), what="without a workspace")
    got = ca.compact_attn_permute(out, lay, inverse=True)
    for b in range(batch):
        _say(b, compare(to_f64(got[b]), OA.dense_attention(to_f64(q[b]), to_f64(k[b]), to_f64(v[b])), *tolerances("bf16"), what=kernel))
    side = torch.cuda.Stream()
    on_side = torch.full_like(qp, float("nan"))
    side.wait_stream(torch.cuda.current_stream())
    ca.compact_attn_dense(qp, kp, vp, lay, out=on_side, stream=side)
    with_main = ca.compact_attn_dense(qp, kp, vp, lay)               # may overlap with it
    torch.cuda.synchronize()
    assert torch.equal(on_side, out) and torch.equal(with_main, out)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        ca.compact_attn_dense(qp, kp, vp, lay, out=again)
    for rep in range(3):
        again.fill_(float("nan"))
        graph.replay()
        assert torch.equal(ca.compact_attn_dense(qp, kp, vp, lay), out)
        torch.cuda.synchronize()
        assert torch.equal(again, out), f"replay {rep}"


# ---------------------------------------------------------------- calls through the extension

def test_calls_with_other_than_the_usual_arguments():
    """What the extension does not take is served, or refused with its reason, by the binding: given outputs and streams, subclasses and
    tensors under a torch function mode, wrong types, shapes and strides, freed layouts."""
    from torch.overrides import TorchFunctionMode

    class Sub(torch.Tensor):
        pass

    class Mode(TorchFunctionMode):
        seen = 0

        def __torch_function__(self, func, types, args=(), kwargs=None):
            Mode.seen += 1
            return func(*args, **(kwargs or {}))

    wl = make_workload("usual", 3, 9, 17, (1, 8, 8), 64, 2, 64, "bf16", [[(1, (1, 1), ABSENT)]] * 2)
    lay = build_layout(ca, wl)
    q, k, v = make_qkv(wl, DEV)
    x = [ca.compact_attn_permute(t, lay) for t in (q, k, v)]
    want, back = ca.compact_attn_forward(*x, lay), ca.compact_attn_permute(x[0], lay, inverse=True)
    assert torch.equal(back, q) and want.shape == x[0].shape and want.dtype == torch.bfloat16 and not want.requires_grad
    assert torch.equal(ca.compact_attn_forward(*x, lay, out=torch.empty_like(want)), want)
    assert torch.equal(ca.compact_attn_forward(*x, lay, stream=torch.cuda.current_stream()), want)
    assert torch.equal(ca.compact_attn_forward(x[0].clone().requires_grad_(), *x[1:], lay), want)
    sub = ca.compact_attn_permute(q.as_subclass(Sub), lay)
    assert type(sub) is Sub and torch.equal(sub.as_subclass(torch.Tensor), x[0])
    with Mode():
        got = ca.compact_attn_forward(*x, lay)
    assert Mode.seen > 0 and torch.equal(got, want)
    mass = ca.compact_attn_tile_mass(x[0], x[1], lay)
    assert torch.equal(mass, ca.compact_attn_tile_mass(x[0], x[1], lay, out=torch.empty_like(mass))) and mass.dtype == torch.float32
    for bad in (x[0].float(), x[0][:, :, :-1], x[0].transpose(0, 1).contiguous(), x[0].transpose(2, 3).contiguous().transpose(2, 3), x[0].cpu()):
        with pytest.raises(ValueError):
            ca.compact_attn_forward(bad, x[1], x[2], lay)
        with pytest.raises(ValueError):
            ca.compact_attn_permute(bad, lay, inverse=True)
        with pytest.raises(ValueError):
            ca.compact_attn_tile_mass(bad, x[1], lay)
    lay.free()
    with pytest.raises(ca.CompactAttnError):
        ca.compact_attn_forward(*x, lay)


def test_a_call_that_the_library_fails_is_made_once():
    """The status of the first call is what the program sees: another call could succeed, or enqueue work a second time.  Functions that
    report an error in the place of the library's."""
    import ctypes
    from paper_2508_12969_amd import _calls, binding
    wl = make_workload("once", 3, 9, 17, (1, 8, 8), 64, 2, 64, "bf16", [[(1, (1, 1), ABSENT)]] * 2)
    lay = build_layout(ca, wl)
    q, k, v = make_qkv(wl, DEV)
    x = [ca.compact_attn_permute(t, lay) for t in (q, k, v)]
    made = []
    vp, i32 = ctypes.c_void_p, ctypes.c_int32
    forms = ([vp, vp, vp, i32, vp], *[[vp] * 6] * 4, [vp, vp, vp, vp, vp, i32, vp, ctypes.c_int64, vp], [vp] * 5)
    stubs = [ctypes.CFUNCTYPE(ctypes.c_int, *form)(lambda *a, n=n: made.append(n) or ca.binding.CA_ERR_HIP) for n, form in enumerate(forms)]
    try:
        _calls.bind(*(ctypes.cast(f, vp).value for f in stubs), torch._C._cuda_getDevice, torch._C._cuda_getCurrentRawStream,
                    torch._C._cuda_isCurrentStreamCapturing, binding._check)
        for call in (lambda: ca.compact_attn_permute(q, lay), lambda: ca.compact_attn_forward(*x, lay), lambda: ca.compact_attn_forward_natural(q, k, v, lay),
                     lambda: ca.compact_attn_dense(*x, lay), lambda: ca.compact_attn_forward_static(*x, lay), lambda: ca.compact_attn_tile_mass(*x[:2], lay)):
            made.clear()
            with pytest.raises(ca.CompactAttnError) as e:
                call()
            assert e.value.status == ca.binding.CA_ERR_HIP and len(made) == 1
    finally:
        binding._calls_bound = False
        binding._make_calls(lay)
    assert torch.equal(ca.compact_attn_permute(ca.compact_attn_permute(q, lay), lay, inverse=True), q)


@pytest.mark.parametrize("call", ["planes", "closed"])
@pytest.mark.parametrize("given_out", [False, True])
def test_a_passing_shortage_of_memory_for_planes_and_copies(call, given_out):
    """Calls that find no memory for their workspace run without one, say so once, ask for it once each time that they do, and
    have it again when there is memory."""
    import warnings
    dtype = "f32" if call == "planes" else "bf16"
    wl = make_workload("short", 9, 30, 25, (1, 8, 8), 0, 4, 128, dtype, [_GLOBAL] * 4)
    lay = build_layout(ca, wl)
    fn = ca.compact_attn_forward if call == "planes" else ca.compact_attn_dense
    need, kernel = ca.compact_attn_layout_split(lay, dense=call == "closed")
    assert kernel.startswith("f32-planes-" if call == "planes" else "closed-")
    x = [ca.compact_attn_permute(t, lay) for t in make_qkv(wl, DEV)]
    want, plain = fn(*x, lay), _without_workspace(*x, lay, call="forward" if call == "planes" else "dense")
    assert not torch.equal(want, plain)
    outs = [torch.empty_like(want) for _ in range(8)]
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    hogs, asked = [], []
    torch.cuda.set_per_process_memory_fraction(0.0)
    try:
        for size in (need, need // 2, need // 4):         # what is left of the segments in use
            try:
                while True:
                    hogs.append(torch.empty(size, dtype=torch.uint8, device=DEV))
            except torch.cuda.OutOfMemoryError:
                pass
        with warnings.catch_warnings(record=True) as said:
            warnings.simplefilter("always")
            for i in range(8):
                out = outs[i] if given_out else None
                if not given_out:
                    outs[i] = None                       # room for a result, not for the workspace
                before = torch.cuda.memory_stats()["num_ooms"]
                outs[i] = fn(*x, lay, out=out)
                asked.append(torch.cuda.memory_stats()["num_ooms"] - before)
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)
    torch.cuda.synchronize()
    assert asked == [1, 0, 1, 0, 0, 0, 1, 0]              # one call without, then three, seven
    assert len(said) == 1 and "no memory for a workspace" in str(said[0].message) and said[0].filename == __file__
    assert all(torch.equal(o, plain) for o in outs)
    del hogs
    later = [fn(*x, lay) for _ in range(7)]               # six of the seven are left
    assert all(torch.equal(o, plain) for o in later[:6]) and torch.equal(later[6], want)
