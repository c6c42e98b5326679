"""The large-tile grouped GEMM (256- and 320-row tiles) at the edges of its schedule, through
moe_grouped_ffn against the fp64 oracle: segments ending in every 32-row block of a tile (two to five
phases per K slice, an odd number of live blocks), and reductions of one, two, three and more 64-wide
K slices, with and without a partial last slice.  The counts stay on the device, so one call whose
capacity asks for large tiles runs every segment length.  bf16 results of a bf16 activation and
float32 sums: rel. Frobenius 5e-3 per expert, as everywhere; rows outside the segments stay as they were.
"""
import numpy as np
import pytest
import torch

import oracle
from oracle import moe_backward as obwd
from paper_2607_18631_amd import moe
from paper_2607_18631_amd import workloads as wl

from parity_util import REL_TOL, dev_bits, rel_fro

pytestmark = pytest.mark.gpu

COUNTS = [0, 1, 31, 32, 33, 64, 65, 97, 129, 160, 191, 225, 255, 256, 257, 319, 321] * 2
# reductions of one to four or more K slices, without and with a partial last one
WIDTHS = [64, 128, 192, 256] + [40, 72, 136, 200]
# (capacity per expert, d, F, tile of the up-projection, of the down-projection); test_tile_rule.py checks the tiles
SEGMENTS = ([(600, d, 136, "256x256", "256x256" if d >= 320 else "256x128") for d in WIDTHS + [456]] +
            [(700, 1024, F, "256x256", "256x256") for F in WIDTHS + [640]] +
            [(280, d, 640, "320x256", "128x256") for d in WIDTHS + [456]] +
            [(300, 1792, F, "128x256", "320x256") for F in WIDTHS])
FEW_TILES = [(3001, 200, 264), (513, 64, 8), (1000, 1032, 40)]


@pytest.mark.parametrize("case", SEGMENTS, ids=str)
def test_segment_ends_and_slice_counts(case):
    rows_hint, d, F, _, _ = case
    E = len(COUNTS)
    sh = wl.MoEShape(T=rows_hint * E, d=d, E=E, top_k=1, F=F, E_local=E)
    offs = np.concatenate([[0], np.cumsum(COUNTS)]).astype(np.int32)
    n = int(offs[-1])
    rng = np.random.default_rng(d)
    draw = lambda shape, std: wl.f32_to_bf16_bits((rng.standard_normal(shape) * std).astype(np.float32))
    x, w13, w2 = draw((n, d), 1.0), draw((E, 2 * F, d), d ** -0.5), draw((E, d, F), F ** -0.5)
    x_perm = torch.zeros(sh.capacity, d, dtype=torch.bfloat16, device="cuda")
    x_perm[:n] = moe.to_device_bf16(x)
    y = torch.full((sh.capacity, d), -7.0, dtype=torch.bfloat16, device="cuda")
    print(f"[phase gemm] rows_hint {rows_hint} d {d} F {F}", flush=True)
    moe.moe_grouped_ffn(sh, x_perm, torch.from_numpy(offs).cuda(), moe.to_device_bf16(w13), moe.to_device_bf16(w2), y,
                        moe.alloc_workspace(sh, moe.MOE_WS_FFN))
    torch.cuda.synchronize()
    assert (y[n:] == -7.0).all()
    got = oracle.bf16_to_f64(dev_bits(y[:n]))
    for e in range(E):
        a, b = offs[e], offs[e + 1]
        if a < b:
            ref = oracle.swiglu_ffn(oracle.bf16_to_f64(x[a:b]), oracle.bf16_to_f64(w13[e]), oracle.bf16_to_f64(w2[e]))
            assert rel_fro(got[a:b], ref) <= REL_TOL, (e, COUNTS[e])


@pytest.mark.parametrize("T, d, F", FEW_TILES)
def test_few_large_tiles_take_small_ones(T, d, F):
    """One dense segment whose 256-row tiles would cover at most a quarter of the chip runs on 64-row tiles:
    the same results, bit for bit, as the rows in groups of at most 128 (the small tiles of such groups)."""
    rng = np.random.default_rng(T)
    draw = lambda shape, std: moe.to_device_bf16(wl.f32_to_bf16_bits((rng.standard_normal(shape) * std).astype(np.float32)))
    x, w13, w2 = draw((T, d), 1.0), draw((1, 2 * F, d), d ** -0.5), draw((1, d, F), F ** -0.5)
    outs = []
    for E in (1, -(-T // 100)):
        sh = wl.MoEShape(T=T, d=d, E=E, top_k=1, F=F, E_local=E)
        offs = np.minimum(np.arange(E + 1) * (T if E == 1 else 100), T).astype(np.int32)
        y = torch.full((T, d), float("nan"), dtype=torch.bfloat16, device="cuda")
        print(f"[phase gemm] small launch T {T} d {d} F {F} groups {E}", flush=True)
        moe.moe_grouped_ffn(sh, x, torch.from_numpy(offs).cuda(), w13.expand(E, -1, -1).contiguous(),
                            w2.expand(E, -1, -1).contiguous(), y, moe.alloc_workspace(sh, moe.MOE_WS_FFN))
        torch.cuda.synchronize()
        outs.append(dev_bits(y))
    ref = oracle.swiglu_ffn(*(oracle.bf16_to_f64(dev_bits(t)) for t in (x, w13[0], w2[0])))
    assert rel_fro(oracle.bf16_to_f64(outs[0]), ref) <= REL_TOL
    assert np.array_equal(outs[0], outs[1])


BACKWARD_COUNTS = [0, 5, 193, 250, 64, 256, 65, 300, 128, 129, 192, 420] * 4
# (capacity per expert, d, F, tile of dX); test_tile_rule.py checks the tile
BACKWARD = [(200, 1000, 504, "256x256"), (280, 1024, 512, "320x256")]


@pytest.mark.parametrize("rows_hint, d, F, tile", BACKWARD)
def test_backward_slice_counts_between_tiles(rows_hint, d, F, tile):
    """moe_grouped_ffn_backward on 48 segments of none to seven 64-row slices in turn, with more weight-gradient
    tiles than workgroups: a tile's last slices issue the next tile's first ones when both have three or
    more, and every change between such tiles, shorter ones and empty ones follows another.  Output
    edges cut tiles in both directions, and the row products' reductions end in a partial slice; the second case's
    dX runs on 320-row tiles (which take no partial slice).  Each
    gradient within rel. Frobenius 5e-3 (bf16 results of at most two bf16 intermediates)."""
    _check_backward(BACKWARD_COUNTS, rows_hint, d, F)


# (capacity per expert, d, F): short segments into rows of whole and of part lines
SHORT = [(20, 512, 256), (60, 512, 256), (20, 520, 264), (120, 520, 264)]


@pytest.mark.parametrize("rows_hint, d, F", SHORT)
def test_backward_of_short_segments(rows_hint, d, F):
    """The same on segments of at most two slices, empty ones among them, whose weight gradients run on the ring kernel
    or the phase kernel (test_tile_rule.py checks that both do)."""
    counts = [min(c, rows_hint * 3 // 2) for c in [0, 1, 7, 8, 0, 63, 64, 65, 31, 33, 127, 128]] * 9
    _check_backward(counts, rows_hint, d, F)


def _check_backward(counts, rows_hint, d, F):
    E = len(counts)
    sh = wl.MoEShape(T=rows_hint * E, d=d, E=E, top_k=1, F=F, E_local=E)
    offs = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    n = int(offs[-1])
    rng = np.random.default_rng(3)
    draw = lambda shape, std: wl.f32_to_bf16_bits((rng.standard_normal(shape, dtype=np.float32) * np.float32(std)))
    x, dy = draw((n, d), 1.0), draw((n, d), 1.0)
    w13, w2 = draw((E, 2 * F, d), d ** -0.5), draw((E, d, F), F ** -0.5)
    rows = lambda b: torch.cat([moe.to_device_bf16(b), torch.zeros(sh.capacity - n, d, dtype=torch.bfloat16, device="cuda")])
    nan = lambda *s: torch.full(s, float("nan"), dtype=torch.bfloat16, device="cuda")
    dx, dw13, dw2 = nan(sh.capacity, d), nan(E, 2 * F, d), nan(E, d, F)
    print("[phase gemm] backward", flush=True)
    moe.moe_grouped_ffn_backward(sh, rows(x), torch.from_numpy(offs).cuda(), moe.to_device_bf16(w13),
                                 moe.to_device_bf16(w2), rows(dy), dx, dw13, dw2,
                                 moe.alloc_workspace(sh, moe.MOE_WS_FFN_BWD))
    torch.cuda.synchronize()
    f64 = lambda t: oracle.bf16_to_f64(dev_bits(t))
    for e in range(E):
        a, b = offs[e], offs[e + 1]
        if a == b:
            assert not f64(dw13[e]).any() and not f64(dw2[e]).any(), e
            continue
        ref = obwd.swiglu_ffn_backward(oracle.bf16_to_f64(x[a:b]), oracle.bf16_to_f64(w13[e]),
                                       oracle.bf16_to_f64(w2[e]), oracle.bf16_to_f64(dy[a:b]))
        for name, got, want in zip(("dx", "dw13", "dw2"), (dx[a:b], dw13[e], dw2[e]), ref):
            assert rel_fro(f64(got), want) <= REL_TOL, (name, e, counts[e])
