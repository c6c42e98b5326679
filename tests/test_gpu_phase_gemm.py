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
from paper_2607_18631_amd import moe
from paper_2607_18631_amd import workloads as wl

from parity_util import REL_TOL, dev_bits, rel_fro

pytestmark = pytest.mark.gpu

COUNTS = [0, 1, 31, 32, 33, 64, 65, 97, 129, 160, 191, 225, 255, 256, 257, 319, 321]


@pytest.mark.parametrize("rows_hint, F", [(600, 136), (700, 640)], ids=["tile256", "tile320"])
@pytest.mark.parametrize("d", [64, 72, 128, 192, 200, 456])
def test_segment_ends_and_slice_counts(rows_hint, F, d):
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
