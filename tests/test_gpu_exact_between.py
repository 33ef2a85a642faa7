"""The exact library's bf16 rounding where the nearest-even float of an fp64 result lies exactly between
two bf16 values, so that rounding it again would lose which side the fp64 value was on: enough values
that every layout's rotation meets such floats, and all stored values bit-identical to the oracle."""

import numpy as np
import pytest
import torch

import workloads as W
from oracle import splice_oracle as O
from tests.parity_util import host, oracle_plane

pytestmark = pytest.mark.gpu

KINDS = {"interleaved": W.mla_plane(), "lanes": W.gqa_planes(heads=8, dim=128)[0],
         "two_chunk": W.gqa_planes(heads=3, dim=96)[0]}


@pytest.mark.parametrize("kind", list(KINDS))
def test_floats_between_two_bf16_values(kind):
    from paper_2606_01065_amd import leyline as L
    desc, n, delta = KINDS[kind], 6144, -777
    wl = W.Workload(f"between_{kind}", 3, "bf16", [desc], [], [n], capacity=n, seed=31)
    (t,), _ = W.alloc_contig(wl, "cuda:0")
    plane = oracle_plane(desc)
    before = host(t).reshape(wl.n_layers, n, -1)
    want = before.copy()
    between = 0
    for cols in plane.rotary_columns():
        x = O.decode(before[..., cols], O.BF16)
        r = O.rotate(x.reshape(-1, len(cols)), np.full(x.size // len(cols), delta), plane.frequencies(), plane.style)
        f = r.astype(np.float32)
        between += int((((f.view(np.uint32) & 0xffff) == 0x8000) & (f != r)).sum())
        want[..., cols] = O.encode(r, O.BF16).reshape(x.shape)
    assert between > 4, between
    L.use_library(True)
    try:
        cache = L.make_cache([L.PlaneSpec(t, desc.n_heads, desc.head_stride or desc.row_elems, desc.rot_offset,
                                          desc.rot_dim, desc.style, desc.base)])
        L.leyline_rotate_delta(cache, delta, row0=0, n_rows=n)
        torch.cuda.synchronize()
    finally:
        L.use_library(False)
    assert np.array_equal(host(t).reshape(want.shape), want), f"{kind}: {between} floats in between"
