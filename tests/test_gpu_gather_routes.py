"""The two routes of a paged gather and of the in-place rotation of wide bands around their sizes:
one launch in plan order, or (640 MiB gathered, 512 MiB rotated, read and written) the row table in
destination order and the physical-order sort.  Every layer of a pool holds the same rows, so the
layer count alone takes a small splice across the bound: layer 0 is compared with the oracle and all
other layers with layer 0, bit for bit."""

import random

import numpy as np
import pytest
import torch

import workloads as W
from oracle import splice_oracle as O
from tests import test_gpu_paged as TP
from tests.parity_util import assert_rows_match, host, oracle_plane

pytestmark = pytest.mark.gpu

MIB = 1 << 20


def _workload(page, kind, layers, dtype):
    # sequence 0: shift -7 (gathered unless pages hold one token), then a whole number of pages;
    # sequence 1: growth and two more directives a few rows apart; sequence 2: untouched
    dirs = [W.Dir(40, 60, 13, seq=0), W.Dir(600, 600 + 2 * 48 + 7, 14, seq=0),
            W.Dir(0, 5, 300, seq=1), W.Dir(9, 10, 1, seq=1), W.Dir(500, 700, 3, seq=1)]
    planes = {"mla": [W.mla_plane()], "mla_half": [W.PlaneDesc((576,), 1, 576, 512, 64, 1, 10000.0)],
              "gqa8": W.gqa_planes(heads=8, dim=128)}[kind]
    return W.Workload(f"routes_{kind}", layers, dtype, planes, dirs, [1300, 1300, 70], page_size=page, seed=page)


def _counts(wl, flags):
    """Gathered rows, fresh pages, re-used pages; bytes gathered and rotated, read and written."""
    P, fresh, remaps = wl.page_size, 0, 0
    for p in O.plan_paged(wl.seq_lens, TP._odirs(wl), P, remap=not flags):
        fresh += sum(k == O.ASSEMBLE for k in p.kinds)
        remaps += sum(k == O.REMAP for k in p.kinds)
    both = 2 * wl.n_layers * P * (4 if wl.dtype == "f32" else 2)
    return (fresh * P, fresh, remaps, both * fresh * sum(p.row_elems for p in wl.planes),
            both * remaps * sum(p.n_heads * p.rot_dim for p in wl.planes))


@pytest.mark.parametrize("page,kind,flags,layers,dtype", [
    (1, "mla", 1, 3, "bf16"), (1, "mla", 1, 320, "bf16"), (3, "mla", 0, 3, "bf16"), (3, "mla", 0, 320, "bf16"),
    (16, "mla_half", 0, 3, "bf16"), (16, "mla_half", 0, 320, "bf16"), (16, "gqa8", 0, 3, "bf16"),
    (16, "gqa8", 0, 120, "bf16"), (1, "gqa8", 0, 3, "bf16"), (1, "gqa8", 0, 80, "bf16"), (3, "mla", 0, 160, "f32"),
    (16, "gqa8", 0, 60, "f32"), (1, "gqa8", 0, 40, "f32"), (2, "gqa8", 0, 240, "bf16"), (2, "gqa8", 0, 120, "f32")])
def test_both_routes(page, kind, flags, layers, dtype):
    from paper_2606_01065_amd import leyline as L
    wl = _workload(page, kind, 1, dtype)
    plans = O.plan_paged(wl.seq_lens, TP._odirs(wl), page, remap=not flags)
    spare = sum(k == O.ASSEMBLE for p in plans for k in p.kinds) + 3
    pools1, bt, free, stubs1 = W.alloc_paged(wl, "cuda:0", spare_pages=spare)
    before, bt_h, free_h = [host(p) for p in pools1], host(bt), host(free)
    stubs_h = [[host(s).reshape(1, s.shape[1], p.row_elems) for s, p in zip(per, wl.planes)] for per in stubs1]
    wl.n_layers = layers
    rows, fresh, remaps, moved, rotated = _counts(wl, flags)
    if layers > 3 and kind == "gqa8" and page < 3:                    # sorted, in 2 KB rows or more
        assert remaps >= 64 and rotated >= 512 * MIB
    elif layers > 3:                                                  # row table in destination order
        assert rows > 1024 and fresh >= 64 and moved >= 640 * MIB
    else:
        assert moved < 640 * MIB and rotated < 512 * MIB
    print(f"[case] routes page={page} {kind}/{dtype} layers={layers} gather {moved >> 20} MiB rotate {rotated >> 20} MiB",
          flush=True)
    pools = [p.expand(layers, *p.shape[1:]).contiguous() for p in pools1]
    stubs = [[s.expand(layers, *s.shape[1:]).contiguous() for s in per] for per in stubs1]
    bt_out, freed, new_lens = TP._run_gpu(L, wl, pools, bt, free, stubs, flags=flags)
    planes = [oracle_plane(p) for p in wl.planes]
    flat = [b.reshape(b.shape[0], b.shape[1], b.shape[2], -1) for b in before]
    want, want_bt, want_lens, want_freed = O.splice_paged(flat, planes, dtype, bt_h, wl.seq_lens, TP._odirs(wl),
                                                          stubs_h, list(free_h), page, remap=not flags)
    assert new_lens == want_lens
    assert np.array_equal(host(bt_out), want_bt)
    assert list(host(freed)) == want_freed
    for pi, plane in enumerate(planes):
        got = host(pools[pi][:1]).reshape(want[pi].shape)
        assert_rows_match(got, want[pi], plane, dtype, what=f"routes page={page} {kind} plane {pi}")
        assert torch.equal(pools[pi], pools[pi][:1].expand_as(pools[pi])), "layers differ"


SHORT_KINDS = {"mla": [W.mla_plane()], "mla_split": W.mla_split_planes(), "gqa8": W.gqa_planes(heads=8, dim=128),
               "mla_half": [W.PlaneDesc((576,), 1, 576, 512, 64, 1, 10000.0)], "heads96": W.gqa_planes(heads=3, dim=96)}


@pytest.mark.parametrize("kind,dtype", [("mla", "bf16"), ("mla_split", "bf16"), ("gqa8", "bf16"), ("mla_half", "bf16"),
                                        ("heads96", "bf16"), ("mla", "f32"), ("mla_split", "f32")])
def test_many_short_spans(kind, dtype):
    """Gathers whose spans (replacements and rows of one shift) hold one to a few rows, so that nearly every
    workgroup lies across several, in one launch: whole pools against the oracle."""
    from paper_2606_01065_amd import leyline as L
    rng = random.Random(f"{kind}/{dtype}")
    for page, flags in ((1, 0), (1, 1), (3, 0), (16, 0)):
        dirs = []
        for b in range(2):
            at = rng.randint(0, 9)
            for _ in range(60):
                e = at + rng.randint(0, 3)
                dirs.append(W.Dir(at, e, rng.randint(0, 3), seq=b))
                at = e + rng.choice([1, 1, 2, 5, 12])
        lens = [max(d.span_end for d in dirs if d.seq == b) + 7 for b in range(2)]
        wl = W.Workload(f"short_{kind}", 3, dtype, SHORT_KINDS[kind], dirs, lens, page_size=page, seed=page)
        plans = O.plan_paged(lens, TP._odirs(wl), page, remap=not flags)
        print(f"[case] short spans {kind}/{dtype} page={page} flags={flags} lens={lens}", flush=True)
        pools, bt, free, stubs = W.alloc_paged(wl, "cuda:0", spare_pages=3 + sum(k == O.ASSEMBLE for p in plans for k in p.kinds))
        before, bt_h, free_h = [host(p) for p in pools], host(bt), host(free)
        stubs_h = [[host(s).reshape(3, s.shape[1], p.row_elems) for s, p in zip(per, wl.planes)] for per in stubs]
        bt_out, freed, new_lens = TP._run_gpu(L, wl, pools, bt, free, stubs, flags=flags)
        planes = [oracle_plane(p) for p in wl.planes]
        flat = [b.reshape(b.shape[0], b.shape[1], b.shape[2], -1) for b in before]
        want, want_bt, want_lens, want_freed = O.splice_paged(flat, planes, dtype, bt_h, lens, TP._odirs(wl), stubs_h,
                                                              list(free_h), page, remap=not flags)
        assert new_lens == want_lens
        assert np.array_equal(host(bt_out), want_bt)
        assert list(host(freed)) == want_freed
        for pi, plane in enumerate(planes):
            assert_rows_match(host(pools[pi]).reshape(want[pi].shape), want[pi], plane, dtype,
                              what=f"short spans {kind} page={page} plane {pi}")


@pytest.mark.parametrize("kind,page,dtype", [("mla", 1, "bf16"), ("mla", 3, "f32"), ("mla", 64, "bf16"), ("mla_half", 1, "bf16"),
                                             ("gqa8", 1, "bf16"), ("heads96", 16, "bf16"), ("heads96", 64, "f32")])
def test_short_spans_in_a_row_table(kind, page, dtype):
    """More than 1,024 rows in short spans over many layers: resolved once into a row table (without an order
    of its pages below 64 pages).  Every layer holds the same rows, as in test_both_routes."""
    from paper_2606_01065_amd import leyline as L
    rng, dirs, at, layers = random.Random(f"{kind}/{page}"), [], 3, 61
    for _ in range(400):
        e = at + rng.randint(0, 3)
        dirs.append(W.Dir(at, e, rng.randint(0, 3)))
        at = e + rng.choice([1, 2, 5, 9])
    wl = W.Workload(f"table_{kind}", 1, dtype, SHORT_KINDS[kind], dirs, [at], page_size=page, seed=page)
    plans = O.plan_paged(wl.seq_lens, TP._odirs(wl), page, remap=False)
    fresh = sum(k == O.ASSEMBLE for p in plans for k in p.kinds)
    assert fresh * page > 1024 and (fresh < 64) == (page == 64), fresh
    print(f"[case] row table {kind}/{dtype} page={page} rows={fresh * page} spans of {len(dirs)} edits", flush=True)
    pools1, bt, free, stubs1 = W.alloc_paged(wl, "cuda:0", spare_pages=fresh + 3)
    before, bt_h, free_h = [host(p) for p in pools1], host(bt), host(free)
    stubs_h = [[host(s).reshape(1, s.shape[1], p.row_elems) for s, p in zip(per, wl.planes)] for per in stubs1]
    wl.n_layers = layers
    pools = [p.expand(layers, *p.shape[1:]).contiguous() for p in pools1]
    stubs = [[s.expand(layers, *s.shape[1:]).contiguous() for s in per] for per in stubs1]
    bt_out, freed, new_lens, ws = TP._run_gpu(L, wl, pools, bt, free, stubs, flags=1, ws_fill=0x5a)
    table = ws[-(24 * fresh * page + (4 * fresh if fresh >= 64 else 0)):]      # the end of the workspace
    assert not bool((table == 0x5a).all()), "no row table was written"
    planes = [oracle_plane(p) for p in wl.planes]
    flat = [b.reshape(b.shape[0], b.shape[1], b.shape[2], -1) for b in before]
    want, want_bt, want_lens, want_freed = O.splice_paged(flat, planes, dtype, bt_h, wl.seq_lens, TP._odirs(wl), stubs_h,
                                                          list(free_h), page, remap=False)
    assert new_lens == want_lens
    assert np.array_equal(host(bt_out), want_bt)
    assert list(host(freed)) == want_freed
    for pi, plane in enumerate(planes):
        assert_rows_match(host(pools[pi][:1]).reshape(want[pi].shape), want[pi], plane, dtype,
                          what=f"row table {kind} page={page} plane {pi}")
        assert torch.equal(pools[pi], pools[pi][:1].expand_as(pools[pi])), "layers differ"
