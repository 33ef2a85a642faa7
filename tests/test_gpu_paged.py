"""GPU parity of the paged splice (through the C ABI) against the CPU oracle: whole pools on
small ragged cases, and block tables, freed lists and sampled rows at the full batched and
multi-directive sizes."""

import random

import numpy as np
import pytest
import torch

import workloads as W
from oracle import splice_oracle as O
from tests.parity_util import (angle_tables, assert_bands_rotated, assert_rows_match, bits, host,
                               oracle_plane, rotary_mask)

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.fixture(scope="module")
def L():
    from paper_2606_01065_amd import leyline
    return leyline


def _run_gpu(L, wl, pools, bt, free, stubs, flags=0, ws_fill=None):
    """(new block tables, freed list, new lengths) of a checked call, and its workspace where ws_fill says
    what byte it holds before."""
    specs = [L.PlaneSpec(t, p.n_heads, p.head_stride or p.row_elems, p.rot_offset, p.rot_dim,
                         p.style, p.base) for p, t in zip(wl.planes, pools)]
    cache = L.make_cache(specs, paged=True)
    dirs = L.make_directives([dict(span_start=d.span_start, span_end=d.span_end, stub=stubs[j],
                                   seq=d.seq, stub_len=d.stub_len, mode=d.mode)
                              for j, d in enumerate(wl.dirs)])
    new_lens, fresh, n_freed, ws_bytes = L.leyline_paged_query(cache, wl.seq_lens, bt.shape[1], dirs,
                                                                len(wl.dirs), flags)
    bt_out = torch.full_like(bt, -7)
    freed = torch.full((max(1, n_freed),), -7, dtype=torch.int32, device=DEV)
    ws = torch.empty(max(256, ws_bytes), dtype=torch.uint8, device=DEV)
    if ws_fill is not None:
        ws.fill_(ws_fill)
    status = torch.zeros(1, dtype=torch.int32, device=DEV)
    got_lens, got_fresh, got_freed = L.leyline_splice_paged(cache, wl.seq_lens, bt, bt_out, dirs,
                                                            len(wl.dirs), free, freed, ws,
                                                            device_status=status, flags=flags)
    torch.cuda.synchronize()
    assert (got_lens, got_fresh, got_freed) == (new_lens, fresh, n_freed)
    assert int(status.item()) == 0
    if ws_fill is not None:
        return bt_out, freed[:n_freed], new_lens, ws
    return bt_out, freed[:n_freed], new_lens


def _odirs(wl):
    return [O.Directive(d.span_start, d.span_end, d.stub_len, seq=d.seq, mode=d.mode) for d in wl.dirs]


def _random_workload(rng, page, kind, dtype, max_len=None):
    n_seqs = rng.randint(1, 4)
    lens, dirs = [], []
    for b in range(n_seqs):
        n = rng.randint(0, max_len if max_len is not None else 5 * page + 3)
        lens.append(n)
        k = rng.randint(0, 3)
        cuts = sorted(rng.sample(range(n + 1), min(2 * k, n + 1)))
        for i in range(0, len(cuts) - 1, 2):
            s, e = cuts[i], cuts[i + 1]
            r = rng.choice([0, 1, e - s, rng.randint(0, 2 * (e - s) + 3), max(0, e - s - page),
                            e - s + page])
            dirs.append(W.Dir(s, e, r, seq=b))
    if kind == "mla":
        planes = [W.mla_plane()]
    elif kind == "mla_neox":      # half-split rows of 72 chunks: partners in the same wavefront
        planes = [W.PlaneDesc((576,), 1, 576, 512, 64, 1, 10000.0)]
    elif kind == "heads96":       # heads across wavefront ends: two-chunk units, gathered and in place
        planes = W.gqa_planes(heads=3, dim=96)
    elif kind == "heads80":
        planes = W.gqa_planes(heads=10, dim=80)
    elif kind == "gqa8":          # 2 KB rotated per row: re-used pages can rotate in physical order
        planes = W.gqa_planes(heads=8, dim=128)
    elif kind == "mla_split":     # K_pe and c_kv in two arrays: a plane that is all rotary band
        planes = W.mla_split_planes()
    elif kind == "four":          # four planes, rotary bands of both access classes
        planes = [W.mla_plane(), W.PlaneDesc((2, 128), 2, 128, 0, 128, 1, 500000.0), W.PlaneDesc((256,)),
                  W.PlaneDesc((64,), 1, 64, 32, 32, 0, 10000.0)]
    else:
        planes = W.gqa_planes(heads=2, dim=128)
    return W.Workload(f"paged_{kind}", 2, dtype, planes, dirs, lens, page_size=page,
                      seed=rng.randint(0, 10 ** 6))


@pytest.mark.parametrize("kind,dtype", [("mla", "bf16"), ("gqa", "bf16"), ("mla", "f32"),
                                        ("gqa", "f32"), ("mla_neox", "bf16"), ("four", "bf16"),
                                        ("heads96", "bf16"), ("heads80", "bf16"), ("heads96", "f32")])
def test_small_random_paged_whole_pool(L, kind, dtype):
    rng = random.Random({"mla": 97, "gqa": 98, "mla_neox": 99, "four": 100, "heads96": 102,
                         "heads80": 104}[kind] + (dtype == "f32"))
    for page in (1, 4, 16, 64):
        for ci in range(8):
            wl = _random_workload(rng, page, kind, dtype)
            print(f"[case] paged {kind}/{dtype} page={page} case={ci} lens={wl.seq_lens} dirs={wl.dirs}",
                  flush=True)
            pools, bt, free, stubs = W.alloc_paged(wl, DEV, spare_pages=3)
            before = [host(p) for p in pools]
            bt_h, free_h = host(bt), host(free)
            stubs_h = [[host(s).reshape(wl.n_layers, s.shape[1], p.row_elems) for s, p in zip(per, wl.planes)]
                       for per in stubs]
            bt_out, freed, new_lens = _run_gpu(L, wl, pools, bt, free, stubs)
            planes = [oracle_plane(p) for p in wl.planes]
            flat = [b.reshape(b.shape[0], b.shape[1], b.shape[2], -1) for b in before]
            want, want_bt, want_lens, want_freed = O.splice_paged(
                flat, planes, dtype, bt_h, wl.seq_lens, _odirs(wl), stubs_h, list(free_h), page)
            assert new_lens == want_lens
            assert np.array_equal(host(bt_out), want_bt)
            assert list(host(freed)) == want_freed
            for pi, plane in enumerate(planes):
                got = host(pools[pi]).reshape(want[pi].shape)
                assert_rows_match(got, want[pi], plane, dtype, what=f"page={page} case={ci} plane={pi}")


@pytest.mark.parametrize("kind", ["mla", "gqa", "heads96", "heads80"])
def test_page_sizes_not_powers_of_two(L, kind):
    """Pages of 3 and 48 rows: page and row index arithmetic without power-of-two shortcuts;
    whole pools against the oracle."""
    rng = random.Random({"mla": 401, "gqa": 402, "heads96": 403, "heads80": 404}[kind])
    for page in (3, 48):
        for ci in range(5):
            wl = _random_workload(rng, page, kind, "bf16")
            print(f"[case] page={page} {kind} case={ci} lens={wl.seq_lens} dirs={wl.dirs}", flush=True)
            pools, bt, free, stubs = W.alloc_paged(wl, DEV, spare_pages=3)
            before = [host(p) for p in pools]
            bt_h, free_h = host(bt), host(free)
            stubs_h = [[host(s).reshape(wl.n_layers, s.shape[1], p.row_elems) for s, p in zip(per, wl.planes)]
                       for per in stubs]
            bt_out, freed, new_lens = _run_gpu(L, wl, pools, bt, free, stubs)
            planes = [oracle_plane(p) for p in wl.planes]
            flat = [b.reshape(b.shape[0], b.shape[1], b.shape[2], -1) for b in before]
            want, want_bt, want_lens, want_freed = O.splice_paged(
                flat, planes, "bf16", bt_h, wl.seq_lens, _odirs(wl), stubs_h, list(free_h), page)
            assert new_lens == want_lens
            assert np.array_equal(host(bt_out), want_bt)
            assert list(host(freed)) == want_freed
            for pi, plane in enumerate(planes):
                got = host(pools[pi]).reshape(want[pi].shape)
                assert_rows_match(got, want[pi], plane, "bf16", what=f"page={page} case={ci} plane={pi}")


@pytest.mark.parametrize("kind", ["mla", "gqa"])
def test_forget_and_copy_on_write_whole_pool(L, kind):
    """Trailing FORGET directives (prefix trims) and copy-on-write plans (no old page written):
    whole pools against the oracle, and under copy-on-write every old page byte-identical."""
    rng = random.Random({"mla": 301, "gqa": 302}[kind])
    for page in (1, 4, 16):
        for ci in range(6):
            wl = _random_workload(rng, page, kind, "bf16", max_len=300 if page == 1 else None)
            if rng.random() < 0.6:                                   # a FORGET ends some sequences
                dirs = list(wl.dirs)
                for b, n in enumerate(wl.seq_lens):
                    mine = [d for d in dirs if d.seq == b]
                    lo = mine[-1].span_end if mine else 0
                    if lo <= n and rng.random() < 0.6:
                        s = rng.randint(lo, n)
                        dirs.append(W.Dir(s, rng.randint(s, n), 0, seq=b, mode=1))
                dirs.sort(key=lambda d: (d.seq, d.span_start, d.mode))
                wl = W.Workload(wl.name, wl.n_layers, wl.dtype, wl.planes, dirs, wl.seq_lens,
                                page_size=page, seed=wl.seed)
            cow = ci % 2 == 0
            print(f"[case] forget/cow {kind} page={page} case={ci} cow={cow} lens={wl.seq_lens} "
                  f"dirs={wl.dirs}", flush=True)
            # the pool must hold the fresh pages of the copy-on-write plan
            plans = O.plan_paged(wl.seq_lens, _odirs(wl), page, remap=not cow)
            extra = sum(k == O.ASSEMBLE for p in plans for k in p.kinds) + 3
            pools, bt, free, stubs = W.alloc_paged(wl, DEV, spare_pages=extra)
            before = [host(p) for p in pools]
            bt_h, free_h = host(bt), host(free)
            stubs_h = [[host(s).reshape(wl.n_layers, s.shape[1], p.row_elems) for s, p in zip(per, wl.planes)]
                       for per in stubs]
            bt_out, freed, new_lens = _run_gpu(L, wl, pools, bt, free, stubs,
                                               flags=L.PAGED_COPY_ON_WRITE if cow else 0)
            planes = [oracle_plane(p) for p in wl.planes]
            flat = [b.reshape(b.shape[0], b.shape[1], b.shape[2], -1) for b in before]
            want, want_bt, want_lens, want_freed = O.splice_paged(
                flat, planes, "bf16", bt_h, wl.seq_lens, _odirs(wl), stubs_h, list(free_h), page,
                remap=not cow)
            assert new_lens == want_lens
            assert np.array_equal(host(bt_out), want_bt)
            assert list(host(freed)) == want_freed
            old_pages = sorted({int(bt_h[b, k]) for b, n in enumerate(wl.seq_lens)
                                for k in range(O.pages_for(n, page))})
            for pi, plane in enumerate(planes):
                got = host(pools[pi])
                assert_rows_match(got.reshape(want[pi].shape), want[pi], plane, "bf16",
                                  what=f"page={page} case={ci} plane={pi}")
                if cow:
                    assert np.array_equal(got[:, old_pages], before[pi][:, old_pages])


def test_out_of_pool_pages_are_flagged_and_skipped(L):
    """A block-table entry of a REMAP page and the first free-list entry point outside the pool:
    the kernels flag LEYLINE_STATUS_BAD_PAGE and skip that page's rows; every other page equals
    the oracle's result on the uncorrupted inputs, and the two skipped destinations keep their
    contents."""
    P = 4
    dirs = [W.Dir(8, 12, 0, seq=0), W.Dir(10, 13, 1, seq=1)]     # seq 0: shift -4 (REMAP); seq 1: -2
    wl = W.Workload("bad_pages", 2, "bf16", [W.mla_plane()], dirs, [40, 40], page_size=P, seed=77)
    pools, bt, free, stubs = W.alloc_paged(wl, DEV, spare_pages=3)
    before = host(pools[0])
    bt_h, free_h = host(bt), host(free)
    plans = O.plan_paged(wl.seq_lens, _odirs(wl), P)
    assert plans[0].kinds[4] == O.REMAP and plans[0].sources[4] == 5
    assert O.ASSEMBLE in plans[1].kinds
    cap = pools[0].shape[1]
    remap_page, fresh_page = int(bt_h[0, 5]), int(free_h[0])
    bad_bt, bad_free = bt.clone(), free.clone()
    bad_bt[0, 5] = cap + 7
    bad_free[0] = -5
    print(f"[case] out-of-pool pages: remap page {remap_page} -> {cap + 7}, fresh page {fresh_page} -> -5",
          flush=True)
    specs = [L.PlaneSpec(pools[0], 1, 576, 512, 64, L.ROPE_INTERLEAVED, 10000.0)]
    cache = L.make_cache(specs, paged=True)
    ldirs = L.make_directives([dict(span_start=d.span_start, span_end=d.span_end, stub=stubs[j], seq=d.seq,
                                    stub_len=d.stub_len) for j, d in enumerate(wl.dirs)])
    new_lens, fresh, n_freed, ws_bytes = L.leyline_paged_query(cache, wl.seq_lens, bt.shape[1], ldirs, 2)
    bt_out = torch.full_like(bt, -7)
    freed = torch.full((max(1, n_freed),), -7, dtype=torch.int32, device=DEV)
    ws = torch.empty(max(256, ws_bytes), dtype=torch.uint8, device=DEV)
    status = torch.zeros(1, dtype=torch.int32, device=DEV)
    L.leyline_splice_paged(cache, wl.seq_lens, bad_bt, bt_out, ldirs, 2, bad_free, freed, ws, device_status=status)
    torch.cuda.synchronize()
    assert int(status.item()) == L.STATUS_BAD_PAGE
    stubs_h = [[host(s).reshape(wl.n_layers, s.shape[1], 576) for s in per] for per in stubs]
    plane = oracle_plane(wl.planes[0])
    want, want_bt, _, _ = O.splice_paged([before.reshape(before.shape[0], before.shape[1], P, -1)], [plane], "bf16",
                                         bt_h, wl.seq_lens, _odirs(wl), stubs_h, list(free_h), P)
    got = host(pools[0]).reshape(want[0].shape)
    skipped = [remap_page, fresh_page]
    keep = [pg for pg in range(cap) if pg not in skipped]
    assert_rows_match(got[:, keep], want[0][:, keep], plane, "bf16", what="pages with valid indices")
    b = before.reshape(got.shape)
    assert np.array_equal(got[:, skipped], b[:, skipped])
    got_bt = host(bt_out)
    assert got_bt[0, 4] == cap + 7                 # tables carry the entries they were given
    want_bt = want_bt.copy()
    want_bt[0, 4] = cap + 7
    want_bt[want_bt == fresh_page] = -5
    assert np.array_equal(got_bt, want_bt)


@pytest.mark.parametrize("kind", ["mla", "gqa"])
@pytest.mark.parametrize("last_stub", [256, 257])
def test_gathers_of_1024_and_1025_rows(L, kind, last_stub):
    """Token-slot cache, four directives: the downstream slots form four REMAP runs whose
    boundaries fall inside workgroups, and the replacements total 1024 rows or 1025, the first count
    whose route depends on more than itself (few spans and few bytes: one launch, like 1024); whole
    pool against the oracle."""
    dirs = [W.Dir(500, 600, 256), W.Dir(1500, 1510, 256), W.Dir(2500, 2700, 256), W.Dir(4000, 4001, last_stub)]
    planes = [W.mla_plane()] if kind == "mla" else W.gqa_planes(heads=2, dim=128)
    wl = W.Workload(f"slots_{kind}", 2, "bf16", planes, dirs, [5000], page_size=1, seed=61 + last_stub)
    plans = O.plan_paged(wl.seq_lens, _odirs(wl), 1)
    assert sum(k == O.ASSEMBLE for k in plans[0].kinds) == 768 + last_stub
    print(f"[case] slots {kind} gather rows={768 + last_stub}", flush=True)
    pools, bt, free, stubs = W.alloc_paged(wl, DEV, spare_pages=3)
    before = [host(p) for p in pools]
    bt_h, free_h = host(bt), host(free)
    stubs_h = [[host(s).reshape(wl.n_layers, s.shape[1], p.row_elems) for s, p in zip(per, wl.planes)]
               for per in stubs]
    bt_out, freed, new_lens = _run_gpu(L, wl, pools, bt, free, stubs)
    oplanes = [oracle_plane(p) for p in wl.planes]
    flat = [b.reshape(b.shape[0], b.shape[1], b.shape[2], -1) for b in before]
    want, want_bt, want_lens, want_freed = O.splice_paged(
        flat, oplanes, "bf16", bt_h, wl.seq_lens, _odirs(wl), stubs_h, list(free_h), 1)
    assert new_lens == want_lens
    assert np.array_equal(host(bt_out), want_bt)
    assert list(host(freed)) == want_freed
    for pi, plane in enumerate(oplanes):
        got = host(pools[pi]).reshape(want[pi].shape)
        assert_rows_match(got, want[pi], plane, "bf16", what=f"slots {kind} plane {pi}")


@pytest.mark.parametrize("kind,dtype", [("mla", "bf16"), ("gqa", "bf16"), ("mla", "f32"),
                                        ("mla_neox", "bf16"), ("four", "bf16"), ("gqa8", "bf16"),
                                        ("gqa8", "f32"), ("heads96", "bf16"), ("heads80", "f32")])
def test_token_slot_paged_whole_pool(L, kind, dtype):
    """Page sizes 1 and 2 (token-slot caches) with sequences long enough that the in-place
    rotation of remapped slots spans many workgroups and ends in a ragged one, in plan order (these
    calls rotate too little to sort their slots first; test_gpu_gather_routes.py has ones that do)."""
    rng = random.Random({"mla": 197, "gqa": 198, "mla_neox": 199, "four": 200, "gqa8": 201, "heads96": 203,
                         "heads80": 205}[kind] + (dtype == "f32"))
    for page in (1, 2):
        for ci in range(3):
            wl = _random_workload(rng, page, kind, dtype, max_len=900)
            print(f"[case] slots {kind}/{dtype} page={page} case={ci} lens={wl.seq_lens} dirs={wl.dirs}",
                  flush=True)
            pools, bt, free, stubs = W.alloc_paged(wl, DEV, spare_pages=3)
            before = [host(p) for p in pools]
            bt_h, free_h = host(bt), host(free)
            stubs_h = [[host(s).reshape(wl.n_layers, s.shape[1], p.row_elems) for s, p in zip(per, wl.planes)]
                       for per in stubs]
            bt_out, freed, new_lens = _run_gpu(L, wl, pools, bt, free, stubs)
            planes = [oracle_plane(p) for p in wl.planes]
            flat = [b.reshape(b.shape[0], b.shape[1], b.shape[2], -1) for b in before]
            want, want_bt, want_lens, want_freed = O.splice_paged(
                flat, planes, dtype, bt_h, wl.seq_lens, _odirs(wl), stubs_h, list(free_h), page)
            assert new_lens == want_lens
            assert np.array_equal(host(bt_out), want_bt)
            assert list(host(freed)) == want_freed
            for pi, plane in enumerate(planes):
                got = host(pools[pi]).reshape(want[pi].shape)
                assert_rows_match(got, want[pi], plane, dtype, what=f"page={page} case={ci} plane={pi}")


def _sample_positions(rng, wl, b, new_len, extra=24):
    """New positions to check in sequence b: boundaries of every stub and segment, the ends,
    page edges around them, and random positions."""
    pts = {0, new_len - 1}
    shift = 0
    for d in (d for d in wl.dirs if d.seq == b):
        a = d.span_start + shift
        for q in (a - 1, a, a + d.stub_len - 1, a + d.stub_len, a + d.stub_len + 1):
            pts.add(q)
            pts.add((q // wl.page_size) * wl.page_size)
            pts.add((q // wl.page_size) * wl.page_size + wl.page_size - 1)
        shift += d.stub_len - (d.span_end - d.span_start)
    pts.update(rng.randrange(max(1, new_len)) for _ in range(extra))
    return sorted(q for q in pts if 0 <= q < new_len)


class _EveryRow:
    """Checks every row of every sequence, plane and layer at full size by properties:
    non-rotary elements equal their source row's bit for bit, replacement rows equal the
    replacement bit for bit, rows with shift 0 are bit-identical, and every member of every
    rotary pair of a moved row lies within 1.5 ulps of the exact rotation of its stored input by
    its angle phi (assert_bands_rotated: fp64 products with cos phi and sin phi taken from the
    oracle once per distinct shift; implied by the oracle bar of assert_rows_match).
    In three whole layers (first, middle, last) every row's rotary bands are also compared
    element by element with the oracle's rotation of its source bands (Eq. "rotate"), at the
    parity bar of assert_rows_match.
    The rotary bands of all source rows are snapshotted on the device before the call; their
    non-rotary elements are read after it, where they still are (fresh pages are disjoint from
    old ones, a re-used page changes only its rotary bands, copy-on-write writes no old page)."""

    def __init__(self, wl, pools, bt_h, stubs):
        P = wl.page_size
        odirs = _odirs(wl)
        glob = {}
        for j, d in enumerate(wl.dirs):
            glob.setdefault(d.seq, []).append(j)
        stub_base = np.cumsum([0] + [d.stub_len for d in wl.dirs])
        q_old, q_stub, a_old, shift, stub_row, seq_old, seq_stub = ([] for _ in range(7))
        for b, n in enumerate(wl.seq_lens):
            src = O.row_sources(n, [d for d in odirs if d.seq == b])
            kind = np.array([x[0] == "old" for x in src], dtype=bool)
            a = np.array([x[1] for x in src], dtype=np.int64)
            c = np.array([x[2] for x in src], dtype=np.int64)
            q = np.arange(len(src), dtype=np.int64)
            q_old.append(q[kind]); a_old.append(a[kind]); shift.append(c[kind])
            seq_old.append(np.full(int(kind.sum()), b))
            loc = a[~kind]
            stub_row.append(np.array([stub_base[glob[b][j]] for j in loc], dtype=np.int64) + c[~kind])
            q_stub.append(q[~kind]); seq_stub.append(np.full(int((~kind).sum()), b))
        cat = lambda xs: np.concatenate(xs) if xs else np.zeros(0, dtype=np.int64)
        self.q_old, self.a_old, self.shift, self.seq_old = map(cat, (q_old, a_old, shift, seq_old))
        self.q_stub, self.stub_row, self.seq_stub = map(cat, (q_stub, stub_row, seq_stub))
        self.P, self.wl = P, wl
        dev = lambda x: torch.from_numpy(np.ascontiguousarray(x, dtype=np.int64)).to(DEV)
        self.op, self.oo = dev(bt_h[self.seq_old, self.a_old // P]), dev(self.a_old % P)
        self.planes = [oracle_plane(desc) for desc in wl.planes]
        self.rot = [torch.from_numpy(rotary_mask(pl)).to(DEV) for pl in self.planes]
        # rotary bands of every source row, before the call
        self.before = [torch.stack([pools[pi][layer][self.op, self.oo].reshape(len(self.a_old), self.planes[pi].row_elems)[:, self.rot[pi]]
                                    for layer in range(wl.n_layers)])
                       if self.planes[pi].rot_dim else None for pi in range(len(pools))]
        moved = self.shift != 0
        self.angles = [angle_tables(pl, self.shift[moved], DEV) if pl.rot_dim else None for pl in self.planes]
        self.stubs = [torch.cat([s[pi].reshape(wl.n_layers, s[pi].shape[1], self.planes[pi].row_elems)
                                 for s in stubs], dim=1)
                      if len(stubs) else None for pi in range(len(pools))]

    def check(self, pools, bt_out_h, exact=False):
        P, wl = self.P, self.wl
        dev = lambda x: torch.from_numpy(np.ascontiguousarray(x, dtype=np.int64)).to(DEV)
        np_, no = dev(bt_out_h[self.seq_old, self.q_old // P]), dev(self.q_old % P)
        sp, so = dev(bt_out_h[self.seq_stub, self.q_stub // P]), dev(self.q_stub % P)
        moved = dev(self.shift != 0).bool()
        oracle_layers = {0, wl.n_layers // 2, wl.n_layers - 1}
        rows = 0
        for pi, plane in enumerate(self.planes):
            rot = self.rot[pi]
            for layer in range(wl.n_layers):
                pool = pools[pi][layer]
                got = pool[np_, no].reshape(len(self.a_old), plane.row_elems)
                src = pool[self.op, self.oo].reshape(len(self.a_old), plane.row_elems)
                assert torch.equal(bits(got[:, ~rot]), bits(src[:, ~rot])), f"plane {pi} layer {layer}: non-rotary"
                if self.stubs[pi] is not None:
                    gs = pool[sp, so].reshape(len(self.q_stub), plane.row_elems)
                    assert torch.equal(bits(gs), bits(self.stubs[pi][layer, dev(self.stub_row)])), \
                        f"plane {pi} layer {layer}: replacement rows"
                if not plane.rot_dim:
                    continue
                g, b0 = got[:, rot], self.before[pi][layer]
                assert torch.equal(bits(g[~moved]), bits(b0[~moved])), f"plane {pi} layer {layer}: shift-0 rows"
                assert_bands_rotated(b0[moved], g[moved], self.angles[pi], wl.dtype, f"plane {pi} layer {layer}")
                if layer in oracle_layers:
                    self._against_oracle(plane, host(b0), host(g), f"plane {pi} layer {layer}", exact)
            rows += len(self.a_old) + len(self.q_stub)
        print(f"[info] every row checked by properties: {rows} rows x {wl.n_layers} layers; rotary bands "
              f"of layers {sorted(oracle_layers)} against the oracle", flush=True)

    def _against_oracle(self, plane, before, got, what, exact=False):
        """Every row's rotary bands (the plane's rotary selection: each head's band back to back,
        i.e. a plane of n_heads bands of rot_dim elements) against the oracle's R(shift) of the
        bands the row had before the call, one oracle call per distinct shift."""
        bands = O.Plane(row_elems=plane.n_heads * plane.rot_dim, n_heads=plane.n_heads,
                        head_stride=plane.rot_dim, rot_offset=0, rot_dim=plane.rot_dim,
                        style=plane.style, base=plane.base, freqs=plane.freqs)
        want = np.empty_like(before)
        for c in np.unique(self.shift):
            sel = self.shift == c
            want[sel] = O.rotate_rows(before[sel], int(c), bands, self.wl.dtype)
        if exact:     # fp64 pair arithmetic: the oracle's values bit for bit
            assert np.array_equal(got.view(np.uint8), want.view(np.uint8)), f"{what}: rotary bands differ from the oracle"
        else:
            assert_rows_match(got, want, bands, self.wl.dtype, inputs=before, what=f"{what}: rotary bands vs oracle")


def _check_sampled(L, wl, seed, exact=False):
    rng = random.Random(seed)
    print(f"[case] {wl.name}: allocating and filling the pool", flush=True)
    pools, bt, free, stubs = W.alloc_paged(wl, DEV)
    P = wl.page_size
    odirs = _odirs(wl)
    bt_h, free_h = host(bt), host(free)
    cow = bool(wl.paged_flags & L.PAGED_COPY_ON_WRITE)
    want_bt, want_lens, want_freed, plans = O.paged_tables(bt_h, wl.seq_lens, odirs, list(free_h), P,
                                                           remap=not cow)
    # sampled outputs and their sources (old rows read before the call)
    samples = []   # (seq, new position, kind, source index, shift)
    for b, n in enumerate(wl.seq_lens):
        mine = [d for d in odirs if d.seq == b]
        src = O.row_sources(n, mine)
        for q in _sample_positions(rng, wl, b, want_lens[b]):
            s = src[q]
            samples.append((b, q) + tuple(s))
    pages_old = torch.tensor([bt_h[b, a // P] if kind == "old" else 0 for b, q, kind, a, c in samples],
                             dtype=torch.long, device=DEV)
    offs_old = torch.tensor([a % P if kind == "old" else 0 for b, q, kind, a, c in samples],
                            dtype=torch.long, device=DEV)
    before = [host(p[:, pages_old, offs_old]) for p in pools]          # [L, S, *row]
    stubs_h = [[host(s) for s in per] for per in stubs]
    dir_index = {}
    for j, d in enumerate(wl.dirs):
        dir_index.setdefault(d.seq, []).append(j)
    every = _EveryRow(wl, pools, bt_h, stubs)
    print(f"[case] {wl.name}: splicing on the GPU", flush=True)
    bt_out, freed, new_lens = _run_gpu(L, wl, pools, bt, free, stubs, flags=wl.paged_flags)
    assert new_lens == want_lens
    assert np.array_equal(host(bt_out), want_bt)
    assert list(host(freed)) == want_freed
    referenced = host(bt_out)[host(bt_out) >= 0]
    assert len(np.unique(referenced)) == len(referenced)
    bt_out_h = host(bt_out)
    pages_new = torch.tensor([bt_out_h[x[0], x[1] // P] for x in samples], dtype=torch.long, device=DEV)
    offs_new = torch.tensor([x[1] % P for x in samples], dtype=torch.long, device=DEV)
    print(f"[case] {wl.name}: comparing {len(samples)} sampled rows x {wl.n_layers} layers", flush=True)
    for pi, desc in enumerate(wl.planes):
        plane = oracle_plane(desc)
        got = host(pools[pi][:, pages_new, offs_new]).reshape(wl.n_layers, len(samples), -1)
        old = before[pi].reshape(wl.n_layers, len(samples), -1)
        want = np.empty_like(got)
        for i, (b, q, kind, a, c) in enumerate(samples):
            if kind == "old":
                want[:, i] = O.rotate_rows(old[:, i], c, plane, wl.dtype)
            else:
                j = dir_index[b][a]
                want[:, i] = stubs_h[j][pi].reshape(wl.n_layers, -1, plane.row_elems)[:, c]
        if exact:
            assert np.array_equal(got.view(np.uint8), want.view(np.uint8)), f"{wl.name} plane {pi}: sampled rows differ"
        else:
            assert_rows_match(got, want, plane, wl.dtype, what=f"{wl.name} plane {pi}")
        if cow:   # the old rows the samples came from are untouched
            old_now = host(pools[pi][:, pages_old, offs_old]).reshape(wl.n_layers, len(samples), -1)
            from_old = [i for i, x in enumerate(samples) if x[2] == "old"]
            assert np.array_equal(old_now[:, from_old], old[:, from_old])
    every.check(pools, bt_out_h, exact)
    del every
    return pools, bt, bt_out, new_lens, plans


def test_mla_dsv3_paged_b64_full(L):
    wl = W.mla_dsv3_paged_b64()
    pools, bt, bt_out, new_lens, plans = _check_sampled(L, wl, seed=11)
    kinds = [k for p in plans for k in p.kinds]
    print(f"[info] pages: identity={kinds.count(O.IDENTITY)} remap={kinds.count(O.REMAP)} "
          f"assemble={kinds.count(O.ASSEMBLE)}", flush=True)


def test_mla_dsv3_paged_131k_full_and_sequential(L):
    """Eight directives in one call; sampled rows against the one-call oracle, and whole
    sequences of two layers against sequential application of the directives."""
    wl = W.mla_dsv3_paged_131k()
    P = wl.page_size
    # snapshot two layers of the logical sequence before the call
    layers = (0, wl.n_layers - 1)
    pools, bt, free, stubs = W.alloc_paged(wl, DEV)
    n = wl.seq_lens[0]
    idx = torch.arange(n, device=DEV)
    bt_row = bt[0].long()
    pages, offs = bt_row[idx // P], idx % P
    logical_before = {l: host(pools[0][l, pages, offs]) for l in layers}
    stubs_h = [host(s[0]) for s in stubs]
    bt_out, freed, new_lens = _run_gpu(L, wl, pools, bt, free, stubs)
    n_new = new_lens[0]
    idx = torch.arange(n_new, device=DEV)
    bt_row = bt_out[0].long()
    plane = oracle_plane(wl.planes[0])
    odirs = [O.Directive(d.span_start, d.span_end, d.stub_len) for d in wl.dirs]
    for l in layers:
        print(f"[case] sequential reference, layer {l}", flush=True)
        got = host(pools[0][l, bt_row[idx // P], idx % P])
        cache = logical_before[l][None]
        st = [s[l][None] for s in stubs_h]
        want, nw = O.splice_sequential(cache, n, odirs, st, plane, wl.dtype)
        assert nw == n_new
        assert_rows_match(got, want[0, :n_new], plane, wl.dtype, what=f"sequential layer {l}")
    del pools
    torch.cuda.empty_cache()
    _check_sampled(L, wl, seed=13)


def test_token_slot_copy_on_write_full(L):
    """The full-size MLA token-slot splice with copy-on-write: every downstream token is rotated
    into a fresh slot, the prefix keeps its slots, and no old slot is written."""
    wl = W.mla_dsv3_slots_cow_32k()
    pools, bt, bt_out, new_lens, plans = _check_sampled(L, wl, seed=19)
    kinds = [k for p in plans for k in p.kinds]
    d = wl.dirs[0]
    assert kinds.count(O.ASSEMBLE) == d.stub_len + wl.seq_lens[0] - d.span_end
    assert kinds.count(O.REMAP) == 0
    assert kinds.count(O.IDENTITY) == d.span_start


def _whole_page_shift_131k(flags):
    base = W.mla_dsv3_paged_131k()
    # replacements sized so that every shift is a whole number of pages: downstream pages are
    # re-used in place (REMAP) unless copy-on-write asks for fresh ones
    dirs = [W.Dir(d.span_start, d.span_end, (d.span_end - d.span_start) % 64) for d in base.dirs]
    odirs = [O.Directive(d.span_start, d.span_end, d.stub_len) for d in dirs]
    assert any(k == O.REMAP for k in O.plan_paged(base.seq_lens, odirs, 64)[0].kinds)
    return W.Workload("mla_dsv3_paged_131k_page_shifts", base.n_layers, base.dtype, base.planes, dirs,
                      base.seq_lens, page_size=base.page_size, paged_flags=flags, seed=base.seed)


def test_paged_131k_whole_page_shifts_full(L):
    """The 8-directive 131K-token splice with whole-page shifts: about 1400 downstream pages keep
    their physical page and have their K_pe bands rotated in place."""
    pools, bt, bt_out, new_lens, plans = _check_sampled(L, _whole_page_shift_131k(0), seed=29)
    kinds = [k for p in plans for k in p.kinds]
    assert kinds.count(O.REMAP) > 1000


def test_paged_131k_copy_on_write_full(L):
    """The 8-directive 131K-token splice on 64-token pages with copy-on-write: no page is re-used
    with a shift (whole-page shifts are assembled too) and no old page is written."""
    pools, bt, bt_out, new_lens, plans = _check_sampled(L, _whole_page_shift_131k(L.PAGED_COPY_ON_WRITE), seed=23)
    kinds = [k for p in plans for k in p.kinds]
    assert kinds.count(O.REMAP) == 0 and kinds.count(O.ASSEMBLE) > 0


@pytest.mark.parametrize("name", ["mla_dsv3_slots_32k", "gqa_llama3_8b_slots_16k", "mla_dsv3_slots_split_32k"])
def test_token_slot_splice_full(L, name):
    """Full-size splices on token-slot caches: every downstream token keeps its slot (its
    rotary band is rotated in place), only the replacement tokens take fresh slots.  The split
    MLA layout keeps K_pe and c_kv in separate arrays."""
    wl = W.WORKLOADS[name]()
    pools, bt, bt_out, new_lens, plans = _check_sampled(L, wl, seed=17)
    kinds = [k for p in plans for k in p.kinds]
    d = wl.dirs[0]
    assert kinds.count(O.ASSEMBLE) == d.stub_len
    assert kinds.count(O.REMAP) == wl.seq_lens[0] - d.span_end
    assert kinds.count(O.IDENTITY) == d.span_start
