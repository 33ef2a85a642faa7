"""What the planner counts of a paged gather, and what it decides by it, on the host
(tests/gather_route_check.cpp): spans of rows of one page run and one segment, against the oracle's
page plan and row sources."""

import os
import random
import shutil
import subprocess

import pytest

import workloads as W
from oracle import splice_oracle as O

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    """ask([(workload, flags)]) -> the program's numbers per call."""
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    exe, csrc = str(tmp_path_factory.mktemp("routes") / "check"), os.path.join(ROOT, "paper_2606_01065_amd", "csrc")
    subprocess.run([gxx, "-O2", "-std=c++17", "-Wall", "-Wextra", "-Werror", "-I" + os.path.join(ROOT, "include"),
                    "-I" + csrc, os.path.join(ROOT, "tests", "gather_route_check.cpp"),
                    os.path.join(csrc, "plan.cpp"), "-o", exe], check=True)

    def run(calls):
        text = []
        for wl, flags in calls:
            text.append(f"{int(wl.dtype == 'f32')} {wl.n_layers} {wl.page_size} {flags} {len(wl.planes)}")
            text += [f"{p.row_elems} {p.n_heads} {p.head_stride or p.row_elems} {p.rot_offset} {p.rot_dim} {p.style}"
                     for p in wl.planes]
            text.append(" ".join(map(str, [len(wl.seq_lens)] + list(wl.seq_lens) + [len(wl.dirs)])))
            text += [f"{d.seq} {d.span_start} {d.span_end} {d.stub_len}" for d in wl.dirs]
        out = subprocess.run([exe], input="\n".join(text), capture_output=True, text=True)
        assert out.returncode == 0, out
        return [tuple(map(int, ln.split())) for ln in out.stdout.split("\n") if ln]
    return run


def _odirs(wl):
    return [O.Directive(d.span_start, d.span_end, d.stub_len, seq=d.seq, mode=d.mode) for d in wl.dirs]


def counts(wl, flags):
    """(gathered rows, fresh pages, spans) from the oracle: a span ends where a page is not assembled, a
    replacement begins or ends, or the shift changes."""
    P, pages, spans = wl.page_size, 0, 0
    plans = O.plan_paged(wl.seq_lens, _odirs(wl), P, remap=not flags)
    for b, (n, plan) in enumerate(zip(wl.seq_lens, plans)):
        src = O.row_sources(n, [d for d in _odirs(wl) if d.seq == b])
        pages += sum(k == O.ASSEMBLE for k in plan.kinds)
        last = None
        for q, (kind, a, c) in enumerate(src):
            key = None
            if plan.kinds[q // P] == O.ASSEMBLE:
                key = ("old", c) if kind == "old" else ("stub", a)
                spans += key != last
            last = key
    return P * pages, pages, spans


def random_call(rng, page):
    n_seqs, lens, dirs = rng.randint(1, 4), [], []
    for b in range(n_seqs):
        n = rng.randint(0, 400)
        lens.append(n)
        cuts = sorted(rng.sample(range(n + 1), min(2 * rng.randint(0, 20), (n + 1) // 2 * 2)))
        for s, e in zip(cuts[::2], cuts[1::2]):
            dirs.append(W.Dir(s, e, rng.choice([0, 1, e - s, e - s + page, rng.randint(0, 9)]), seq=b))
    return W.Workload("spans", 2, "bf16", [W.mla_plane()], dirs, lens, page_size=page)


def test_spans_of_a_gather(ask):
    rng = random.Random(5)
    calls = [(random_call(rng, page), cow) for page in (1, 3, 16) for cow in (0, 1) for _ in range(60)]
    for (wl, cow), (rows, pages, spans, short, _) in zip(calls, ask(calls)):
        assert (rows, pages, spans) == counts(wl, cow), (wl.page_size, cow, wl.seq_lens, wl.dirs)
        assert short == (rows < 4 * spans)


def turned_spans(rows, k):
    """Copy-on-write token slots: every row moves by one place, spans of k replacement rows and k old rows in turn."""
    dirs = [W.Dir(5 + 2 * k * i, 5 + 2 * k * i + k, k + (i == 0)) for i in range(rows // (2 * k))]
    return dirs, [5 + 2 * k * len(dirs)]


def one_edit_each(seqs, tokens):
    return [W.Dir(tokens // 4, tokens // 4 + 7, 11, seq=b) for b in range(seqs)], [tokens] * seqs


MLA, GQA8 = [W.mla_plane()], W.gqa_planes(heads=8, dim=128)


@pytest.mark.parametrize("planes,layers,page,call,table", [
    (MLA, 61, 1, turned_spans(4000, 3), 1), (MLA, 61, 1, turned_spans(4000, 24), 1), (MLA, 16, 1, turned_spans(1100, 3), 0),
    (MLA, 16, 1, turned_spans(4000, 3), 1), (MLA, 2, 1, turned_spans(4000, 3), 0), (MLA, 2, 1, turned_spans(12000, 3), 1),
    (MLA, 61, 1, turned_spans(1000, 3), 0), (W.mla_split_planes(), 2, 1, turned_spans(12000, 3), 0),
    (GQA8, 16, 1, turned_spans(4000, 3), 1), (GQA8, 16, 1, turned_spans(4000, 24), 0), (GQA8, 4, 1, turned_spans(1100, 3), 0),
    (MLA, 61, 16, one_edit_each(64, 64), 1), (MLA, 16, 16, one_edit_each(32, 200), 0), (MLA, 16, 64, one_edit_each(128, 100), 1),
    (MLA, 61, 64, ([W.Dir(100, 160, 44)], [3000]), 0), (MLA, 61, 64, ([W.Dir(100, 160, 44)], [6000]), 1)])
def test_row_table_or_one_launch(ask, planes, layers, page, call, table):
    """Calls whose two routes were timed: each takes the faster one (the last two differ in bytes alone)."""
    dirs, lens = call
    (rows, pages, spans, _, got), = ask([(W.Workload("route", layers, "bf16", planes, dirs, lens, page_size=page), 1)])
    assert got == table, (rows, pages, spans)
