"""Which half-split rows have their partner chunks exchanged between lanes: on the host the
planner's choice (tests/lane_exchange_check.cpp), on the GPU rows that are neither whole wavefronts
nor a divisor of one, against the oracle, with and without a workspace for the ordered tiles."""

import ctypes
import os
import random
import shutil
import subprocess

import pytest
import torch

import workloads as W
from tests.parity_util import bits

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_planner_exchanges_only_within_a_wavefront(tmp_path):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("g++ not available")
    exe, csrc = str(tmp_path / "check"), os.path.join(ROOT, "paper_2606_01065_amd", "csrc")
    subprocess.run([gxx, "-O2", "-std=c++17", "-Wall", "-Wextra", "-Werror", "-I" + os.path.join(ROOT, "include"),
                    "-I" + csrc, os.path.join(ROOT, "tests", "lane_exchange_check.cpp"),
                    os.path.join(csrc, "plan.cpp"), "-o", exe], check=True)
    out = subprocess.run([exe], capture_output=True, text=True)
    assert out.returncode == 0, (out.returncode, out.stdout)
    lanes = [tuple(map(int, ln.split())) for ln in out.stdout.split("\n") if ln]
    assert lanes == [(1, 1), (1, 1), (1, 0), (1, 1), (1, 1), (1, 1), (1, 0), (1, 0),
                     (0, 0), (0, 0), (0, 0), (0, 0), (0, 0)]


KINDS = {"mla": [W.PlaneDesc((576,), 1, 576, 512, 64, 1, 10000.0)],
         "heads5": W.gqa_planes(heads=5, dim=128), "heads10": W.gqa_planes(heads=10, dim=64),
         "partial": [W.PlaneDesc((3, 64), 3, 64, 32, 32, 1, 10000.0)],
         "heads96": W.gqa_planes(heads=3, dim=96)}                    # two-chunk units, ordered chains


@pytest.mark.gpu
@pytest.mark.parametrize("kind,dtype", [("mla", "bf16"), ("mla", "f32"), ("heads5", "bf16"), ("heads10", "bf16"),
                                        ("heads10", "f32"), ("partial", "bf16"), ("heads96", "bf16")])
def test_ragged_half_split_rows(kind, dtype):
    from paper_2606_01065_amd import leyline as L
    from tests import test_gpu_contig as TC
    rng = random.Random(f"{kind}/{dtype}")
    for n, dirs in [(65, [W.Dir(3, 4, 0)]), (700, [W.Dir(30, 31, 0)]), (700, [W.Dir(100, 100, 3)]),
                    (1500, [W.Dir(7, 40, 12), W.Dir(300, 310, 50), W.Dir(900, 1000, 1)]), (900, [W.Dir(10, 500, 16)])]:
        wl = TC._small_workload(rng, "heads", dtype, 3, n, dirs)
        wl.planes = KINDS[kind]
        planes, stubs = W.alloc_contig(wl, "cuda:0")
        pristine = [t.clone() for t in planes]
        new_len = TC._run_and_check(L, wl, planes, stubs, f"ragged {kind}/{dtype} n={n}")
        # no workspace, one that is misaligned, one too small for the tiles' flags: the same bits without tiles
        dd = L.make_directives(TC._dir_dicts(wl, stubs))
        buf = torch.empty(1 << 20, dtype=torch.uint8, device="cuda:0")
        for ptr, size in ((None, 0), (buf.data_ptr() + 128, 1 << 19), (buf.data_ptr(), 256)):
            other, got = [t.clone() for t in pristine], ctypes.c_int64(0)
            cache = L.make_cache(TC._specs(L, wl, other))
            assert L._lib.leyline_splice_contig(ctypes.byref(cache), n, dd, len(dirs), ctypes.byref(got), None, ptr, size,
                                                L._stream(None)) == 0
            assert got.value == new_len
            for a, b in zip(planes, other):
                assert torch.equal(bits(a[:, :new_len]), bits(b[:, :new_len])), f"{kind}/{dtype} n={n} workspace {size}"


@pytest.mark.gpu
@pytest.mark.parametrize("layers", [3, 60000])
def test_noalloc_within_and_beyond_its_scratch(layers):
    """Ragged half-split rows through the entry without a workspace: as ordered tiles in the library's scratch
    array, or (five edits of 60,000 layers need 300,000 flags of 4 bytes) without them; the same bits."""
    from paper_2606_01065_amd import leyline as L
    from tests import test_gpu_contig as TC
    n, dirs = 60, [W.Dir(3, 5, 1)] + [W.Dir(27 + 6 * i, 29 + 6 * i, 1) for i in range(4)]   # 22 rows by -1 first
    wl = W.Workload("noalloc_half", 1, "bf16", KINDS["mla"], dirs, [n], capacity=n, seed=11)
    (one,), stubs1 = W.alloc_contig(wl, "cuda:0")
    stubs = [[s.expand(layers, *s.shape[1:]).contiguous() for s in per] for per in stubs1]
    dd = L.make_directives([dict(span_start=d.span_start, span_end=d.span_end, stub=stubs[j], stub_len=1)
                            for j, d in enumerate(dirs)])
    outs = []
    for call in (L.leyline_splice_contig, L.leyline_splice_contig_noalloc):
        t = one.expand(layers, *one.shape[1:]).contiguous()
        cache = L.make_cache(TC._specs(L, wl, [t]))
        assert (L.leyline_contig_query(cache, n, dd, 5).workspace_bytes > L.SCRATCH_BYTES) == (layers > 3)
        print(f"[case] no-alloc ragged half-split, {layers} layers, {call.__name__}", flush=True)
        assert call(cache, n, dd, 5) == n - 5
        torch.cuda.synchronize()
        assert torch.equal(bits(t), bits(t[:1]).expand_as(t)), "layers differ"
        outs.append(t[0, :n - 5].clone())
    assert torch.equal(bits(outs[0]), bits(outs[1]))
    assert not torch.equal(bits(outs[0]), bits(one[0, :n - 5]))
