"""Register and scratch use of the built kernels, as the compiler reported it
when the library was last built: no kernel may spill to scratch memory (a
spill turns every register access of the epilogue or inner loop into a
memory round trip, which is how a small code change can double a kernel's
time without changing its results)."""
import os

import pytest

from paper_2609_35139_amd import build as _b


def _rows():
    if not os.path.exists(_b.RESOURCES):
        pytest.skip("library not built here (run __graft_entry__.build())")
    rows = []
    for line in open(_b.RESOURCES):
        name, *kv = line.split()
        rows.append((name, dict(x.split("=") for x in kv)))
    return rows


def test_every_source_reported():
    rows = _rows()
    for kernel in ("gemm_nt_kernel", "gemm_skinny_kernel", "gemm_phase_kernel",
                   "compress_segments_kernel"):
        assert any(kernel in n for n, _ in rows)
    assert any("attention_kernel" in n for n, _ in rows)
    assert any("layernorm_kernel" in n for n, _ in rows)


def test_no_kernel_spills_to_scratch():
    bad = [(n, r) for n, r in _rows() if r.get("scratch") not in ("0",)]
    assert not bad, bad


def test_no_kernel_that_the_tile_choice_cannot_reach():
    """64x64 tiles split over K by wave: for bf16 bias epilogues of long K, and
    for the rotating output add, whose threads own two segments."""
    names = [n for n, _ in _rows() if "SkinnyTileI" in n and "Li2ELi2ELi4ELi2EEE" in n]
    bias = [n for n in names if "EpiBiasIDF16b" in n]
    rope = [n for n in names if "EpiExpandRopeI" in n]
    assert len(bias) == 2 and len(rope) == 2 and len(names) == 4, names


def test_resource_remarks_parse():
    text = ("x.hip:1:1: remark: Function Name: _Z3fooPf [-Rpass-analysis=kernel-resource-usage]\n"
            "x.hip:1:1: remark:     VGPRs: 12 [-Rpass-analysis=kernel-resource-usage]\n"
            "x.hip:1:1: remark:     ScratchSize [bytes/lane]: 16 [-Rpass-analysis=kernel-resource-usage]\n"
            "x.hip:1:1: remark:     Occupancy [waves/SIMD]: 8 [-Rpass-analysis=kernel-resource-usage]\n")
    assert _b._resources(text) == [{"kernel": "_Z3fooPf", "VGPRs": 12, "ScratchSize": 16,
                                     "Occupancy": 8}]
