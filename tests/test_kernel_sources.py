"""Ordering rules of the kernels that no run can show to be broken (the order a
rule fixes is nearly always the one that happens), checked on their source."""

import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2508_16471_amd", "csrc")


def _kernels():
    """(name, text) of every kernel: from its __global__ to the closing brace."""
    for f in sorted(os.listdir(CSRC)):
        if not f.endswith((".hip", ".h")):
            continue
        with open(os.path.join(CSRC, f)) as fh:
            for part in fh.read().split("__global__")[1:]:
                text = part[:part.index("\n}\n") + 3] if "\n}\n" in part else part
                name = re.search(r"\b(k_\w+)\s*\(", text)
                if name:
                    yield name.group(1), text


def _clears_its_gate(text):
    return "upd_scalars<" in text or re.search(r"\bactive\[\w+\] = 0;", text)


def test_gates_that_a_launch_clears_are_read_once_per_workgroup():
    """A right-hand side's activity flag that the leading workgroup clears while
    the others start: waves of one workgroup must not read it one by one."""
    names = []
    for name, text in _kernels():
        if not _clears_its_gate(text):
            continue
        names.append(name)
        gate = text[:text.index("upd_scalars<")] if "upd_scalars<" in text else text
        assert "group_flag(active + " in gate, name
        assert "int* __restrict__ active" not in text, name
    assert sorted(names) == ["k_fft_x_fwd_c", "k_plane_fwd", "k_rt_pupd", "k_rt_supd"]


def test_lines_written_over_their_transform_are_fenced():
    """The plane passes put a line back into the LDS that its own wave has just
    transformed it in, without a barrier: each write comes after a wave fence."""
    writes = 0
    for name, text in _kernels():
        if name not in ("k_plane_fwd", "k_plane_inv"):
            continue
        after = text.split("plane_fft<")[1:]
        assert len(after) == 1, name
        at = after[0].index("line[pidx(t + q * X::TT)] = v[q];")
        assert "wave_fence();" in after[0][:at], name
        writes += 1
        reads = after[0][at:].find("line[pidx(xi)]")
        if reads >= 0:
            assert "wave_fence();" in after[0][at:at + reads], name
    assert writes == 2


def test_traffic_records_cover_every_product_source():
    """A counter record is stamped with the sources it was taken from: all files
    of the FFT passes, and what they include."""
    from paper_2508_16471_amd.profsum import PRODUCT_SOURCES

    want = {f for f in os.listdir(CSRC) if f.startswith("fft")}
    for f in sorted(want):
        with open(os.path.join(CSRC, f)) as fh:
            want |= set(re.findall(r'#include "(\w+\.h)"', fh.read()))
    assert {os.path.basename(f) for f in PRODUCT_SOURCES} == want
