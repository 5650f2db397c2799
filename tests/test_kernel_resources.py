"""Registers of the built kernels, as the compiler's metadata in the library's gfx950 code object gives them: what decides how
many workgroups a compute unit holds.  No GPU needed."""
import re
import struct
import subprocess

import pytest

READELF = "/opt/rocm/llvm/bin/llvm-readelf"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{mangled name: {"vgpr_count": n, "vgpr_spill_count": n, "group_segment_fixed_size": bytes}}"""
    from paper_2601_18383_amd import build
    data = open(build.build(force=False), "rb").read()
    at = data.index(b"__CLANG_OFFLOAD_BUNDLE__")
    count, pos = struct.unpack_from("<Q", data, at + 24)[0], at + 32
    code = None
    for _ in range(count):
        offset, size, length = struct.unpack_from("<QQQ", data, pos)
        if b"gfx950" in data[pos + 24:pos + 24 + length]:
            code = data[at + offset:at + offset + size]
        pos += 24 + length
    path = tmp_path_factory.mktemp("code") / "gfx950.co"
    path.write_bytes(code)
    notes = subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True, check=True).stdout
    out = {}
    for block in notes.split("\n  - .a")[1:]:
        field = lambda k: re.search(r"\.%s:\s*(\S+)" % k, block)
        if field("symbol"):
            out[field("name").group(1)] = {k: int(field(k).group(1)) for k in
                                           ("vgpr_count", "vgpr_spill_count", "group_segment_fixed_size")}
    assert len(out) > 50
    return out


def test_head_dim_64_launches_keep_two_workgroups_per_compute_unit(kernels):
    """The eight-wave attention kernels of head_dim 64 that launches of more than 256 workgroups take (dense, inside the
    memory-side cache, chunks merged four at a time): 512 registers a SIMD lane, four waves of 128 each."""
    plain = {n: k for n, k in kernels.items() if re.search(r"attend_kernelILi64ELi8ELb1ELb[01]ELb[01]ELb0EL[bi]0ELb[01]ELb0EE", n)}
    assert len(plain) == 8  # with and without the owed update, the append, kept logits
    for name, k in plain.items():
        assert k["vgpr_count"] <= 128 and k["vgpr_spill_count"] == 0, name
        assert 2 * k["group_segment_fixed_size"] <= 160 * 1024, name


def test_eight_wave_attention_kernels_do_not_spill(kernels):
    eight = {n: k for n, k in kernels.items() if re.search(r"attend_kernelILi(64|128)ELi8E", n)}
    assert len(eight) > 40
    for name, k in eight.items():
        assert k["vgpr_spill_count"] == 0, name


def test_passes_over_k_alone_keep_two_workgroups_per_compute_unit(kernels):
    """The score update by itself, eight waves: short caches of many units hang on the second workgroup."""
    alone = {n: k for n, k in kernels.items() if re.search(r"attend_kernelILi(64|128)ELi8ELb0E", n)}
    assert len(alone) >= 8
    for name, k in alone.items():
        assert k["vgpr_count"] <= 128 and 2 * k["group_segment_fixed_size"] <= 160 * 1024, name


def test_steps_on_large_paged_caches_of_head_dim_64_keep_two_workgroups_per_compute_unit(kernels):
    burst = {n: k for n, k in kernels.items() if re.search(r"attend_kernelILi64ELi8ELb1ELb1ELb1ELb1ELi2ELb0ELb0EE", n)}
    assert len(burst) == 1
    for name, k in burst.items():
        assert k["vgpr_count"] <= 128 and 2 * k["group_segment_fixed_size"] <= 160 * 1024, name


def test_kernels_for_runs_of_steps_do_not_spill(kernels):
    """The cache stays in registers from the first step to the last: none of it, and nothing else, in scratch memory.  Two waves a SIMD."""
    run = {n: k for n, k in kernels.items() if re.search(r"(resident|merge_run|run_scores)_kernelILi(64|128)E", n)}
    assert len(run) == 10  # one and two tiles a wave, chunks; the two kernels behind them
    for name, k in run.items():
        assert k["vgpr_spill_count"] == 0 and k["vgpr_count"] <= 256 and k["group_segment_fixed_size"] <= 160 * 1024, name
