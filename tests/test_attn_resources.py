"""Registers and scratch of the built attention kernels, from their metadata:
what decides how many waves a SIMD holds.  An instance past a line here still
gives the right results, only slower, so no other test would notice."""
import functools
import pathlib
import re
import subprocess

import pytest

from paper_2106_04718_amd import _native as N
from paper_2106_04718_amd.build import hipcc

TOOLS = pathlib.Path(hipcc()).parents[1] / "llvm" / "bin"


@functools.lru_cache(maxsize=None)
def resources():
    """{mangled kernel name: (registers, bytes of scratch)} of the library."""
    import tempfile
    out = {}
    with tempfile.TemporaryDirectory() as d:
        d = pathlib.Path(d)
        subprocess.run([TOOLS / "llvm-objcopy", "--dump-section", f".hip_fatbin={d / 'fat'}", N.LIB_PATH, d / "copy"],
                       check=True)
        data = (d / "fat").read_bytes()
        at = [m.start() for m in re.finditer(b"__CLANG_OFFLOAD_BUNDLE__", data)]
        for n, p in enumerate(at):
            (d / "bundle").write_bytes(data[p:at[n + 1] if n + 1 < len(at) else len(data)])
            subprocess.run([TOOLS / "clang-offload-bundler", "--type=o", "--unbundle", f"--input={d / 'bundle'}",
                            f"--output={d / 'code'}", "--targets=hipv4-amdgcn-amd-amdhsa--gfx950"], check=True)
            notes = subprocess.run([TOOLS / "llvm-readelf", "--notes", d / "code"], check=True, capture_output=True,
                                   text=True).stdout
            for block in notes.split("  - .agpr_count:")[1:]:
                field = lambda key: re.search(rf"\.{key}:\s+(\S+)", block).group(1)
                out[field("name")] = (int(field("vgpr_count")), int(field("private_segment_fixed_size")))
    return out


def instances(D, bf16, k, split, waves, table=False):
    """Every attn_whole_kernel of these sizes (waves: of a workgroup)."""
    pre = f"attn_whole_kernelILi{D}ELb{int(bf16)}ELi{k}ELb{int(split)}ELi{waves // 4}ELb{int(table)}E"
    got = [r for name, r in resources().items() if pre in name]
    assert got, pre
    return got


needs_tools = pytest.mark.skipif(not (TOOLS / "clang-offload-bundler").exists(), reason="no ROCm tools")


@needs_tools
@pytest.mark.parametrize("k", range(1, 9))
def test_encoder_decoder_bf16(k):
    # 512 registers a SIMD lane: four waves per SIMD up to 128 each
    for waves in (4, 8, 16):
        assert max(instances(64, True, k, False, waves)) <= (128, 0), waves
    for D in (32, 64, 128):   # sixteen waves have 128 each in any case: no scratch
        assert all(scratch == 0 for _, scratch in instances(D, True, k, False, 16)), D
    assert max(instances(32, True, k, False, 4))[0] <= 128


@needs_tools
@pytest.mark.parametrize("k", range(1, 9))
def test_fp32(k):
    for D in (32, 64, 128):
        # without generated tokens: no scratch, four waves per SIMD in
        # workgroups of eight (D = 64 and 32)
        assert all(scratch == 0 for _, scratch in instances(D, False, k, False, 16)), D
        if D < 128:
            assert max(instances(D, False, k, False, 8)) <= (128, 0), D
        # with them, not through a table: no scratch either, but for a few words
        # of five beams at once (D = 32)
        few = 40 if D == 32 and k in (4, 5) else 0
        assert all(scratch <= few for _, scratch in instances(D, False, k, True, 16)), D
        # through one, the walk of a beam per wave has none, and the tasks of up
        # to four beams leave four waves per SIMD
        assert min(scratch for _, scratch in instances(D, False, k, True, 16, table=True)) == 0, D
        if k <= 4:
            assert min(instances(D, False, k, True, 8, table=True)) <= (128, 0), D
