"""Registers of the built kernels, read from the metadata that the compiler leaves in the library: more registers
mean fewer resident wavefronts, and every launch of the kernel pays for its hungriest path."""
import os
import re
import struct
import subprocess

import pytest

from paper_2012_15198_amd import cxmix as cx

READELF = "/opt/rocm/llvm/bin/llvm-readelf"
BUNDLE = b"__CLANG_OFFLOAD_BUNDLE__"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{demangled kernel name: (registers, bytes of scratch per lane)} of libcxmix.so."""
    if not os.path.exists(READELF):
        pytest.skip("no llvm-readelf")
    data = open(cx.LIB_PATH, "rb").read()
    folder, notes, pos = tmp_path_factory.mktemp("code"), [], data.find(BUNDLE)
    while pos >= 0:                                            # one bundle per translation unit
        entry = pos + 32
        for _ in range(struct.unpack_from("<Q", data, pos + 24)[0]):
            offset, size, length = struct.unpack_from("<QQQ", data, entry)
            if size and b"gfx950" in data[entry + 24:entry + 24 + length]:
                path = folder / f"{pos}.co"
                path.write_bytes(data[pos + offset:pos + offset + size])
                notes.append(subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True, check=True).stdout)
            entry += 24 + length
        pos = data.find(BUNDLE, pos + 1)
    found = {}
    for block in re.split(r"\n\s*- \.agpr_count", "".join(notes))[1:]:
        number = {key: int(value) for key, value in re.findall(r"\.(\w+):\s+(\d+)\s*$", block, re.M)}
        found[re.search(r"\.name:\s+(_Z\S+)", block).group(1)] = (number["vgpr_count"], number["private_segment_fixed_size"])
    plain = subprocess.run(["c++filt"], input="\n".join(found), capture_output=True, text=True, check=True).stdout.split("\n")
    return {name.replace("(anonymous namespace)::", "").split("(")[0].replace("void ", ""): value
            for name, value in zip(plain, found.values())}


# wavefronts per SIMD of the default out-of-place kernels (one slice per lane, non-temporal stores)
@pytest.mark.parametrize("op,waves", [
    ("MeanOp<1>", 8), ("MeanOp<2>", 7), ("MeanOp<3>", 5), ("MeanOp<4>", 4), ("MeanOp<5>", 4), ("MeanOp<6>", 4),
    ("MeanOp<7>", 4), ("MeanOp<8>", 3), ("FusedOp", 5), ("HierFusedOp<1>", 5), ("HierFusedOp<2>", 4), ("HierFusedOp<3>", 4),
    ("HierFusedOp<4>", 3), ("HierFusedOp<7>", 3), ("Row16Op<false, 1>", 8), ("Row16Op<false, 4>", 3), ("Row16Op<false, 8>", 3),
    ("HierFused16Op<false, 4>", 3)])
def test_boundary_tiles_do_not_cost_the_out_of_place_kernels_wavefronts(kernels, op, waves):
    registers = kernels[f"gather_kernel<{op}, 1, true, false>"][0]
    assert 512 // (-(-registers // 8) * 8) >= waves, registers


def wavefronts(kernels, op, slices):
    return 512 // (-(-kernels[f"gather_kernel<{op}, {slices}, true, false>"][0] // 8) * 8)


# those that matrices beyond the last-level cache take: stores written through, tiles on the rows' own lines (push-sum has two slices)
@pytest.mark.parametrize("op,slices,waves", [
    ("ThroughOp", 1, 8), ("OnLines<ThroughOp>", 1, 8), ("OnLines<FusedOp>", 1, 5), ("OnLines<PushOp>", 2, 5), ("OnLines<Push16Op<false> >", 2, 4),
    ("OnLines<Push16Op<true> >", 2, 4), ("OnLines<Fused16Op<false> >", 1, 4), ("OnLines<Fused16Op<true> >", 1, 4)])
def test_rows_on_their_own_lines_keep_their_wavefronts(kernels, op, slices, waves):
    assert wavefronts(kernels, op, slices) >= waves
    plain = op.removeprefix("OnLines<").removesuffix(">").strip()
    assert wavefronts(kernels, op, slices) >= wavefronts(kernels, plain, slices)


def test_no_mixing_kernel_keeps_registers_in_scratch(kernels):
    """fits() in cx_launch.hpp admits shapes that stay in registers: scratch is slow, and the runtime would reserve it
    on the first launch, where no call may allocate."""
    mixing = {name: scratch for name, (_, scratch) in kernels.items() if name.startswith(("mix_kernel<", "gather_kernel<"))}
    assert len(mixing) > 400 and not {name: scratch for name, scratch in mixing.items() if scratch}


def test_no_kernel_of_split_rows_keeps_registers_in_scratch(kernels):
    """Nor more registers than its largest workgroup leaves a wavefront (kPartWaves in cx_kernels.hpp)."""
    parts = {name: value for name, value in kernels.items() if name.startswith("parts_kernel<")}
    assert len(parts) > 50 and not {name: scratch for name, (_, scratch) in parts.items() if scratch}
    assert parts["parts_kernel<MeanOp<1>, 1, 4>"][0] <= 128 and parts["parts_kernel<FusedOp, 1, 2>"][0] <= 128
