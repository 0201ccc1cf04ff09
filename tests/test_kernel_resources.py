"""Registers of the built search kernels, read from the code objects of libvns.so: what decides how many of their workgroups
a compute unit holds.  CPU only."""
import re
import struct
import subprocess
from pathlib import Path

import pytest

from paper_1704_05132_amd.build import PKG

READELF = Path("/opt/rocm/llvm/bin/llvm-readelf")
BUNDLE = b"__CLANG_OFFLOAD_BUNDLE__"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{mangled kernel name: (VGPRs, static LDS bytes)}"""
    if not READELF.exists():
        pytest.skip("no llvm-readelf")
    lib, out = (PKG / "libvns.so").read_bytes(), {}
    for m in re.finditer(BUNDLE, lib):
        at = m.start() + len(BUNDLE)
        n, at = struct.unpack_from("<Q", lib, at)[0], at + 8
        for _ in range(n):
            off, size, length = struct.unpack_from("<QQQ", lib, at)
            triple, at = lib[at + 24:at + 24 + length], at + 24 + length
            if b"gfx950" not in triple:
                continue
            f = tmp_path_factory.mktemp("co") / "device.o"
            f.write_bytes(lib[m.start() + off:m.start() + off + size])
            text = subprocess.run([str(READELF), "--notes", str(f)], capture_output=True, text=True, check=True).stdout
            for k in re.split(r"\n  - ", text[text.index("amdhsa.kernels"):])[1:]:
                if ".symbol:" not in k:   # the metadata after the kernels
                    continue
                field = lambda key: re.search(rf"\.{key}:\s+'?([\w.]+)", k).group(1)
                out[field("symbol").removesuffix(".kd")] = (int(field("vgpr_count")), int(field("group_segment_fixed_size")))
    return out


def family(kernels, name):
    """The instantiations of vns::`name` (a template or not)."""
    found = {k: v for k, v in kernels.items() if re.match(rf"_ZN3vns{len(name)}{name}(I|E)", k)}
    assert found, name
    return found


@pytest.mark.parametrize("name", ["k_run", "k_run_short", "k_run_spec"])
def test_four_wavefronts_per_simd(kernels, name):
    """A SIMD has 512 VGPRs: at most 128 leave room for four wavefronts, two workgroups of eight to a compute unit."""
    for k, (vgprs, _) in family(kernels, name).items():
        assert vgprs <= 128, (k, vgprs)


@pytest.mark.parametrize("name", ["k_run", "k_run_short", "k_run_coop", "k_run_learned", "k_run_learned_coop"])
def test_static_lds(kernels, name):
    """Side-by-side and best-of-G searches need their workgroups resident at once: 38 x 52 with disposal, best of 16 on 96
    chains in workgroups of two wavefronts, is six workgroups to a compute unit's 160 KB, 15808 bytes of each its rows."""
    for k, (_, lds) in family(kernels, name).items():
        assert lds + 15808 <= 160 * 1024 // 6, (k, lds)
