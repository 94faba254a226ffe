"""What the compiler made of the kernels, read from the built library: registers, LDS and instructions that decide how many
workgroups a compute unit holds, or that stop more than their own wave."""
import re
import struct
import subprocess

import pytest

from paper_2312_08053_amd.binding import LIB_PATH

LLVM = "/opt/rocm/llvm/bin/"
LDS, WAVES, REGISTERS = 160 * 1024, 8, 512           # of a compute unit, of a SIMD (of four), of a SIMD's lane


@pytest.fixture(scope="module")
def code(tmp_path_factory):
    """The library's gfx950 code object, as a file."""
    blob = open(LIB_PATH, "rb").read()
    at = blob.index(b"__CLANG_OFFLOAD_BUNDLE__")
    (entries,) = struct.unpack_from("<Q", blob, at + 24)
    p = at + 32
    for _ in range(entries):
        off, size, idlen = struct.unpack_from("<QQQ", blob, p)
        name = blob[p + 24:p + 24 + idlen].decode()
        p += 24 + idlen
        if name.endswith("gfx950"):
            path = tmp_path_factory.mktemp("code") / "kimad.co"
            path.write_bytes(blob[at + off:at + off + size])
            return str(path)
    raise AssertionError("no gfx950 code in the library")


@pytest.fixture(scope="module")
def kernels(code):
    """name -> dict of the kernel's metadata (all instantiations of a template under one name, the largest of each)."""
    text = subprocess.run([LLVM + "llvm-readelf", "--notes", code], check=True, capture_output=True, text=True).stdout
    out = {}
    for block in re.split(r"\n  - \.a", text)[1:]:
        name = re.search(r"\.name: +_ZN5kimad\d+(k_[a-z0-9_]+?)(?:E|I[LN])", block)
        if not name:
            continue
        d = out.setdefault(name[1], {})
        for key in ("vgpr_count", "group_segment_fixed_size", "max_flat_workgroup_size", "private_segment_fixed_size", "agpr_count"):
            m = re.search(r"\." + key + r": +(\d+)", "  .a" + block)
            d[key] = max(d.get(key, 0), int(m[1]) if m else 0)
    return out


def resident(k):
    """Workgroups that a compute unit holds at a time."""
    waves = -(-k["max_flat_workgroup_size"] // 64)
    regs = -(-max(k["vgpr_count"], 1) // 8) * 8
    per_simd = min(WAVES, REGISTERS // regs)
    return min(4 * per_simd // waves, LDS // max(k["group_segment_fixed_size"], 1))


def test_two_recount_workgroups_share_a_compute_unit(kernels):
    """One clears its tables, waits at its barriers and adds them up while the other counts."""
    k = kernels["k_hist2"]
    assert resident(k) >= 2, k
    assert k["private_segment_fixed_size"] == 0, k


def test_the_exact_pass_counts_with_all_waves(kernels):
    """Its counting is bound by the loads and additions under way: what the scan takes must not cost it waves."""
    k = kernels["k_hist3p"]
    assert resident(k) * -(-k["max_flat_workgroup_size"] // 64) == 4 * WAVES, k
    assert k["private_segment_fixed_size"] == 0, k


@pytest.mark.parametrize("kernel", ["k_hist2", "k_hist3p"])
def test_a_finished_layer_writes_no_cache_back(code, kernel):
    """A workgroup that finds a layer complete reads sums that were added beyond the caches: nothing is to be written back, and
    a write-back holds up everything that goes through that cache (twice the time of a recount)."""
    symbols = subprocess.run([LLVM + "llvm-readelf", "--symbols", "--wide", code], check=True, capture_output=True, text=True).stdout
    names = re.findall(r"\b(_ZN5kimad\d+" + kernel + r"E\w+)$", symbols, re.M)
    assert names
    text = subprocess.run([LLVM + "llvm-objdump", "-d", "--disassemble-symbols=" + ",".join(names), code], check=True,
                          capture_output=True, text=True).stdout
    assert "s_endpgm" in text and "buffer_wbl2" not in text
