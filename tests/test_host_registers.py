"""Registers and scratch memory of kernels whose comments count on a number of waves a SIMD (512 registers each 8 by 8: 128 for
four waves, 96 for five, 80 for six), read from the notes of the built library's own code objects (CPU)."""
import os
import re
import shutil
import struct
import subprocess

import pytest

ROCM_LLVM = "/opt/rocm/llvm/bin"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{kernel<arguments>: (vector registers, bytes of scratch memory a lane)}"""
    readelf, objcopy = (os.path.join(ROCM_LLVM, "llvm-" + n) for n in ("readelf", "objcopy"))
    if not (os.path.exists(readelf) and os.path.exists(objcopy) and shutil.which("c++filt")):
        pytest.skip("no LLVM tools")
    from paper_2505_14371_amd import build, qoda

    if not os.path.exists(qoda.LIB_PATH):
        build.build()
    d = tmp_path_factory.mktemp("code")
    fat = str(d / "fat")
    subprocess.check_call([objcopy, "--dump-section", ".hip_fatbin=" + fat, qoda.LIB_PATH, str(d / "rest")], stderr=subprocess.DEVNULL)
    data = open(fat, "rb").read()
    out = {}
    for m in re.finditer(b"__CLANG_OFFLOAD_BUNDLE__", data):
        at = m.start()
        entries, = struct.unpack_from("<Q", data, at + 24)
        pos = at + 32
        for _ in range(entries):
            off, size, n = struct.unpack_from("<QQQ", data, pos)
            target, pos = data[pos + 24:pos + 24 + n].decode(), pos + 24 + n
            if "gfx950" not in target:
                continue
            obj = d / "object"
            obj.write_bytes(data[at + off:at + off + size])
            text = subprocess.run([readelf, "--notes", str(obj)], capture_output=True, text=True, check=True).stdout
            for blk in text.split("- .agpr_count")[1:]:
                get = {k: re.search(r"\." + k + r":\s+(\S+)", blk).group(1) for k in ("name", "vgpr_count", "private_segment_fixed_size")}
                name = subprocess.run(["c++filt", get["name"]], capture_output=True, text=True).stdout
                out[re.sub(r"^void |qoda::|\(.*", "", name.strip())] = (int(get["vgpr_count"]), int(get["private_segment_fixed_size"]))
    assert len(out) > 100
    return out


@pytest.mark.parametrize("bucket", ["false", "true"])
@pytest.mark.parametrize("bits", range(2, 10))
def test_alt_decode_in_eight_waves_fits_a_cu_twice(kernels, bits, bucket):
    early = "true" if bits <= 6 else "false"
    assert kernels[f"k_decode<{bits}, 2, {bucket}, 8, {early}>"][0] <= 128


@pytest.mark.parametrize("mode", [0, 1, 3])
def test_whole_octets_of_five_bits_under_bucket_scope_run_six_waves(kernels, mode):
    assert kernels[f"k_decode<5, {mode}, true, 8, false>"][0] <= 80


@pytest.mark.parametrize("bits", range(2, 7))
def test_quantize_without_previous_message_runs_six_waves(kernels, bits):
    assert kernels[f"k_quantize<{bits}, false, false>"][0] <= 80


def test_quantize_of_nine_bits_with_previous_message_runs_five_waves(kernels):
    assert kernels["k_quantize<9, true, false>"][0] <= 96


@pytest.mark.parametrize("prev", ["false", "true"])
@pytest.mark.parametrize("bits", range(2, 10))
def test_held_tiles_four_workgroups_a_cu_and_nothing_spilled(kernels, bits, prev):
    """Three with nine bits; a workgroup is a wave on each SIMD."""
    registers, scratch = kernels[f"k_quantize_held<{bits}, {prev}>"]
    assert registers <= (168 if bits == 9 else 128) and scratch == 0
