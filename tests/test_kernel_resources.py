"""What the compiler made of the kernels (CPU only): every device function is inlined
(a call costs its kernel a stack in memory), the persistent multi-table kernels
have the registers and LDS for the occupancy that sizes their grids, and every 16-byte
store of a slot is followed by the wait states that its data registers need."""
import os
import re
import struct
import subprocess

import pytest

import paper_2509_16407_amd as hw

LLVM = "/opt/rocm/llvm/bin/"
pytestmark = pytest.mark.skipif(not os.path.exists(LLVM + "llvm-readelf"), reason="no LLVM tools")
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def code_objects(so, tmp):
    """The gfx950 code objects of the library, one per source with kernels."""
    fat = os.path.join(tmp, "fat")
    subprocess.check_call([LLVM + "llvm-objcopy", "--dump-section", ".hip_fatbin=" + fat, so, os.path.join(tmp, "x.so")])
    d = open(fat, "rb").read()
    at = d.find(MAGIC)
    while at >= 0:
        n, = struct.unpack_from("<Q", d, at + 24)
        p = at + 32
        for _ in range(n):
            off, size, tlen = struct.unpack_from("<QQQ", d, p)
            triple = d[p + 24: p + 24 + tlen]
            p += 24 + tlen
            if b"gfx950" in triple and size:
                path = os.path.join(tmp, "co%d" % at)
                with open(path, "wb") as f:
                    f.write(d[at + off: at + off + size])
                yield path
        at = d.find(MAGIC, at + 1)


@pytest.fixture(scope="module")
def objects(tmp_path_factory):
    return list(code_objects(hw.LIB_PATH, str(tmp_path_factory.mktemp("co"))))


@pytest.fixture(scope="module")
def kernels(objects):
    """name -> (VGPRs, LDS bytes) of every kernel, and the functions that are none."""
    res, other = {}, []
    for co in objects:
        text = subprocess.run([LLVM + "llvm-readelf", "-W", "-s", "--notes", co], capture_output=True, text=True,
                              check=True).stdout
        funcs = set(re.findall(r" FUNC .* (\S+)$", text, re.M))
        own = {}
        for doc in re.split(r"^  - \.ag", text, flags=re.M)[1:]:
            f = dict(re.findall(r"\.(name|vgpr_count|group_segment_fixed_size): +(\S+)$", doc, re.M))
            own[f["name"]] = (int(f["vgpr_count"]), int(f["group_segment_fixed_size"]))
        assert own and set(own) <= funcs
        res.update(own)
        other += sorted(funcs - set(own))
    names = subprocess.run(["c++filt"], input="\n".join(res), capture_output=True, text=True, check=True).stdout.split("\n")
    return dict(zip(names, res.values())), other


def test_no_device_function_is_called(kernels):
    assert len(kernels[0]) > 100
    assert kernels[1] == []


def test_multi_table_kernels_meet_their_occupancy(kernels):
    """Waves per SIMD: as many as registers (512 per lane, granules of 8) and LDS (160 KB,
    blocks of one wave per SIMD) allow, at least the kernel's target."""
    seen = 0
    for name, (vgprs, lds) in kernels[0].items():
        if "k_multi<" not in name:
            continue
        solo = re.search(r"k_multi<hw::Solo<.*, (\d+)> ?>\(", name)
        waves = int(solo.group(1)) if solo else 4 if "Cfg<unsigned long, 7," in name else 6
        assert min(512 // (-(-vgprs // 8) * 8), 163840 // max(lds, 1)) >= waves, (name[:120], vgprs, lds)
        seen += 1
    assert seen >= 30


def test_slot_stores_keep_their_registers(objects):
    """A store of more than 8 bytes reads its data up to two states after it issues; written
    in inline assembly it brings them itself, whatever instruction comes next."""
    stores = 0
    for co in objects:
        text = subprocess.run([LLVM + "llvm-objdump", "-d", "--no-show-raw-insn", "--no-leading-addr", co],
                              capture_output=True, text=True, check=True).stdout.split("\n")
        for a, b in zip(text, text[1:]):
            if "global_store_dwordx4" in a and "sc1" in a:
                stores += 1
                assert b.split()[:2] == ["s_nop", "1"], (a, b)
    assert stores > 100
