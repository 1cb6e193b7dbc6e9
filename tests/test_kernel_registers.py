"""Registers of the kernels, from the metadata of the built library (no GPU): a few registers more than a wave's share and a
compute unit holds a block less, which no result shows."""
import os
import re
import struct

import msgpack
import pytest

from paper_2210_09887_amd import binding as B

LDS = 160 * 1024


def kernels():
    """Metadata of every gfx950 kernel, by its mangled name: the notes of the code objects within the library."""
    B.lib()
    path = os.path.join(os.path.dirname(os.path.abspath(B.__file__)), "libmdcnn.so")
    data, found = open(path, "rb").read(), {}
    for m in re.finditer(b"__CLANG_OFFLOAD_BUNDLE__", data):
        n, = struct.unpack_from("<Q", data, m.start() + 24)
        p = m.start() + 32
        for _ in range(n):
            off, size, length = struct.unpack_from("<QQQ", data, p)
            if b"gfx950" in data[p + 24:p + 24 + length]:
                elf = data[m.start() + off:m.start() + off + size]
                shoff, = struct.unpack_from("<Q", elf, 40)
                shentsize, shnum = struct.unpack_from("<HH", elf, 58)
                for s in range(shnum):
                    kind, _, _, at, length_ = struct.unpack_from("<IQQQQ", elf, shoff + s * shentsize + 4)
                    if kind != 7:                                            # SHT_NOTE
                        continue
                    namesz, descsz, _ = struct.unpack_from("<III", elf, at)
                    desc = at + 12 + (namesz + 3) // 4 * 4
                    for k in msgpack.unpackb(elf[desc:desc + descsz], raw=False)["amdhsa.kernels"]:
                        found[k[".name"]] = k
            p += 24 + length
    return found


def waves_per_simd(k):
    return min(8, 512 // (-(-(k[".vgpr_count"]) // 8) * 8))                  # (.vgpr_count: both register files)


@pytest.fixture(scope="module")
def meta():
    found = kernels()
    assert len(found) > 100
    return found


def test_gather_tiles_leave_room_for_the_blocks_that_fit_the_lds(meta):
    """TiledCfg::WAVES with single buffering: as many blocks (four waves, one to a SIMD) as the LDS holds, up to four where a wave
    has one accumulator, three with two, two with four; nothing spilled to memory."""
    seen = 0
    for name, k in meta.items():
        m = re.search(r"k_conv_mfma_tiledILi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)ELi(\d+)ELi1E", name)
        if not m:
            continue
        WM, WN, TM, TN, KC = map(int, m.groups())
        BM, BN = 32 * WM * TM, 32 * WN * TN
        lds = max((BM + BN) * (KC + 8) * 2, BM * (BN + 4) * 4) + (4 * BM + 8) * 4
        want = min(LDS // lds, {1: 4, 2: 3, 4: 2}.get(TM * TN, 1))
        assert waves_per_simd(k) >= want, (name, k[".vgpr_count"], want)
        assert k[".vgpr_spill_count"] == 0 or TM * TN > 4, name
        seen += 1
    assert seen > 30


def test_stems_run_five_waves_to_a_simd(meta):
    """The 3-channel stem lives on the waves that cover its round trips."""
    stems = [k for name, k in meta.items() if "k_conv_stem_mfma" in name]
    assert len(stems) == 2
    for k in stems:
        assert waves_per_simd(k) >= 5 and k[".vgpr_spill_count"] == 0, (k[".name"], k[".vgpr_count"])


def test_convolutions_the_rules_choose_from_keep_their_registers(meta):
    """Nothing in scratch memory but in tiles that only options reach: 256-entry index ranges of 64 couts, gather tiles of eight
    accumulators or two stages."""
    for name, k in meta.items():
        option = re.search(r"k_conv_haloILi1ELi2ELi2ELi4ELi2E|k_conv_mfma_tiledILi\d+ELi\d+ELi\d+ELi\d+ELi\d+ELi2E|k_conv_mfma_tiledILi2ELi2ELi2ELi4E", name)
        assert option or k[".vgpr_spill_count"] == 0, (name, k[".vgpr_spill_count"])
