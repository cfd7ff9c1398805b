"""What the compiler made of the kernels, from the metadata of the built library: registers, LDS and scratch that
the launch rules and the figures in the comments count on."""
import re
import struct

import pytest

import paper_2410_18248_amd as P

msgpack = pytest.importorskip("msgpack")


def _code_objects(blob):
    """The gfx950 code objects in the clang offload bundles of a host library."""
    for m in re.finditer(b"__CLANG_OFFLOAD_BUNDLE__", blob):
        base = m.start()
        n, = struct.unpack_from("<Q", blob, base + 24)
        at = base + 32
        for _ in range(n):
            off, size, length = struct.unpack_from("<QQQ", blob, at)
            triple = blob[at + 24:at + 24 + length]
            at += 24 + length
            if b"gfx950" in triple and size:
                yield blob[base + off:base + off + size]


def _metadata(elf):
    """The kernels of the AMDGPU metadata note."""
    phoff, = struct.unpack_from("<Q", elf, 32)
    phentsize, phnum = struct.unpack_from("<HH", elf, 54)
    for i in range(phnum):
        kind, = struct.unpack_from("<I", elf, phoff + i * phentsize)
        offset, = struct.unpack_from("<Q", elf, phoff + i * phentsize + 8)
        size, = struct.unpack_from("<Q", elf, phoff + i * phentsize + 32)
        at = offset
        while kind == 4 and at < offset + size:                          # PT_NOTE
            namesz, descsz, note = struct.unpack_from("<III", elf, at)
            desc = at + 12 + (namesz + 3) // 4 * 4
            if note == 32 and elf[at + 12:at + 18] == b"AMDGPU":
                return msgpack.unpackb(elf[desc:desc + descsz])["amdhsa.kernels"]
            at = desc + (descsz + 3) // 4 * 4
    return []


@pytest.fixture(scope="module")
def kernels():
    found = {k[".name"]: k for co in _code_objects(open(P.lib_path(), "rb").read()) for k in _metadata(co)}
    assert len(found) > 60
    return found


def _prefill(kernels):
    """(D, tiled, columns, stages per barrier, split) -> metadata."""
    out = {}
    for name, k in kernels.items():
        m = re.search(r"prefill_mfmaILi(\d+)ELb(\d)ELi(\d+)ELi(\d+)ELb(\d)E", name)
        if m:
            out[tuple(int(x) for x in m.groups())] = k
    assert len(out) >= 18
    return out


def _workgroups(k):
    """Workgroups of 256 threads a CU holds: 512 registers per lane and SIMD in steps of 8, 160 KiB of LDS."""
    regs = (k[".vgpr_count"] + 7) // 8 * 8               # (accumulation registers are counted in)
    return min(512 // regs, (160 << 10) // max(k[".group_segment_fixed_size"], 1))


def test_nothing_spills_into_a_loop(kernels):
    """A handful of values may go out before a kernel's loop and come back behind it; a reload inside waits for
    every load on its way."""
    for name, k in kernels.items():
        assert k[".private_segment_fixed_size"] <= 16, (name, k[".private_segment_fixed_size"])


def test_prefill_workgroups_per_cu(kernels):
    """Launches of up to 512 workgroups count on two per CU, except those with tiles of 128 columns of head size
    256, which are dealt their tiles in order for that."""
    for (D, tiled, cols, stages, split), k in _prefill(kernels).items():
        assert (_workgroups(k) >= 2) == (not (D >= 256 and cols > 16)), (D, tiled, cols, stages, split, k[".vgpr_count"])
    for name, k in kernels.items():
        if "prefill_tiles_f32" in name:
            assert _workgroups(k) >= 2, name


def test_decode_workgroups_per_cu(kernels):
    """A launch is as wide as the chip holds of it: what the loops of the plain-layout reducers need, and no less for the
    plan in front of them."""
    least = {"Lb1ELi8ELi1ELi2EEELb0": 6, "Lb1ELi8ELi1ELi2EEELb1": 5, "Lb0ELi8ELi1ELi2EEELb0": 7, "Lb0ELi8ELi1ELi2EEELb1": 6,
             "Lb0ELi8ELi2ELi2EEELb0": 5, "Lb0ELi8ELi2ELi2EEELb1": 5, "Lb0ELi8ELi4ELi1EEELb0": 5, "Lb0ELi8ELi4ELi1EEELb1": 5}
    seen = 0
    for name, k in kernels.items():
        m = re.search(r"decode_balanced.*ValuReducerI(\w+?)EEEvNS", name)
        if m:
            assert _workgroups(k) >= least.get(m.group(1), 4), (name, k[".vgpr_count"])
            seen += m.group(1) in least
    assert seen == len(least)


def test_cut_decode_workgroups_per_cu(kernels):
    """The spare workgroups of a launch that cuts ranges, 1 024 on the vector path and 512 on the matrix path, are about what the chip holds at once."""
    seen = 0
    for name, k in kernels.items():
        m = re.search(r"decode_cut.*(Valu|Mfma)ReducerI(\w+?)EE", name)
        if m:
            assert _workgroups(k) >= (4 if m.group(1) == "Valu" else 1 if "256" in m.group(2) else 2), (name, k[".vgpr_count"])
            seen += 1
    assert seen == 15


def test_teams_have_a_cu_to_themselves_and_no_scratch(kernels):
    """Two waves of a workgroup to a SIMD; and the waits for the loads of a stage count every load and store, which one to scratch memory
    between them would be."""
    seen = [k for name, k in kernels.items() if "prefill_teams" in name]
    assert len(seen) == 4
    for k in seen:
        assert k[".vgpr_count"] <= 256 and k[".private_segment_fixed_size"] == 0, k[".name"]
