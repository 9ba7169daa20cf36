"""What the compiler gave the kernels of the built library (the metadata of its gfx950 code objects): registers that do not spill
where a kernel also carries a rare path, and the residency that the host's rules count on."""
import re
import struct

import msgpack
import pytest

from paper_2605_23200_amd import binding as B


def _kernels(path):
    """[(name, template arguments, metadata)] of every gfx950 kernel in the library's offload bundles."""
    data = open(path, "rb").read()
    out, at = [], data.find(b"__CLANG_OFFLOAD_BUNDLE__")
    while at >= 0:
        p = at + 32
        for _ in range(struct.unpack_from("<Q", data, at + 24)[0]):
            off, size, n = struct.unpack_from("<QQQ", data, p)
            if b"gfx950" in data[p + 24:p + 24 + n] and size:
                elf = data[at + off:at + off + size]
                sections, = struct.unpack_from("<Q", elf, 0x28)
                entry, count = struct.unpack_from("<HH", elf, 0x3A)
                for s in range(sections, sections + entry * count, entry):
                    if struct.unpack_from("<I", elf, s + 4)[0] == 7:                       # SHT_NOTE
                        note, = struct.unpack_from("<Q", elf, s + 24)
                        name, desc = struct.unpack_from("<II", elf, note)
                        start = note + 12 + (name + 3) // 4 * 4
                        for k in msgpack.unpackb(elf[start:start + desc])["amdhsa.kernels"]:
                            m = re.search(r"\d([a-z][a-z_]*_kernel)(?:I((?:L[bi]\d+E)+)E)?", k[".name"])
                            args = tuple(int(x) for x in re.findall(r"L[bi](\d+)E", m[2] or ""))
                            out.append((m[1], args, k))
            p += 24 + n
        at = data.find(b"__CLANG_OFFLOAD_BUNDLE__", at + 24)
    return out


@pytest.fixture(scope="module")
def kernels():
    B.lib()
    found = _kernels(B.LIB_PATH)
    assert len(found) > 100
    return found


def _spills(kernels, name):
    return {args: k[".vgpr_spill_count"] for n, args, k in kernels if n == name}


def test_tails_cost_the_first_sweep_no_registers(kernels):
    """Causal instances carry the tails of the units next to the plain blocks: they spill no more than those without."""
    spills = _spills(kernels, "score_stats_kernel")         # bf16, column blocks, causal, moments, channels, keys
    causal = {a: n for a, n in spills.items() if a[2]}
    assert len(causal) >= 24
    worse = {a: (n, spills[a[:2] + (0,) + a[3:]]) for a, n in causal.items() if n > spills[a[:2] + (0,) + a[3:]]}
    assert not worse


def test_small_tiles_of_the_one_launch_scorer_leave_a_cu_two_workgroups(kernels):
    """512 threads each: 128 registers, half of the LDS (the query window comes on top, NB * 32 rows)."""
    small = {a: k for n, a, k in kernels if n == "score_unit_kernel" and a[0] and a[1] <= (2 if a[3] == 64 else 1)}
    assert len(small) == 18                                 # bf16, column blocks, mode, channels, cuts
    for a, k in small.items():
        assert k[".vgpr_count"] <= 128 and 2 * (k[".group_segment_fixed_size"] + a[1] * 32 * (a[3] * 2 + 16)) <= 160 * 1024, a


def test_tails_cost_the_second_sweep_no_registers(kernels):
    """bf16 caches: the fp32 instances of 65 to 128 queries and 128 channels fill all 256 registers without a tail."""
    spills = _spills(kernels, "score_usage_kernel")         # bf16, column blocks, mode, causal, channels, keys, fold
    causal = {a: n for a, n in spills.items() if a[0] and a[3]}
    assert len(causal) >= 50
    worse = {a: (n, spills[a[:3] + (0,) + a[4:]]) for a, n in causal.items() if n > spills[a[:3] + (0,) + a[4:]]}
    assert not worse


def test_every_kernel_is_in_the_library_once(kernels):
    names = [k[".name"] for _, _, k in kernels]
    assert sorted({n for n in names if names.count(n) > 1}) == []
