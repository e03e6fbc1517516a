"""Registers and scratch of the built kernels, read from the code objects inside libtwilight.so: where a dispatch rule
counts on several workgroups per compute unit, the kernel has to fit them (512 vector registers per lane of a SIMD,
allocated in eights; 4 SIMDs; a 1024-thread workgroup is 4 waves on each)."""
import os
import re
import struct
import subprocess

import pytest

msgpack = pytest.importorskip("msgpack")


@pytest.fixture(scope="module")
def kernels():
    """{demangled name: metadata} of every kernel in the library."""
    import paper_2502_02770_amd as T
    if not os.path.exists(T.binding.LIB_PATH):
        from paper_2502_02770_amd.build import build
        build(verbose=False)
    blob = open(T.binding.LIB_PATH, "rb").read()
    found, magic = {}, b"__CLANG_OFFLOAD_BUNDLE__"
    at = blob.find(magic)
    while at >= 0:
        n, = struct.unpack_from("<Q", blob, at + len(magic))
        pos = at + len(magic) + 8
        for _ in range(n):
            off, size, idlen = struct.unpack_from("<QQQ", blob, pos)
            name = blob[pos + 24:pos + 24 + idlen]
            pos += 24 + idlen
            if b"gfx950" in name:
                elf = blob[at + off:at + off + size]
                for k in _metadata(elf):
                    found[k[".name"]] = dict(k, elf=elf)
        at = blob.find(magic, at + 1)
    names = list(found)
    plain = subprocess.run(["c++filt"], input="\n".join(names), capture_output=True, text=True, check=True).stdout.splitlines()
    return {re.sub(r"^void |\(anonymous namespace\)::|\(.*$", "", p.replace("(anonymous namespace)::", "")): found[n] for n, p in zip(names, plain)}


def _metadata(elf):
    """amdhsa.kernels of a code object: the AMDGPU note (type 32) of its note sections."""
    shoff, = struct.unpack_from("<Q", elf, 40)
    shentsize, shnum = struct.unpack_from("<HH", elf, 58)
    for i in range(shnum):
        _, kind, _, _, off, size = struct.unpack_from("<IIQQQQ", elf, shoff + i * shentsize)
        if kind != 7:
            continue
        end = off + size
        while off < end:
            namesz, descsz, ntype = struct.unpack_from("<III", elf, off)
            desc = off + 12 + (namesz + 3 & ~3)
            if ntype == 32:
                return msgpack.unpackb(elf[desc:desc + descsz], strict_map_key=False)["amdhsa.kernels"]
            off = desc + (descsz + 3 & ~3)
    return []


def _fits(k, workgroups):
    """Do `workgroups` workgroups of the kernel's size share a compute unit by its vector registers?"""
    regs = (k[".vgpr_count"] + 7) // 8 * 8
    waves = k[".max_flat_workgroup_size"] // 64
    return (waves * workgroups + 3) // 4 * regs <= 512


@pytest.mark.parametrize("unit", [16, 1])
@pytest.mark.parametrize("slots", [8, 16])
def test_selection_of_up_to_16384_entries_runs_two_workgroups_per_cu(kernels, slots, unit):
    k = kernels["page_select_reg_kernel<1024, %d, %d>" % (slots, unit)]
    assert _fits(k, 2), k[".vgpr_count"]


@pytest.mark.parametrize("bits", [2, 4, 8])
@pytest.mark.parametrize("candidates,workgroups,spilled", [(8, 4, 8), (16, 3, 0)])
def test_one_launch_pruner_of_many_heads_shares_the_cu(kernels, candidates, workgroups, spilled, bits):
    """The launch bounds make the registers fit, by spilling if need be: what they may spill is what was measured to pay."""
    for G in (1, 2, 4, 8):
        k = kernels["topp_head_kernel<512, %d, %d, false, 2, %d>" % (candidates, G, bits)]
        assert _fits(k, workgroups), k[".vgpr_count"]
        assert k[".vgpr_spill_count"] <= spilled and k[".private_segment_fixed_size"] <= (0 if not spilled else 68 if G == 1 else 36)
        assert k[".group_segment_fixed_size"] * workgroups <= 160 * 1024


@pytest.mark.parametrize("bits", [2, 4, 8])
@pytest.mark.parametrize("threads,workgroups", [(512, 4), (256, 8)])
def test_one_launch_pruner_of_short_lists_fills_the_cu(kernels, threads, workgroups, bits):
    """4 candidates per thread: 64 registers, every wave slot of the CU taken."""
    for G in (1, 2, 4, 8):
        k = kernels["topp_head_kernel<%d, 4, %d, false, 2, %d>" % (threads, G, bits)]
        assert _fits(k, workgroups), k[".vgpr_count"]
        assert k[".group_segment_fixed_size"] * workgroups <= 160 * 1024


def test_pruner_kernels_without_a_spill(kernels):
    """All but the forms that four to a CU are paid for with (8 candidates per thread in LDS), which the test above bounds."""
    heads = {n: k for n, k in kernels.items() if n.startswith("topp_head_kernel") and not re.search(r"<512, 8, \d, false, 2, ", n)}
    spilled = {n: (k[".vgpr_spill_count"], k[".private_segment_fixed_size"]) for n, k in heads.items()}
    assert len(spilled) > 100 and not any(v != (0, 0) for v in spilled.values()), {n: v for n, v in spilled.items() if v != (0, 0)}


def test_the_selection_kernels_spill_no_vector_registers(kernels):
    spilled = {n: k[".vgpr_spill_count"] for n, k in kernels.items() if n.startswith("page_select")}
    assert len(spilled) == 14 and not any(spilled.values()), spilled


@pytest.mark.parametrize("dots,pages", [(False, 4), (True, 2)])
def test_scoring_of_two_heads_per_page_keeps_its_waves(kernels, dots, pages):
    """4-bit codes, every page a candidate, two query heads per KV head: eight waves per SIMD with the integer dots stored, six
    with four pages in flight."""
    k = kernels["int4_score_kernel<2, true, %s, %d, 4>" % ("true" if dots else "false", pages)]
    assert _fits(k, 8 if dots else 6), k[".vgpr_count"]
    assert not k[".vgpr_spill_count"] and not k[".private_segment_fixed_size"]


@pytest.mark.parametrize("tokens", ["false", "true"])
def test_top_p_on_stored_scores_reads_its_arguments_once(kernels, tokens, tmp_path):
    """These forms hold all arguments in scalar registers from the start.  Read again behind the search's barriers they were 23 to 31
    scalar loads instead of 12, each a trip to the scalar cache in a chain of phases: 256 heads' token lists 8.0 us instead of 7.55."""
    for shape in ("512, 4", "512, 8", "1024, 4", "1024, 8"):
        k = kernels["topp_head_kernel<%s, 4, %s, 0, 4>" % (shape, tokens)]
        assert not k[".sgpr_spill_count"]
        (tmp_path / "code").write_bytes(k["elf"])
        out = subprocess.run([os.environ.get("LLVM_OBJDUMP", "/opt/rocm/llvm/bin/llvm-objdump"), "-d", "--disassemble-symbols=" + k[".name"], str(tmp_path / "code")],
                             capture_output=True, text=True, check=True).stdout
        assert "s_endpgm" in out
        assert len(re.findall(r"\bs_load_dword", out)) <= 16, shape


def test_forms_that_share_a_cu_spill_few_scalar_registers(kernels):
    """Four workgroups of 8 candidates per thread to a CU: 21, 40 with the arguments of the last phases held; all other forms of the
    one-launch pruner none, up to 16 so."""
    spilled = {n: k[".sgpr_spill_count"] for n, k in kernels.items() if n.startswith("topp_head_kernel")}
    four = {n: v for n, v in spilled.items() if re.search(r"<512, 8, \d, false, 2, ", n)}
    assert len(four) == 12 and max(four.values()) <= 24, four
    assert not any(v for n, v in spilled.items() if n not in four), {n: v for n, v in spilled.items() if v}
