"""The kernels with hand-placed LDS waits are only correct for compiler output in which nothing touches the
destination registers of an LDS read before the wait that covers it.  These CPU tests pin the compiler version
that was validated, run the static check on what this compiler generates, and show on small planted mistakes
that the check sees what it is meant to see."""
import os
import re
from concurrent.futures import ThreadPoolExecutor

import pytest

from paper_2407_12075_amd import asm_check, build as hip_build


def test_hipcc_is_the_validated_version():
    text = hip_build.hipcc_version()
    assert hip_build.VALIDATED_HIP_VERSION in text and hip_build.VALIDATED_CLANG in text, (
        "hipcc differs from the version the inline-assembly LDS reads were validated with "
        f"({hip_build.VALIDATED_HIP_VERSION}, {hip_build.VALIDATED_CLANG}); run `python -m paper_2407_12075_amd.asm_check` "
        "and the GPU tests with the new compiler, then update paper_2407_12075_amd/build.py.\n" + text)


def test_generated_assembly_has_no_early_use_of_pending_reads():
    srcs = [os.path.join(hip_build.CSRC, s) for s in asm_check.CHECKED_SOURCES]
    with ThreadPoolExecutor(max_workers=4) as ex:
        texts = list(ex.map(asm_check.compile_to_asm, srcs))
    for src, text in zip(srcs, texts):
        names, findings = asm_check.check_asm_text(text)
        assert names, f"no kernel found in the assembly of {src}"
        followed = sum(l.startswith("ds_read") and not l.endswith(asm_check._MANAGED) for body in asm_check._split_kernels(text).values() for l in body)
        assert followed >= 20, f"{src}: {followed} reads placed by hand"
        assert not findings, f"{src}:\n" + "\n".join(findings[:20])


_GOOD = """
kernel_a:
    s_load_dwordx2 s[0:1], s[4:5], 0x0
    s_waitcnt lgkmcnt(0)
    ds_read_b128 v[4:7], v1
    ds_read_b128 v[8:11], v1 offset:16
    v_add_u32_e32 v2, v2, v3
    s_waitcnt lgkmcnt(1)
    v_mfma_f32_32x32x16_bf16 a[0:15], v[4:7], v[12:15], a[0:15]
    s_waitcnt lgkmcnt(0)
    v_mfma_f32_32x32x16_bf16 a[0:15], v[8:11], v[12:15], a[0:15]
    s_endpgm
    .end_amdhsa_kernel
"""


def _check(text):
    names, findings = asm_check.check_asm_text(text)
    assert names == ["kernel_a"]
    return findings


def test_checker_accepts_correct_waits():
    assert _check(_GOOD) == []


@pytest.mark.parametrize("old,new,what", [
    # the wait that covers the first read lets one more read stay pending: the MFMA reads v[4:7] too early
    ("s_waitcnt lgkmcnt(1)", "s_waitcnt lgkmcnt(2)", "touches registers of a pending LDS read"),
    # a register copy out of a pending read (what a compiler-inserted move would look like)
    ("v_add_u32_e32 v2, v2, v3", "v_mov_b32_e32 v20, v9", "touches registers of a pending LDS read"),
    # an LDS read whose address register is the destination of a read that is still pending
    ("ds_read_b128 v[8:11], v1 offset:16", "ds_read_b128 v[8:11], v5 offset:16", "uses registers of a pending LDS read"),
    # a scalar load shares the counter but returns out of order
    ("v_add_u32_e32 v2, v2, v3", "s_load_dword s6, s[0:1], 0x0", "scalar load"),
    # reads still in flight at the end of the program
    ("    s_waitcnt lgkmcnt(0)\n    v_mfma_f32_32x32x16_bf16 a[0:15], v[8:11], v[12:15], a[0:15]\n", "", "pending at s_endpgm"),
])
def test_checker_sees_planted_mistakes(old, new, what):
    assert old in _GOOD
    findings = _check(_GOOD.replace(old, new))
    assert any(what in f for f in findings), findings


def test_checker_follows_branches():
    # the read is pending on the path that skips the wait
    text = """
kernel_a:
    ds_read_b128 v[4:7], v1
    s_cbranch_scc1 .LBB0_2
    s_waitcnt lgkmcnt(0)
.LBB0_2:
    v_add_f32_e32 v8, v4, v4
    s_waitcnt lgkmcnt(0)
    s_endpgm
    .end_amdhsa_kernel
"""
    assert any("touches registers" in f for f in _check(text))


# As hipcc writes it: reads placed by hand between markers, one of the compiler's own (v[16:19]) with a wait of its own.
_MARKED = """
kernel_a:
    ds_read_b128 v[16:19], v2
    ;;#ASMSTART
    ds_read_b128 v[4:7], v1
    ;;#ASMEND
    ;;#ASMSTART
    ds_read_b128 v[8:11], v1 offset:16
    ;;#ASMEND
    s_waitcnt lgkmcnt(2)
    v_add_f32_e32 v20, v16, v17
    ;;#ASMSTART
    s_waitcnt lgkmcnt(0)
    ;;#ASMEND
    v_mfma_f32_32x32x16_bf16 a[0:15], v[4:7], v[8:11], a[0:15]
    ds_read_b32 v3, v2
    s_waitcnt lgkmcnt(0)
    s_endpgm
    .end_amdhsa_kernel
"""


def test_checker_tells_reads_placed_by_hand_from_the_compilers():
    assert _check(_MARKED) == []
    # a read of the compiler's own is not followed: its use is the compiler's business
    assert _check(_MARKED.replace("lgkmcnt(2)", "lgkmcnt(3)")) == []
    assert _check(_MARKED.replace("    ds_read_b32 v3, v2\n    s_waitcnt lgkmcnt(0)\n", "    ds_read_b32 v3, v2\n")) == []
    # without the markers every read is
    bare = "\n".join(l for l in _MARKED.splitlines() if "#ASM" not in l)
    assert _check(bare) == []
    assert any("touches registers" in f for f in _check(bare.replace("lgkmcnt(2)", "lgkmcnt(3)")))


@pytest.mark.parametrize("old,new,what", [
    # the product in front of the wait, and behind one that leaves the second read pending
    ("s_waitcnt lgkmcnt(0)\n    ;;#ASMEND\n    v_mfma", "s_nop 0\n    ;;#ASMEND\n    v_mfma", "touches registers of a pending LDS read"),
    ("s_waitcnt lgkmcnt(0)\n    ;;#ASMEND\n    v_mfma", "s_waitcnt lgkmcnt(1)\n    ;;#ASMEND\n    v_mfma", "touches registers of a pending LDS read"),
    # the compiler's instruction, inside or outside the markers, on a register of a pending read
    ("v_add_f32_e32 v20, v16, v17", "v_mov_b32_e32 v20, v9", "touches registers of a pending LDS read"),
    # a read of the compiler's own: its destination, then its address in registers of a pending one
    ("    s_waitcnt lgkmcnt(2)\n", "    ds_read_b32 v5, v2\n    s_waitcnt lgkmcnt(3)\n", "uses registers of a pending LDS read"),
    ("    s_waitcnt lgkmcnt(2)\n", "    ds_read_b32 v22, v10\n    s_waitcnt lgkmcnt(3)\n", "uses registers of a pending LDS read"),
    # a read by hand behind one of the compiler's own that has not landed either: the wait counts both
    ("    s_waitcnt lgkmcnt(2)\n", "    ds_read_b32 v22, v2\n    s_waitcnt lgkmcnt(1)\n    v_mov_b32_e32 v21, v8\n    v_mov_b32_e32 v23, v4\n    s_waitcnt lgkmcnt(0)\n", None),
    ("    s_waitcnt lgkmcnt(2)\n", "    ds_read_b32 v22, v2\n    s_waitcnt lgkmcnt(2)\n    v_mov_b32_e32 v21, v8\n    s_waitcnt lgkmcnt(0)\n", "touches registers of a pending LDS read"),
])
def test_checker_sees_planted_mistakes_between_markers(old, new, what):
    assert _MARKED.count(old) == 1
    findings = _check(_MARKED.replace(old, new))
    assert any(what in f for f in findings) if what else findings == [], findings


def test_tile_kernel_requests_a_chunk_before_the_products_of_the_one_before():
    """The bfloat16 kernel with one wave per 32 rows has one chunk in flight: its loads have to stand before the loop's matrix
    instructions, where the compiler does not leave them by itself."""
    text = asm_check.compile_to_asm(os.path.join(hip_build.CSRC, "tbn_linear_tile.hip"))
    loops = 0
    for name, lines in asm_check._split_kernels(text).items():
        if "linear_tile_kernelIt" not in name:
            continue
        block = []
        for line in lines + [".LBB_end:"]:
            if not line.startswith(".L"):
                block.append(line)
                continue
            loads = [i for i, l in enumerate(block) if l.startswith("global_load_dwordx")]
            products = [i for i, l in enumerate(block) if l.startswith("v_mfma")]
            if loads and products:
                loops += 1
                assert loads[-1] < products[0], f"{name}: loads behind the first of {len(products)} matrix instructions"
            block = []
    assert loops == 12   # with and without ReLU, one and two column tiles, one, four and eight slices of K


def test_float32_tile_kernel_keeps_the_plain_loop_for_few_columns_with_k_split():
    """One column tile with four or eight slices of K and two with eight are faster without the pipeline over steps."""
    text = asm_check.compile_to_asm(os.path.join(hip_build.CSRC, "tbn_linear_tile.hip"))
    built = {tuple(map(int, m)) for m in re.findall(r"linear_tile_kernelIfLb[01]ELi(\d)ELi(\d)ELi(\d)E", text)}   # column tiles, slices, chunks ahead
    split = {(nt, kw, 0 if (nt, kw) in {(1, 4), (1, 8), (2, 8)} else 1) for nt in (1, 2, 3, 4) for kw in (4, 8)}
    assert built == split | {(nt, 1, ahead) for nt in (1, 2, 3, 4) for ahead in (1, 2)}


def test_scalars_of_sign_bits_out_are_loaded_without_branches():
    """The 64 x 64 blocks with sign bits out load eight scalars per lane; a branch around each, for layers with a single one, makes eight round
    trips of them.  (Such a branch loads the single one by a scalar load.)"""
    text = asm_check.compile_to_asm(os.path.join(hip_build.CSRC, "tbn_binact.hip"))
    bodies = [b for n, b in asm_check._split_kernels(text).items() if "binact_staged_kernelIfLb0ELb1E" in n]
    assert len(bodies) == 2 and not any(l.startswith("s_load_dword ") for b in bodies for l in b)


def test_registers_that_lanes_are_read_from_are_held_in_all_lanes():
    """The kernels on sign bits keep the scalar of replica t in lane t and read it by v_readlane where only some lanes may be on.  Behind the
    products, where all are, the source marks the register as used; the marked register has to be the one that is read, every narrowing of
    the execution mask between the last product and the mark undone, and nothing may load the register again behind it."""
    text = asm_check.compile_to_asm(os.path.join(hip_build.CSRC, "tbn_binact.hip"))
    checked = 0
    functions = re.split(r"^(_Z\w+):.*$", text, flags=re.M)      # what stands before the first, then name, text, name, text ...
    for body in zip(functions[1::2], functions[2::2]):
        lines = re.split(r"^\s*\.section", body[1], maxsplit=1, flags=re.M)[0].splitlines()
        if not re.search(r"binact_(?:mfma|staged)_kernel", body[0]):
            continue
        read = {re.search(r"v_readlane_b32 \S+ (v\d+)", l).group(1) for l in lines if "v_readlane_b32" in l}
        if not read:
            continue
        marks = [i for i, l in enumerate(lines) if "held in all lanes:" in l]
        last = max(i for i, l in enumerate(lines) if l.strip().startswith("v_mfma"))
        assert len(marks) == 1 and read == {lines[marks[0]].split(":")[1].strip()}, (body[0], read)
        between = lines[last:marks[0]]
        masks = [l for l in between if "_saveexec" in l or re.match(r"\s*s_or_b64 exec, exec,", l)]
        assert marks[0] > last and not any("s_endpgm" in l for l in between) and not ("_saveexec" in masks[-1] if masks else False), body[0]
        register = lines[marks[0]].split(":")[1].strip()
        assert not any(re.match(r"\s*(?!v_readlane)\S+ " + register + r"\b", l) for l in lines[marks[0] + 1:]), body[0]
        checked += 1
    assert checked == 13   # nine of the 128 x 128 blocks, four of the 64 x 64 with real outputs
