"""What the compiler made of the kernels, read from the built library's own code object: properties that the sources' main loops
rely on and that no result shows."""
import collections
import os
import re
import struct
import subprocess

import pytest
import yaml

from paper_2505_24034_amd import binding, build

LLVM = os.path.join(build.rocm_root(), "llvm", "bin")


def _run(tool, *args):
    return subprocess.run([os.path.join(LLVM, tool), *args], stdout=subprocess.PIPE, text=True, check=True).stdout


@pytest.fixture(scope="module")
def code_object(tmp_path_factory):
    """the gfx950 part of libllamarl.so: a bundle of (offset, size, length of the target's name, the name)"""
    data = open(build.LIB_PATH, "rb").read()
    start = data.index(b"__CLANG_OFFLOAD_BUNDLE__")
    at = start + 32
    for _ in range(struct.unpack_from("<Q", data, start + 24)[0]):
        offset, size, n = struct.unpack_from("<QQQ", data, at)
        if data[at + 24:at + 24 + n].endswith(b"gfx950"):
            path = tmp_path_factory.mktemp("code") / "gfx950.elf"
            path.write_bytes(data[start + offset:start + offset + size])
            return str(path)
        at += 24 + n
    raise AssertionError("no gfx950 code in " + build.LIB_PATH)


@pytest.fixture(scope="module")
def kernels(code_object):
    """mangled name -> the compiler's record"""
    notes = _run("llvm-readelf", "--notes", code_object)
    records = yaml.safe_load(notes[notes.index("amdhsa.kernels:"):].split("\n...")[0])
    return {k[".name"]: k for k in records["amdhsa.kernels"]}


@pytest.fixture(scope="module")
def loops(code_object):
    """mangled name -> counts of the instructions of each block that branches back to its own start"""
    out, kernel, block, counts = collections.defaultdict(list), None, None, None
    for line in _run("llvm-objdump", "-d", "--no-show-raw-insn", "--symbolize-operands", code_object).splitlines():
        if m := re.match(r"[0-9a-f]+ <(_Z\w+)>:", line):
            kernel, block, counts = m.group(1), None, collections.Counter()
        elif m := re.match(r"[0-9a-f]+ <(L\d+)>:", line):
            block, counts = m.group(1), collections.Counter()
        elif m := re.match(r"\s+([a-z]\w+) ?(\S*)", line):
            op = m.group(1)
            counts["mfma" if "mfma" in op else op.split("_")[0]] += 1
            if op.startswith("s_cbranch"):
                if m.group(2) == block:
                    out[kernel].append(counts)
                block = None                          # what follows does not belong to the loop
    return out


@pytest.mark.parametrize("kernel,scalar", [("k_fwd_partials", 52), ("k_bwd_dz", 50)])
def test_order_of_slabs_in_the_loop_of_long_contractions(loops, kernel, scalar):
    # 64 MFMAs of a wavefront a slab: 256 columns, and the narrow loop's left half.  In order 49 scalar instructions: three for each of
    # the eight requests, the waits and the barrier, addresses, the count and the branch.  The forward's ring adds two, the
    # general order (narrow loop, few columns of dz) four or five, and registers.
    found = [c["s"] for name, blocks in loops.items() if re.match(r"_ZN7llamarl\d+%sINS_8TileGemmI" % kernel, name)
             for c in blocks if c["mfma"] == 64]
    assert found
    assert min(found) <= scalar, found


def test_no_kernel_keeps_vector_registers_in_memory(kernels):
    # reloads wait for what was requested before them, a tile's first slabs for instance
    spilled = {n: (k[".vgpr_spill_count"], k[".private_segment_fixed_size"]) for n, k in kernels.items()
               if k[".vgpr_spill_count"] or k[".private_segment_fixed_size"]}
    assert not spilled


def test_two_long_contractions_in_a_launch_run_at_once(kernels):
    rules, seen = binding._load_native(), 0
    for name, k in kernels.items():
        if "k_gemm_store_pairINS_13TileGemmSplit" not in name:
            continue
        # TileGemmSplit<TileShape<four numbers>, what a CU holds of it by itself, ..> of dH and dW, the second abbreviated if equal
        own = [int(n) for n in re.findall(r"ILi\dELi\dELi\dELi\dEEELi(\d)E", name)]
        h, w = own if len(own) == 2 else 2 * own
        held = 512 // (-(-k[".vgpr_count"] // 8) * 8)          # a workgroup is a wavefront on each SIMD, of 512 registers
        for cus in (256, 255, 8, 1):
            assert rules.pair_workgroups(cus, h, w, 1, 1) + rules.pair_workgroups(cus, w, h, 1, 1) <= cus * held, name
        seen += 1
    assert seen == 8


def test_bf16_dH_is_built_in_its_one_output_form(kernels):
    # k_gemm_store<TileGemmTN.., MODE>: a bf16 dH is stored in bf16 and never added to what is there (MODE 3)
    modes = {re.match(r"_ZN7llamarl12k_gemm_storeINS_\d+TileGemmTN(?:Small.*EEE|E)Li(\d)E", n).group(1)
             for n in kernels if "k_gemm_storeINS_10TileGemmTNE" in n or "k_gemm_storeINS_15TileGemmTNSmall" in n}
    assert modes == {"3"}
