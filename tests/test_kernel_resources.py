"""What the compiler made of the kernels, read from the code objects inside the built library: the prefill
kernels with hand-counted waits must not touch scratch memory, because a reload there waits for every direct
load that was issued before it."""
import re
import struct
import subprocess

from paper_2512_19720_amd import binding as pd

READELF = "/opt/rocm/llvm/bin/llvm-readelf"
EM_AMDGPU = 224


def kernels(tmp_path):
    """{mangled name: metadata text} of every kernel of the library."""
    blob = open(pd.lib()._name, "rb").read()
    out = {}
    for k, m in enumerate(re.finditer(rb"\x7fELF\x02\x01", blob)):
        if m.start() == 0 or struct.unpack_from("<H", blob, m.start() + 18)[0] != EM_AMDGPU:
            continue
        path = tmp_path / f"{k}.elf"
        path.write_bytes(blob[m.start():])
        text = subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True).stdout
        for entry in re.split(r"\n  - (?=\.)", text):
            name = re.search(r"\.symbol:\s+(\S+)\.kd", entry)
            if name:
                out[name.group(1)] = entry
    return out


def test_prefill_kernels_do_not_spill(tmp_path):
    found = {n: e for n, e in kernels(tmp_path).items() if "linear_gemm_big_kernel" in n or "linear_gemm_pipe_kernel" in n}
    assert sum("linear_gemm_big_kernel" in n for n in found) == 6            # two operand types, three kinds of scales
    for name, entry in found.items():
        assert re.search(r"\.vgpr_spill_count:\s+0\b", entry) and re.search(r"\.private_segment_fixed_size:\s+0\b", entry), name


def test_kernels_with_direct_loads_do_not_spill(tmp_path):
    found = {n: e for n, e in kernels(tmp_path).items() if "linear_skinny_dma_kernel" in n or "linear_gemm_roles_kernel" in n}
    assert len(found) == 72 + 6                                      # two operand types, three kinds of scales; 4 x 3 decode tiles
    for name, entry in found.items():
        assert re.search(r"\.vgpr_spill_count:\s+0\b", entry) and re.search(r"\.private_segment_fixed_size:\s+0\b", entry), name


# Registers that a kernel may keep in scratch memory; every other kernel none.  The variants kernels hold the sums of 16 slots
# (17 accumulators) beside what is in flight; the general prefill and gradient kernels run where no faster one does.
SPILLS = {"linear_gemm_kernel": 31, "linear_variants_slab_kernel": 76, "linear_variants_kernel": 2, "grad_tile_kernel": 5}


def test_spilled_registers_of_every_kernel(tmp_path):
    found = kernels(tmp_path)
    names = {n: re.match(r"_ZN6pdelta(\d+)", n) for n in found}
    assert all(names.values())
    seen = set()
    for name, entry in found.items():
        at = names[name].end()
        family = name[at:at + int(names[name].group(1))]
        seen.add(family)
        spilled = int(re.search(r"\.vgpr_spill_count:\s+(\d+)", entry).group(1))
        scratch = int(re.search(r"\.private_segment_fixed_size:\s+(\d+)", entry).group(1))
        # 4 bytes a lane for each spilled register, and the alignment of the area
        assert spilled <= SPILLS.get(family, 0), (name, spilled)
        assert scratch <= (4 * SPILLS[family] + 16 if family in SPILLS else 0), (name, scratch)
    assert {"grad_big_kernel", "grad_tile_pipe_kernel", "linear_skinny_kernel", "linear_skinny_staged_kernel",
            "linear_gemm_small_kernel", "pack_main_kernel", "patch_kernel"} | set(SPILLS) <= seen
