"""Registers of built kernels: what the key loop of the window backward holds must not go to scratch memory, because a reload
waits together with the tile loads in flight."""
import os
import re
import subprocess

from paper_2602_10016_amd import build

LLVM = "/opt/rocm/llvm/bin/"


def metadata(source, tmp_path, field):
    """Mangled kernel name -> a number of the metadata of the object that was built from `source`."""
    build.build()
    bundle, code = tmp_path / "bundle", tmp_path / "code"
    subprocess.run([LLVM + "llvm-objcopy", "--dump-section", f".hip_fatbin={bundle}", os.path.join(build.OBJ, source.replace(".hip", ".o")), os.devnull],
                   check=True)
    subprocess.run([LLVM + "clang-offload-bundler", "--type=o", "--unbundle", f"--input={bundle}", "--targets=hipv4-amdgcn-amd-amdhsa--gfx950",
                    f"--output={code}"], check=True)
    notes = subprocess.run([LLVM + "llvm-readelf", "--notes", str(code)], check=True, capture_output=True, text=True).stdout
    return {name: int(n) for name, n in re.findall(r"\.name: +(\S+)\n(?:(?!\.name).)*?\." + field + r": +(\d+)", notes, flags=re.S)}


def spilled_vector_registers(source, tmp_path):
    return metadata(source, tmp_path, "vgpr_spill_count")


def test_the_window_backward_keeps_its_registers(tmp_path):
    spilled = {n: s for n, s in spilled_vector_registers("attn_bwd_tiled_mfma.hip", tmp_path).items() if re.search(r"bwd_(dq|dkdv)_kernel", n)}
    assert len(spilled) == 35 and not any(spilled.values()), spilled


def test_tile_tables_cost_the_backward_no_registers_of_the_other_mappings(tmp_path):
    """115 since before there was another mapping; 118 with the search for an example in the same kernel."""
    found = {n: r for n, r in metadata("attn_bwd_tiled_mfma.hip", tmp_path, "vgpr_count").items() if "bwd_dkdv_kernelILi32ELi4ELb0E" in n}
    assert len(found) == 2 and min(found.values()) <= 115, found


def test_the_search_for_an_example_costs_no_workgroup_per_compute_unit(tmp_path):
    """Query-tiled forward, tiles by offsets (mapping 2) beside by tables (0): 512 registers per SIMD, granted by eights."""
    found = metadata("attn_fwd_ring_mfma.hip", tmp_path, "vgpr_count")
    for d in (32, 64, 128):
        tables, offsets = ([512 // ((r + 7) // 8 * 8) for n, r in found.items() if f"qtile_fwd_mfma_kernelILi{d}ELi4ELi2ELb0ELi{m}E" in n] for m in (0, 2))
        assert len(tables) == 1 and tables == offsets, (d, found)
