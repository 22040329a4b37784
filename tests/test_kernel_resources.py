"""What the built kernels take of the machine, from the notes that the compiler leaves in the library: no register of theirs is kept in
scratch memory, and those whose speed rests on how many of their waves run at a time leave room for them."""
import os
import re
import subprocess

import pytest

from paper_2605_12245_amd import build

LLVM = os.path.join(os.path.dirname(os.path.dirname(os.path.realpath(build.HIPCC))), "lib", "llvm", "bin")


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """name -> notes of every kernel"""
    at = tmp_path_factory.mktemp("notes")
    run = lambda *cmd: subprocess.run(cmd, check=True, stdout=subprocess.PIPE, stderr=subprocess.PIPE, text=True).stdout
    run("objcopy", "-O", "binary", "--only-section=.hip_fatbin", build.OUT, str(at / "fatbin"))
    run(f"{LLVM}/clang-offload-bundler", "--unbundle", "--type=o", "--targets=hipv4-amdgcn-amd-amdhsa--gfx950", f"--input={at}/fatbin",
        f"--output={at}/code")
    notes = run(f"{LLVM}/llvm-readelf", "--notes", str(at / "code"))
    found = {}
    for entry in notes.split("  - .agpr_count:")[1:]:
        name = run("c++filt", re.search(r"\.name:\s+(\S+)", entry)[1]).strip()
        name = re.sub(r"^void |\(anonymous namespace\)::", "", name)
        found[name[:name.rindex("(")]] = {k: int(v) for k, v in re.findall(r"\.(\w+):\s+(\d+)\s", entry)}
    assert len(found) > 40
    return found


def test_no_register_of_a_batch_kernel_lies_in_scratch_memory(kernels):
    batch = {k: v for k, v in kernels.items() if k.startswith("k_resident_batch<")}
    assert len(batch) == 8
    assert not {k: v for k, v in batch.items() if v["vgpr_spill_count"] or v["private_segment_fixed_size"]}


def test_no_register_of_the_shared_launch_of_the_later_iterations_lies_in_scratch_memory(kernels):
    """and as many of its workgroups are on a compute unit as deal_shares gives shares to: 512 registers a lane and four workgroups' waves share a SIMD"""
    rest = {k: v for k, v in kernels.items() if k.startswith("k_iter_rest<")}
    assert len(rest) == 6
    assert not {k: v for k, v in rest.items() if v["vgpr_spill_count"] or v["private_segment_fixed_size"]}
    for name, v in rest.items():
        closed = "(Iterate)0" in name or "CLOSED_FORM" in name
        assert 512 // (-(-v["vgpr_count"] // 8) * 8) >= (6 if closed else 5), name
        assert 160 * 1024 // (v["group_segment_fixed_size"] + 2048 * 4 * (not closed)) >= (6 if closed else 5), name


def test_an_mxfp4_search_of_one_tile_has_no_place_for_more(kernels):
    """the kernel for workgroups of one tile stages no sums: LDS for the trees only"""
    lds = {k: v["group_segment_fixed_size"] for k, v in kernels.items() if k.startswith("k_mx<")}
    assert len(lds) == 10
    staged = {k for k in lds if k.endswith("true>")}
    assert len(staged) == 2 and all(lds[k] > 8 * 1024 for k in staged)
    assert all(v < 4 * 1024 for k, v in lds.items() if k not in staged and "(Mx)0" not in k)
