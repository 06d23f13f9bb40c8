"""What the built gfx950 code holds, from its own metadata and listing (no GPU needed)."""
import os
import re
import subprocess

import pytest

import paper_1410_1914_amd as pkg

LLVM = "/opt/rocm/llvm/bin"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects(lib, tmp):
    """Paths of the gfx950 code objects in a built library."""
    so = os.path.join(os.path.dirname(pkg.__file__), lib)
    if not os.path.exists(so):
        pytest.skip(f"{lib} is not built")
    fat = os.path.join(tmp, "fat")
    subprocess.run([f"{LLVM}/llvm-objcopy", "--dump-section", f".hip_fatbin={fat}", so, os.devnull], check=True)
    data = open(fat, "rb").read()
    starts = [m.start() for m in re.finditer(MAGIC, data)]
    out = []
    for n, (a, b) in enumerate(zip(starts, starts[1:] + [len(data)])):
        bundle, co = os.path.join(tmp, f"{n}.bundle"), os.path.join(tmp, f"{n}.co")
        with open(bundle, "wb") as f:
            f.write(data[a:b])
        subprocess.run([f"{LLVM}/clang-offload-bundler", "--type=o", "--unbundle", f"--input={bundle}", f"--output={co}",
                        "--targets=hipv4-amdgcn-amd-amdhsa--gfx950"], check=True)
        out.append(co)
    return out


def _kernels(lib, tmp):
    """{mangled name: metadata} of every kernel."""
    found = {}
    for co in _code_objects(lib, str(tmp)):
        notes = subprocess.run([f"{LLVM}/llvm-readelf", "--notes", co], check=True, capture_output=True, text=True).stdout
        for part in notes.split("  - .agpr_count:")[1:]:
            meta = dict(re.findall(r"^    \.(\w+): +(\S+)$", part, re.M))
            found[meta["name"]] = meta
    return found


def test_arguments_of_a_step_fill_one_line(tmp_path):
    """Steps of a small grid are bound by their launches, and every 64-byte line of arguments
    fetched after the first makes one longer."""
    steps = {k: v for k, v in _kernels("_liblbm.so", tmp_path).items() if "6k_stepI" in k}
    assert len(steps) == 96  # 4 x 3 tilings, 2 x 2 problems, one or several instances
    assert {int(v["kernarg_segment_size"]) for v in steps.values()} == {64}


def test_the_reach_leaves_room_for_its_own_lds(tmp_path):
    """A sheet may take 160 KB but for a kilobyte, which the kernel's own LDS has to fit."""
    sheets = [v for k, v in _kernels("_liblbm.so", tmp_path).items() if "13k_reach_sheetI" in k]
    assert len(sheets) == 4
    assert all(int(v["group_segment_fixed_size"]) <= 1024 for v in sheets)
