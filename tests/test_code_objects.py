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
    assert len(steps) == 144  # 4 x 3 tilings, 2 x 2 problems, whole, in blocks of planes, several instances
    assert {int(v["kernarg_segment_size"]) for v in steps.values()} == {64}


def test_whole_d3q19_steps_take_no_ranges(tmp_path):
    """The 8 ranges of a block of planes (16 bytes each) are arguments of its steps alone."""
    steps = {k: int(v["kernarg_segment_size"]) for k, v in _kernels("_liblbm.so", tmp_path).items() if "k_d3q19I" in k}
    cut = [n for k, n in steps.items() if "D19CutArgs" in k]
    assert len(steps) == 6 and len(cut) == 2  # 2 problems: whole, measured, in blocks of planes
    assert {n + 128 for k, n in steps.items() if "D19CutArgs" not in k} == set(cut)


def test_the_reach_leaves_room_for_its_own_lds(tmp_path):
    """A sheet may take 160 KB but for a kilobyte, which the kernel's own LDS has to fit."""
    sheets = [v for k, v in _kernels("_liblbm.so", tmp_path).items() if "13k_reach_sheetI" in k]
    assert len(sheets) == 4
    assert all(int(v["group_segment_fixed_size"]) <= 1024 for v in sheets)


def _steps(lib, tmp, kernel):
    """What each step between two barriers issues, in the listing's order: {name: [string]} with
    s stores, c copies into LDS, m matrix products, l other loads (scalar ones apart)."""
    out = {}
    for co in _code_objects(lib, str(tmp)):
        text = subprocess.run([f"{LLVM}/llvm-objdump", "-d", "--no-show-raw-insn", co], check=True, capture_output=True,
                              text=True).stdout
        for name, body in re.findall(r"^[0-9a-f]+ <(\S+)>:\n(.*?)(?=^[0-9a-f]+ <|\Z)", text, re.M | re.S):
            if kernel not in name:
                continue
            ops = ""
            for line in body.splitlines():
                op = line.split()[0] if line.split() else ""
                if op == "s_barrier":
                    ops += "|"
                elif "_store_" in op:
                    ops += "s"
                elif op.startswith(("buffer_load", "global_load", "flat_load")):
                    ops += "c" if " lds" in line else "l"
                elif op.startswith("v_mfma"):
                    ops += "m"
            out[name] = ops.split("|")[1:]  # from the first barrier on
    return out


def test_marching_convolutions_wait_for_what_they_issue(tmp_path):
    """A step of the marching form waits until no more than two planes' stores and copies are
    out: its body has to issue the plane's stores (4, or 1 with the head), then its copies (a
    tile's halo in 16-byte pieces over 256 threads), then 56 products, and nothing of one step
    may have moved into another."""
    kernels = _steps("_libunet.so", tmp_path, "12k_conv_marchI")
    assert len(kernels) == 8
    for name, steps in kernels.items():
        s, head, mask, xg = (int(v) for v in re.search(r"ILi(\d)ELb(\d)ELb(\d)ELi(\d)E", name).groups())
        pieces = 2 * (16 * xg + 2) * (16 // (s * xg) + 2)
        copies = -(-pieces // 256)
        assert len(steps) == 4, name  # the loop's, the last one up to the kernel's end
        for body in steps:
            before = "l*" if head or mask else ""  # the head's base, the mask
            assert re.match(f"{before}s{{{1 if head else 4}}}c{{{copies}}}m{{56}}", body), (name, body)
        for body in steps[:3]:
            assert re.fullmatch("l*s*c*m{56}s{0,4}", body), (name, body)  # the FP32 results may follow


def test_ring_convolutions_wait_for_what_they_issue(tmp_path):
    """A step of the ring waits by the copies and the weights fetched since its plane's: three
    copies, then the plane's products, then 0, 4 or 5 chunks of weights."""
    (steps,) = _steps("_libunet.so", tmp_path, "11k_conv_ringI").values()
    assert len(steps) == 12  # six planes, in the first stage and in the others
    for n, body in enumerate(steps[:-1]):
        k = n % 6
        products = (16, 36, 56, 56, 40, 20)[k]
        weights = (0, 0, 0, 4, 5, 5)[k]
        # a copy may be listed twice, once for either source
        m = re.fullmatch(f"(c+)(m{{{products}}})(l{{{weights}}})", body)
        assert m and 3 <= len(m.group(1)) <= 6, (n, body)
