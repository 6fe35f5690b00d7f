"""What can be told from the built library's own device code, without a GPU.  No kernel keeps registers in scratch memory.  And what
the compiler does not check in statements written as assembly: a DPP operand must not be read within two wait states of its being
written by a vector instruction."""
import glob
import os
import re
import shutil
import subprocess

import pytest

OBJDUMP, READELF = "/opt/rocm/llvm/bin/llvm-objdump", "/opt/rocm/llvm/bin/llvm-readelf"
REG = re.compile(r"^v(?:\[(\d+):(\d+)\]|(\d+))$")


def _regs(op):
    m = REG.match(op.strip().lstrip("-|").rstrip("|"))
    if not m:
        return set()
    lo, hi = (int(m[1]), int(m[2])) if m[1] else (int(m[3]), int(m[3]))
    return set(range(lo, hi + 1))


def _too_close(listing):
    """Lines whose DPP operand was written fewer than two wait states before (in the order of the listing)."""
    bad, seen, found = [], [], 0
    for line in listing.splitlines():
        line = line.split("//")[0].strip()
        if not line or line.endswith(":"):
            continue
        op, _, rest = line.partition(" ")
        args = rest.split(",")
        if op.startswith("v_") and (op.endswith("_dpp") or "row_newbcast" in rest):
            found += 1
            src, waited = _regs(args[1].split()[0]), 0
            for prev, prev_args in reversed(seen):
                if waited >= 2:
                    break
                if prev.startswith("v_") and _regs(prev_args[0]) & src:
                    bad.append(line)
                    break
                waited += int(prev_args[0]) + 1 if prev == "s_nop" else 1
        seen = (seen + [(op, args)])[-4:]
    return bad, found


def test_the_scan_sees_a_distance_that_is_too_short():
    close = "v_add_f64 v[2:3], v[4:5], v[6:7]\ns_nop 0\nv_fmac_f64_dpp v[0:1], v[2:3], v[8:9] row_newbcast:1 row_mask:0xf bank_mask:0xf\n"
    assert _too_close(close)[0] and not _too_close(close.replace("s_nop 0", "s_nop 1"))[0]


@pytest.fixture(scope="module")
def device_objects(tmp_path_factory):
    if not os.path.exists(OBJDUMP):
        pytest.skip("no llvm-objdump")
    from paper_2510_03246_amd import strp
    if not os.path.exists(strp.LIB_PATH):
        import __graft_entry__
        __graft_entry__.build()
    tmp_path = tmp_path_factory.mktemp("device")
    lib = shutil.copy(strp.LIB_PATH, tmp_path / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", str(lib)], check=True, capture_output=True, cwd=tmp_path)
    return sorted(glob.glob(str(tmp_path / "*gfx950*")))


def test_no_kernel_uses_scratch(device_objects):
    kernels = {}
    for obj in device_objects:
        notes = subprocess.run([READELF, "--notes", obj], check=True, capture_output=True, text=True).stdout
        for entry in notes.split("- .agpr_count")[1:]:
            fields = dict(re.findall(r"^ *\.(name|private_segment_fixed_size|vgpr_spill_count): +(\S+)$", entry, re.M))
            kernels[fields["name"]] = (int(fields["private_segment_fixed_size"]), int(fields["vgpr_spill_count"]))
    assert len(kernels) > 50
    assert not {k: v for k, v in kernels.items() if v != (0, 0)}


def test_dpp_operands_are_read_two_wait_states_after_they_were_written(device_objects):
    found = 0
    for obj in device_objects:
        bad, n = _too_close(subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", obj], check=True, capture_output=True, text=True).stdout)
        assert not bad, bad[:5]
        found += n
    assert found > 300      # the factorisation chain's broadcasts are among them
