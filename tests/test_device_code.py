"""The machine code the build makes for gfx950: wait states between vector compares and the selects that read their masks."""
import os
import re
import subprocess

import pytest

from paper_1804_08378_amd import build

BIN = "/opt/rocm/lib/llvm/bin"
WAIT_STATES = 2  # between a vector instruction that writes a lane mask (VCC or a scalar pair) and a vector instruction that reads it


def device_code(obj: str, tmp: str) -> str:
    """File with the device code inside an object that build() made."""
    bundle, code = os.path.join(tmp, "bundle"), os.path.join(tmp, "code")
    subprocess.run([f"{BIN}/llvm-objcopy", f"--dump-section=.hip_fatbin={bundle}", obj, os.path.join(tmp, "rest.o")], check=True)
    subprocess.run([f"{BIN}/clang-offload-bundler", "--type=o", "--unbundle", f"--input={bundle}",
                    "--targets=hipv4-amdgcn-amd-amdhsa--gfx950", f"--output={code}"], check=True)
    return code


def disassemble(obj: str, tmp: str) -> str:
    return subprocess.run([f"{BIN}/llvm-objdump", "-d", "--no-show-raw-insn", "--no-leading-addr", device_code(obj, tmp)], check=True,
                          capture_output=True, text=True).stdout


def mask_reads(lines):
    """(line, wait states since the vector compare that wrote its mask) of every select; straight-line code only: what a jump
    lands on is not followed."""
    written, now = {}, 0
    for line in lines:
        op, _, rest = line.partition(" ")
        if not op or op.endswith(":") or op.startswith(("s_branch", "s_cbranch", "s_setpc", "s_swappc")):
            written.clear()
            continue
        args = [a.strip() for a in rest.split("//")[0].split(",")]
        if op.startswith("v_cndmask"):
            mask = args[3] if len(args) > 3 else "vcc"
            if mask in written:
                yield line, now - written[mask] - 1
        now += int(args[0], 0) + 1 if op == "s_nop" else 1
        if op.startswith("v_cmp") and not op.startswith("v_cmpx"):
            written[args[0]] = now - 1
        elif args[0] in written:  # written by something else (a scalar instruction: no wait states)
            del written[args[0]]


@pytest.mark.parametrize("source", [s for s in build.SOURCES if s.endswith(".hip")])
def test_selects_wait_for_the_compares_that_write_their_masks(source, tmp_path):
    """The compiler keeps the wait states in its own code; it does not look inside asm blocks."""
    build.build(force=False)
    obj = os.path.join(build.HERE, "_build", source + ".o")
    if not os.path.exists(obj) or not os.path.exists(BIN):
        pytest.skip("needs the build's objects and the ROCm toolchain")
    text = disassemble(obj, str(tmp_path))
    lines = [re.sub(r"\s+", " ", l).strip() for l in text.split("\n")]
    pairs, short = 0, []
    for line, states in mask_reads(lines):
        pairs += 1
        if states < WAIT_STATES:
            short.append((states, line))
    print(f"{source}: {pairs} compare-select pairs")
    assert not short, (len(short), short[:5])


@pytest.mark.parametrize("source", ["bs_backward.hip", "bs_backward_strip.hip", "bs_chain.hip", "bs_chain_nhwc.hip", "bs_nhwc.hip", "bs_kernels.hip", "bs_chain_window.hip",
                                    "bs_chain_window_nhwc.hip", "bs_pool_band.hip"])
def test_kernels_keep_nothing_in_scratch_memory(source, tmp_path):
    """The factors of up to four residual gradients, rings and row buffers are arrays that must become registers."""
    build.build(force=False)
    obj = os.path.join(build.HERE, "_build", source + ".o")
    if not os.path.exists(obj) or not os.path.exists(BIN):
        pytest.skip("needs the build's objects and the ROCm toolchain")
    notes = subprocess.run([f"{BIN}/llvm-readelf", "--notes", device_code(obj, str(tmp_path))], check=True, capture_output=True, text=True).stdout
    sizes = re.findall(r"\.name:\s+(_Z\w+).*?\.private_segment_fixed_size:\s+(\d+)", notes, re.S)
    assert sizes
    scratch = [(name, int(n)) for name, n in sizes if int(n)]
    assert not scratch, (len(scratch), scratch[:5])


@pytest.mark.parametrize("source,kernel,instances", [
    # storage type, levels, columns of a row beyond whole vectors
    ("bs_chain_window.hip", "chain_window_kernel", {(0, l, r) for l in range(2, 11) for r in range(4)} | {(1, l, r) for l in range(4, 11) for r in range(4)}),
    # storage type, channels of a vector, levels
    ("bs_chain_window_nhwc.hip", "chain_window_nhwc_kernel", {(d, v, l) for d in range(3) for v in (1, 4) for l in range(4, 11)}),
    # storage type, maximum?, window, padding, picks?
    ("bs_pool_band.hip", "pool_band_kernel", {(d, 1, 3, p, i) for d in range(3) for p in (0, 1) for i in (0, 1)} | {(0, m, 2, 0, 0) for m in (0, 1)}),
])
def test_only_instances_that_a_plan_reaches_are_compiled(source, kernel, instances, tmp_path):
    """The planner's rules keep some types and sizes with other kernels: no machine code for those."""
    build.build(force=False)
    obj = os.path.join(build.HERE, "_build", source + ".o")
    if not os.path.exists(obj) or not os.path.exists(BIN):
        pytest.skip("needs the build's objects and the ROCm toolchain")
    notes = subprocess.run([f"{BIN}/llvm-readelf", "--notes", device_code(obj, str(tmp_path))], check=True, capture_output=True, text=True).stdout
    args = re.findall(r"\.name:\s+_Z\w*?" + kernel + r"I((?:L[ib]\d+E)+)E", notes)
    assert len(args) == len(instances) and {tuple(int(v) for v in re.findall(r"L[ib](\d+)E", a)) for a in args} == instances


def test_audit_builds_check_every_access_of_the_backward_strip_kernels():
    """bs_bwd_device.h says that a build with -DBS_BWD_AUDIT checks every offset into the three tensors: each load and store of the
    strip kernels passes its offset through the check, runs of elements with their length, and such a build compiles."""
    text = open(os.path.join(build.CSRC, "bs_backward_strip.hip")).read()
    accesses = re.findall(r"^.*\b(?:load_run|store_run|store_elems)<.*$", text, re.M)
    assert len(accesses) >= 4
    for line in accesses:
        assert "audited_bytes<" in line, line.strip()
    helpers = open(os.path.join(build.CSRC, "bs_bwd_device.h")).read()
    assert "uint64_t)off + n" in helpers and "template <typename OFF>\nBS_DEV OFF audited" in helpers  # 64-bit offsets, too
    # nothing else in the file reads or writes through a pointer of the argument block (k.params: the parameter table)
    code = re.sub(r"//.*", "", text)
    assert not re.search(r"k\.(?:a|g_out|g_in)\s*\[|\*\s*k\.(?:a|g_out|g_in)\b", code)
