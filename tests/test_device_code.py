"""What the compiler made of the kernels that count their own waits, read from the built library (no GPU)."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2311_15806_amd", "libpipe_hip.so")
OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
KERNEL = re.compile(r"gemm_bins_kernelILi(\d)ELi(\d)ELi(\d)ELi(\d)ELb([01])ELi(\d)ELi(\d)E")   # bits, token blocks, waves, mode, conv, groups, ahead


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """{name of a kernel: its instructions}"""
    if not os.path.exists(OBJDUMP):
        pytest.skip("no llvm-objdump")
    there = tmp_path_factory.mktemp("code")
    lib = shutil.copy(LIB, there / "lib.so")     # (the code objects are extracted beside it)
    subprocess.run([OBJDUMP, "--offloading", lib], check=True, capture_output=True)
    out = {}
    for obj in there.glob("lib.so.*gfx950"):
        names = subprocess.run([OBJDUMP, "--syms", str(obj)], check=True, capture_output=True, text=True).stdout
        if "gemm_bins_kernel" not in names and "gemm_stream_kernel" not in names:
            continue
        name = None
        for line in subprocess.run([OBJDUMP, "-d", "--mcpu=gfx950", str(obj)], check=True, capture_output=True, text=True).stdout.splitlines():
            head = re.match(r"[0-9a-f]+ <(\S+)>:", line)
            if head:
                name = head.group(1)
                out[name] = []
            elif name is not None and line.startswith("\t"):
                out[name].append(line.split("//")[0].strip())
    return out


def _runs(code):
    """The stretches of a kernel without a barrier or a branch."""
    at = 0
    for i, ins in enumerate(code):
        if ins.startswith(("s_barrier", "s_cbranch", "s_branch", "s_endpgm")):
            yield code[at:i]
            at = i + 1


def test_stages_wait_for_nothing_in_flight(kernels):
    """Single-pass kernel with two stages in flight: a stage that multiplies and requests never waits for the loads of the stage after
    it, which are as many as it requests itself -- neither before its first multiply nor behind it."""
    checked = 0
    for name, code in kernels.items():
        m = KERNEL.search(name)
        if m is None or m.group(7) != "2" or m.group(5) == "1":     # (a convolution's stages branch between loads)
            continue
        stages = 0
        for body in _runs(code):
            loads = sum(ins.startswith(("buffer_load", "global_load")) for ins in body)
            if loads == 0 or not any(ins.startswith("v_mfma") for ins in body):
                continue
            stages += 1
            waits = [int(v) for ins in body for v in re.findall(r"vmcnt\((\d+)\)", ins)]
            assert waits and min(waits) >= loads, (m.groups(), waits, loads)
            assert not any(ins.startswith("scratch_") for ins in body), m.groups()
        assert stages >= 3, m.groups()
        checked += 1
    assert checked >= 20


def test_gathers_are_as_many_as_the_loads_they_replace(kernels):
    """A convolution's stage requests each fragment at one place, at an address that was ready before (whether or not a stage has several
    taps): its kernel holds no more loads into LDS than the one for patches that lie in memory."""
    count = {}
    for name, code in kernels.items():
        m = KERNEL.search(name)
        if m is not None and m.group(4) == "0":
            count[m.groups()] = sum(ins.startswith("buffer_load") and ins.endswith(" lds") for ins in code)
    convolutions = [k for k in count if k[4] == "1"]
    assert len(convolutions) >= 9
    for k in convolutions:
        plain = k[:4] + ("0",) + k[5:]
        assert 0 < count[k] <= count[plain], (k, count[k], count[plain])


def test_streaming_kernel_raises_a_slot_once(kernels):
    """The maxima of a workgroup's outputs reach a member's slot by one raise per side, not by one per wave, row block and member."""
    counts = {name: sum("atomic" in ins and "max" in ins for ins in code) for name, code in kernels.items()
              if re.search(r"gemm_stream_kernelILi\dELi\dELi\dELb0E", name)}
    plain = [name for name in counts if "StreamPlain" in name]       # the instance of few arguments takes no maxima
    assert len(plain) == 4 and not any(counts.pop(name) for name in plain)
    assert len(counts) >= 9 and all(0 < c <= 2 for c in counts.values()), counts


def test_streaming_kernel_asks_for_two_tiles_at_8_bits(kernels):
    """Its instances for two tiles at a time: both stand before the loop and in it, and the loop waits once for both."""
    found = {name: code for name, code in kernels.items() if re.search(r"gemm_stream_kernelILi8E.*ELb0ENS_12StreamParamsELi2EE", name)}
    assert len(found) == 4
    for name, code in found.items():
        assert sum(ins.startswith("buffer_load_dwordx4") for ins in code) == 2 * 2 * 5, name
        first = next(i for i, ins in enumerate(code) if ins.startswith("v_mfma"))
        assert any("vmcnt(0)" in ins for ins in code[first - 4:first]), name
    wide = {name: code for name, code in kernels.items() if re.search(r"gemm_stream_multi_kernelILi8ELi8ELi1E", name)}
    assert len(wide) == 3
    for name, code in wide.items():
        assert sum(ins.startswith("global_load_dwordx4") for ins in code) >= 2 * 2 * 5, name
