"""What the built library's own device code has to hold, read from its disassembly (no GPU needed)."""
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
OBJDUMP, READOBJ = "/opt/rocm/llvm/bin/llvm-objdump", "/opt/rocm/llvm/bin/llvm-readobj"


@pytest.fixture(scope="module")
def code_objects(tmp_path_factory):
    """The gfx950 code objects of libfineserve.so."""
    lib = os.path.join(ROOT, "paper_2509_06261_amd", "libfineserve.so")
    if not os.path.exists(OBJDUMP) or not os.path.exists(lib):
        pytest.skip("llvm-objdump or the built library not found")
    tmp = tmp_path_factory.mktemp("device_code")
    lib = shutil.copy(lib, tmp)
    subprocess.run([OBJDUMP, "--offloading", lib], check=True, cwd=tmp, stdout=subprocess.DEVNULL)
    found = [os.path.join(tmp, name) for name in sorted(os.listdir(tmp)) if name.endswith("gfx950")]
    assert found
    return found


@pytest.fixture(scope="module")
def kernels(code_objects):
    """{kernel name: its instructions in order}."""
    found = {}
    for path in code_objects:
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", "--no-leading-addr", path], check=True, stdout=subprocess.PIPE,
                              text=True).stdout
        for part in re.split(r"^<", text, flags=re.M)[1:]:
            head, _, body = part.partition(">:")
            found[head] = [line.split("//")[0].strip() for line in body.splitlines() if line.strip()]
    return found


def test_decode_and_column_kernels_hold_their_scalars(code_objects):
    """Scalars parked in vector registers cost the smallest calls, which run every instruction once: the tile code of all
    formats is in one kernel per head_dim, and one format's look-ups must not push out what the others hold."""
    if not os.path.exists(READOBJ):
        pytest.skip("llvm-readobj not found")
    spills = {}
    for path in code_objects:
        notes = subprocess.run([READOBJ, "--notes", path], check=True, stdout=subprocess.PIPE, text=True).stdout
        for kernel in re.split(r"^  - \.a", notes, flags=re.M)[1:]:
            name = re.search(r"^\s+\.name:\s+(\S+)", kernel, flags=re.M)
            spills[name.group(1)] = (int(re.search(r"\.sgpr_spill_count:\s+(\d+)", kernel).group(1)),
                                     int(re.search(r"\.vgpr_spill_count:\s+(\d+)", kernel).group(1)))
    most = {"mfma_direct_kernelILi64E": 8, "mfma_direct_kernelILi128E": 4, "mfma_direct_kernelILi256E": 8, "mfma_attention_kernelILi64E": 0,
            "mfma_attention_kernelILi128E": 0, "mfma_attention_kernelILi256E": 0, "prefill_kernelILi64E": 28, "prefill_kernelILi128E": 28,
            "prefill_kernelILi256E": 28}
    for key, limit in most.items():
        found = [v for k, v in spills.items() if key in k]
        assert len(found) == 1 and found[0][0] <= limit and found[0][1] == 0, (key, found)


def test_pieces_are_complete_before_they_are_counted(kernels):
    """Prefill kernels with split items: a wave's stores of its piece go to where all XCDs see them (sc1, agent scope), the
    wave waits for its own stores before the barrier in front of the count (a barrier waits for none), and the pieces are read
    from there as well; or the piece is written back and invalidated as a whole by every wave."""
    split = {k: v for k, v in kernels.items() if "prefill_wg_kernel" in k and any("cmpswap_x2" in i for i in v)}
    assert len(split) == 4  # one for each format
    for name, code in split.items():
        count = next(i for i, x in enumerate(code) if "cmpswap_x2" in x)
        before = max(i for i in range(count) if code[i] == "s_barrier")
        stores = [i for i in range(before) if code[i].startswith("global_store")][-32:]
        wait = code[stores[-1] + 1 : before]
        assert any(x.startswith("s_waitcnt vmcnt(0)") for x in wait), name
        assert all(code[i].endswith(" sc1") for i in stores) or "buffer_wbl2 sc1" in wait, name
        after = min(i for i in range(count, len(code)) if code[i] == "s_barrier")
        loads = [i for i in range(after, len(code)) if code[i].startswith("global_load")][:32]
        assert all(code[i].endswith(" sc1") for i in loads) or "buffer_inv sc1" in code[after : loads[0]], name
