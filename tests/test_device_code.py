"""What the compiled kernels must contain where a missing wait could not be seen in a result for sure: checked in the
device code of the library as it was built here."""
import os
import re
import shutil
import subprocess

import pytest

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """Instructions of every kernel, by mangled name."""
    from paper_2604_10539_amd import binding
    if not os.path.exists(OBJDUMP):
        pytest.skip("no disassembler")
    d = tmp_path_factory.mktemp("device_code")
    shutil.copy(binding.LIB_PATH, d / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", "lib.so"], cwd=d, check=True, capture_output=True)  # (writes the bundles beside it)
    out = {}
    for f in sorted(os.listdir(d)):
        if not f.endswith("gfx950"):
            continue
        text = subprocess.run([OBJDUMP, "-d", f], cwd=d, check=True, capture_output=True, text=True).stdout
        name = None
        for line in text.splitlines():
            m = re.match(r"[0-9a-f]+ <(.*)>:", line)
            if m:
                name = m.group(1)
                out[name] = []
            elif name and line.strip():
                out[name].append(line.split("//")[0].strip())
    return out


def test_a_share_of_the_split_attention_arrives_after_its_stores(kernels):
    """A workgroup counts itself as arrived only once every wave's partial results have reached memory: between a wave's
    last store and the barrier in front of the arrival counter's update it waits for its vector memory operations."""
    split = {k: v for k, v in kernels.items() if "attend_split_kernel" in k}
    assert len(split) >= 8
    for name, code in split.items():
        arrive = next(i for i, x in enumerate(code) if x.startswith("global_atomic_add"))
        barrier = max(i for i in range(arrive) if code[i].startswith("s_barrier"))
        stores = [i for i in range(barrier) if re.match(r"(global|flat|buffer)_store", code[i])]
        assert any("sc1" in code[i] for i in stores), name  # (the partial results: device-scope words)
        assert not any(re.match(r"(global|flat|buffer)_store", code[i]) for i in range(barrier, arrive)), name
        assert any("s_waitcnt" in code[i] and "vmcnt(0)" in code[i] for i in range(stores[-1], barrier)), name


def test_the_assignment_keeps_its_operands_in_registers(kernels):
    """The centroid operand, the seeds and the accumulators of a wave fill the register file almost to the last; nothing of
    them goes through scratch memory in any form of the kernel."""
    assign = {k: v for k, v in kernels.items() if "13assign_kernelI" in k}
    assert len(assign) == 16  # (1, 2, 4, 8 or 16 tiles; transformed or not; 4 and more: slices that are full or not)
    for name, code in assign.items():
        assert not any(x.startswith("scratch_") for x in code), name


def test_a_later_rounds_assignment_keeps_its_operands_in_registers(kernels):
    """... and the form of a build's later rounds, which holds every form of a few centroids and the full one: nothing goes
    through scratch memory on raw keys.  On transformed keys, whose operands leave no register, a few addresses do, never
    while direct loads are on their way, which such an access would wait for."""
    later = {k: v for k, v in kernels.items() if "15reassign_kernelI" in k}
    assert len(later) == 4  # (transformed or not; slices that are full or not)
    for name, code in later.items():
        scratch = [i for i, x in enumerate(code) if x.startswith("scratch_")]
        assert len(scratch) <= (0 if "kernelILb0E" in name else 12), name
        for i in scratch:
            loads = [j for j in range(i) if "global_load_lds" in code[j]]
            waits = [j for j in range(i) if code[j].startswith("s_waitcnt") and "vmcnt(0)" in code[j]]
            assert not loads or waits[-1] > loads[-1], (name, i)


def test_the_rounds_of_large_builds_keep_their_operands_in_registers(kernels):
    """... and their three launches, by the near centroids: nothing goes through scratch memory."""
    rounds = {k: v for k, v in kernels.items() if "13marked_kernelI" in k or "11near_kernelI" in k or "17near_lists_kernelI" in k}
    assert len(rounds) == 4 + 6 + 2  # (transformed or not; slices that are full or not; a cluster in one piece, in a few, in many)
    for name, code in rounds.items():
        assert not any(x.startswith("scratch_") for x in code), name


def test_an_import_copies_through_registers(kernels):
    code = next(v for k, v in kernels.items() if "import_kernel" in k)
    assert not any(x.startswith("scratch_") for x in code)
