"""What the compiler made of the sweep kernels, on the CPU: their gfx950
assembly, built from the sources with the library's own flags."""
import os
import re
import subprocess

import pytest

from paper_2407_14675_amd import build


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """source -> {kernel symbol: assembly}."""
    def compiled(source):
        out = tmp_path_factory.mktemp("asm") / (source + ".s")
        subprocess.run([build.HIPCC, *build.FLAGS, "-S", "--cuda-device-only", os.path.join(build.CSRC, source), "-o",
                        str(out)], check=True, stderr=subprocess.DEVNULL)
        text = out.read_text()
        found = {m[1]: m[0] for m in re.finditer(r"\n(_Z\w+):[^\n]*\n.*?\n\.Lfunc_end", text, re.S)}
        # the kernel's record (registers, spills) after its code
        for m in re.finditer(r"\.name:\s+(_Z\w+)\n.*?\.wavefront_size", text, re.S):
            found[m[1]] += m[0]
        assert found
        return found

    return {s: compiled(s) for s in ("dpo_batch.hip", "dpo_kernels.hip")}


@pytest.mark.parametrize("source,name,count", [("dpo_batch.hip", "k_batch_sweep", 2), ("dpo_kernels.hip", "k_sweep_fast", 4)])
def test_sweeps_address_global_memory(kernels, source, name, count):
    """No flat access, which cannot take a scalar base and waits on the LDS counter too."""
    found = {k: v for k, v in kernels[source].items() if name in k}
    assert len(found) == count
    for k, text in found.items():
        assert len(re.findall(r"\tglobal_load", text)) > 10, k
        assert not re.findall(r"\tflat_\w+", text), k


def test_no_wave_waits_for_the_angle_table(kernels):
    """The scan + golden and seeded sweeps have the residual's barriers and no other."""
    barriers = [len(re.findall(r"\ts_barrier", kernels["dpo_kernels.hip"][f"_ZN3dpo12k_sweep_fastILi{m}EEEvNS_9SweepArgsE"]))
                for m in (0, 1, 2)]
    assert barriers[0] > 0 and barriers[1] == barriers[2] == barriers[0]


@pytest.mark.parametrize("source,name,count", [("dpo_batch.hip", "k_batch_sweep", 2), ("dpo_kernels.hip", "k_sweep_fast", 4)])
def test_sweeps_spill_nothing(kernels, source, name, count):
    """Neither vector registers to scratch nor scalar ones to lanes of vector registers."""
    found = {k: v for k, v in kernels[source].items() if name in k}
    assert len(found) == count
    for k, text in found.items():
        for what in ("vgpr_spill_count", "sgpr_spill_count", "private_segment_fixed_size"):
            assert re.search(r"\.%s:\s+(\d+)" % what, text)[1] == "0", (k, what)
