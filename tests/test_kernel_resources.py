"""What the compiler gave the kernels whose chains of dependent steps must not go through memory."""
import os
import re
import subprocess

import pytest

from paper_2507_13681_amd import build

# the kernels of a source, by the beginning of their names, that must do without scratch memory
NO_SCRATCH = {
    "ls_decode.hip": ["decode_kernel"],
    "ls_prefill.hip": ["plan_kernel", "sched_kernel", "prefill_bf16_kernel", "combine_kernel"],
    "ls_score.hip": ["stats_kernel", "range_stats_kernel", "merge_kernel", "lines_kernel", "retain_kernel", "diagonals_kernel", "finish_kernel"],
    "ls_select.hip": ["order_kernel", "walk_kernel", "walk_exact_kernel", "emit_kernel", "redo_kernel", "merge_lines_kernel", "topb_one_kernel"],
}


# instances of which a CU is to have so many waves on each of its SIMDs at once, by what their names contain: 512 registers are shared by them
WAVES = {"ls_score.hip": {"lines_kernelINS_6bf16_t": 4}, "ls_select.hip": {"emit_kernelILb0E": 8}}


def _kernels(tmp_path, source):
    """Of each kernel of the source, what the assembler is told about it."""
    out = tmp_path / "source.s"
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    subprocess.run([hipcc, *build.FLAGS, "--cuda-device-only", "-S", os.path.join(build.CSRC, source), "-o", str(out)],
                   check=True, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)
    return {re.search(r"^\s*\.name:\s+(\S+)", k, flags=re.M)[1]: k for k in out.read_text().split("  - .agpr_count:")[1:]}


def _field(kernel, name):
    return int(re.search(rf"^\s*\.{name}:\s+(\d+)", kernel, flags=re.M)[1])


@pytest.mark.parametrize("source", NO_SCRATCH)
def test_registers_stay_out_of_memory(tmp_path, source):
    """Arrays of registers that are picked from by a computed index, or more values than registers, end in scratch memory: every
    instance of these kernels has none, and every kernel named here is there.  Kernels whose launches fill the chip by several workgroups a CU leave them the registers."""
    kernels = _kernels(tmp_path, source)
    for name in NO_SCRATCH[source]:
        instances = {n: _field(k, "private_segment_fixed_size") for n, k in kernels.items() if re.search(rf"\d{name}(E|I)", n)}
        assert instances, name
        assert set(instances.values()) == {0}, instances
    for name, waves in WAVES.get(source, {}).items():
        instances = {n: _field(k, "vgpr_count") for n, k in kernels.items() if name in n}
        assert instances, name
        assert max(instances.values()) <= 512 // waves // 8 * 8, instances
