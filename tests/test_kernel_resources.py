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
    "ls_score.hip": ["stats_kernel", "range_stats_kernel", "merge_kernel", "lines_kernel", "diagonals_kernel", "finish_kernel"],
    "ls_select.hip": ["order_kernel", "walk_kernel", "walk_exact_kernel", "emit_kernel", "merge_lines_kernel", "topb_one_kernel"],
}


@pytest.mark.parametrize("source", NO_SCRATCH)
def test_registers_stay_out_of_memory(tmp_path, source):
    """Arrays of registers that are picked from by a computed index, or more values than registers, end in scratch memory: every
    instance of these kernels has none, and every kernel named here is there."""
    out = tmp_path / "source.s"
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    subprocess.run([hipcc, *build.FLAGS, "--cuda-device-only", "-S", os.path.join(build.CSRC, source), "-o", str(out)],
                   check=True, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)
    scratch = {}
    for kernel in out.read_text().split("  - .agpr_count:")[1:]:
        name = re.search(r"^\s*\.name:\s+(\S+)", kernel, flags=re.M)[1]
        scratch[name] = int(re.search(r"^\s*\.private_segment_fixed_size:\s+(\d+)", kernel, flags=re.M)[1])
    for name in NO_SCRATCH[source]:
        instances = {n: s for n, s in scratch.items() if re.search(rf"\d{name}(E|I)", n)}
        assert instances, name
        assert set(instances.values()) == {0}, instances
