"""What the compiler gave the kernels whose chains of dependent steps must not go through memory."""
import os
import re
import subprocess

from paper_2507_13681_amd import build


def test_walks_keep_their_registers_out_of_memory(tmp_path):
    """The greedy loops pick one entry of an array of registers by a computed index; kept in registers, the walks need no
    scratch memory."""
    out = tmp_path / "select.s"
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    subprocess.run([hipcc, *build.FLAGS, "--cuda-device-only", "-S", os.path.join(build.CSRC, "ls_select.hip"), "-o", str(out)],
                   check=True, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)
    scratch = {}
    for kernel in out.read_text().split("  - .agpr_count:")[1:]:
        name = re.search(r"^\s*\.name:\s+(\S+)", kernel, flags=re.M)[1]
        scratch[name] = int(re.search(r"^\s*\.private_segment_fixed_size:\s+(\d+)", kernel, flags=re.M)[1])
    walks = {n: s for n, s in scratch.items() if re.search(r"\d(walk_kernel|walk_exact_kernel|sort_seg_kernel|sort_merge_kernel|emit_kernel|topb_one_kernel)", n)}
    assert len(walks) >= 5
    assert set(walks.values()) == {0}, walks
