"""The kernels wait for their global -> LDS transfers before every barrier that publishes them, on every path of the built code.

The transfers are asm statements, which the compiler does not count among the memory operations it waits for, and a
barrier of gfx950 does not wait for vector memory by itself: a transfer still in flight there could land in LDS that other
waves have taken for something else.  Which waits the compiler happens to put elsewhere must not decide that.
"""
import os
import re
import subprocess

import pytest

from paper_2507_13681_amd import build


def _blocks(lines):
    """Straight-line pieces of a kernel: label -> (instructions, labels that control may go to)."""
    blocks, name, body, fall = {}, "entry", [], True
    for line in lines:
        text = line.split(";")[0].strip()
        label = re.match(r"([.\w$]+):$", text)
        if label:
            blocks[name] = (body, [label[1]] if fall else [])
            name, body, fall = label[1], [], True
        elif text and not text.startswith(".") and fall:
            branch = re.match(r"s_c?branch(_\w+)?\s+(\S+)", text)
            if branch:                                     # the piece ends here; what follows is one of its own
                follow = f"{name}+"
                always = text.startswith("s_branch")
                blocks[name] = (body, [branch[2]] + ([] if always else [follow]))
                name, body, fall = follow, [], not always
            elif text.startswith("s_endpgm"):
                fall = False
            else:
                body.append(text)
    blocks[name] = (body, [])
    return blocks


def _barriers_with_a_transfer_in_flight(lines):
    """How many barriers can be reached with a transfer that no vmcnt(0) came after."""
    blocks = _blocks(lines)
    at_entry = {"entry": False}
    todo, bad = ["entry"], set()
    while todo:
        name = todo.pop()
        flying = at_entry[name]
        body, nexts = blocks[name]
        for i, ins in enumerate(body):
            if "_load_lds_" in ins:
                flying = True
            elif ins.startswith("s_waitcnt") and "vmcnt(0)" in ins:
                flying = False
            elif ins.startswith("s_barrier") and flying:
                bad.add((name, i))
        for n in nexts:
            if n in blocks and (n not in at_entry or flying and not at_entry[n]):
                at_entry[n] = flying
                todo.append(n)
    return len(bad)


def test_path_search_sees_a_missing_wait():
    """The search itself: a transfer on one of two paths, with and without a wait behind it."""
    code = ["s_cbranch_scc1 .L1", "global_load_lds_dwordx4 v[0:1], off", ".L1:", "s_waitcnt lgkmcnt(0)", "s_barrier", "s_endpgm"]
    assert _barriers_with_a_transfer_in_flight(code) == 1
    assert _barriers_with_a_transfer_in_flight(code[:3] + ["s_waitcnt vmcnt(0)"] + code[3:]) == 0
    loop = [".L0:", "s_barrier", "global_load_lds_dwordx4 v[0:1], off", "s_cbranch_scc1 .L0", "s_endpgm"]
    assert _barriers_with_a_transfer_in_flight(loop) == 1


# source: kernels, by the beginning of their names, their instances, and barriers that leave the next chunk of query rows under way
# on purpose: they order LDS that no transfer fills (the slab of diagonals, the rows' reduction)
KERNELS = {
    "ls_decode.hip": [("decode_kernelI", 4, 0)],
    "ls_prefill.hip": [("prefill_bf16_kernelI", 4, 0)],
    "ls_score.hip": [("stats_kernelI", 4, 1), ("range_stats_kernelI", 4, 1), (r"lines_kernelI\w+Li0ELb", 8, 1), (r"lines_kernelI\w+Li4ELb", 8, 1), (r"lines_kernelI\w+Li[123]ELb", 24, 0)],
}


@pytest.mark.parametrize("source", KERNELS)
def test_kernels_wait_before_their_barriers(tmp_path, source):
    out = tmp_path / "source.s"
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    subprocess.run([hipcc, *build.FLAGS, "--cuda-device-only", "-S", os.path.join(build.CSRC, source), "-o", str(out)],
                   check=True, stdout=subprocess.PIPE, stderr=subprocess.STDOUT)
    kernels, current = {}, []
    for line in out.read_text().splitlines():
        start = re.match(r"(_ZN2ls\w+):", line)
        if start:
            kernels[start[1]] = current = []
        elif line.startswith(".Lfunc_end"):
            current = []
        else:
            current.append(line)
    seen = set()
    for name, instances, in_flight in KERNELS[source]:
        found = {k: v for k, v in kernels.items() if re.match(rf"_ZN2ls\d+{name}", k)}
        assert len(found) == instances, (name, list(found))
        for k, lines in found.items():
            assert any("_load_lds_" in x for x in lines) and any("s_barrier" in x for x in lines), k
            assert _barriers_with_a_transfer_in_flight(lines) == in_flight, k
        seen |= set(found)
    # no other kernel of the source has transfers
    assert not [k for k, lines in kernels.items() if k not in seen and any("_load_lds_" in x for x in lines)]
