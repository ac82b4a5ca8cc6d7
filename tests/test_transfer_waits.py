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
    """Straight-line pieces of a kernel: label -> (instructions, labels that control may go to, and for a branch, to the first of them, on what)."""
    blocks, name, body, fall = {}, "entry", [], True
    for line in lines:
        text = line.split(";")[0].strip()
        label = re.match(r"([.\w$]+):$", text)
        if label:
            blocks[name] = (body, [label[1]] if fall else [], "")
            name, body, fall = label[1], [], True
        elif text and not text.startswith(".") and fall:
            branch = re.match(r"s_c?branch(_\w+)?\s+(\S+)", text)
            if branch:                                     # the piece ends here; what follows is one of its own
                follow = f"{name}+"
                always = text.startswith("s_branch")
                blocks[name] = (body, [branch[2]] + ([] if always else [follow]), (branch[1] or "")[1:])
                name, body, fall = follow, [], not always
            elif text.startswith("s_endpgm"):
                fall = False
            else:
                body.append(text)
    blocks[name] = (body, [], "")
    return blocks


MANY = 64                                                  # more than the counter of outstanding operations holds


def _transfers_at_barriers(lines):
    """Barriers that can be reached with transfers in flight: (piece, place in it) -> how many of a wave, at most.  A wait for vmcnt(N) leaves N operations of the wave, and so no more
    transfers (other loads and stores only take their places).

    The compiler makes an else of two guarded parts: a mask is all ones, the first part clears it, and the second is passed by unless it is still there.  So masks that
    are all ones or zero are known along a path, until something else is written to their registers, and a branch on one goes one way."""
    blocks = _blocks(lines)
    seen, todo, found = {("entry", 0, ())}, [("entry", 0, ())], {}
    while todo:                                            # every state in which a piece is entered: transfers in flight, known masks
        name, flying, known = todo.pop()
        masks = dict(known)
        body, ways, branch = blocks[name]
        for i, ins in enumerate(body):
            wait = re.match(r"s_waitcnt\b.*\bvmcnt\((\d+)\)", ins)
            if "_load_lds_" in ins:
                flying = min(flying + 1, MANY)
            elif wait:
                flying = min(flying, int(wait[1]))
            elif ins.startswith("s_barrier") and flying:
                found[name, i] = max(found.get((name, i), 0), flying)
            written = re.match(r"\S+\s+(?:s\[(\d+):(\d+)\]|s(\d+)\b|(vcc))", ins)
            if written:
                lo, hi, one, vcc = written.groups()
                value, test = re.match(r"s_mov_b64 s\[\d+:\d+\], (0|-1)$", ins), re.match(r"s_(and|andn2)_b64 vcc, exec, s\[(\d+):\d+\]$", ins)
                new = masks.get(int(test[2])) if test else None
                masks = {r: v for r, v in masks.items() if (r == "vcc") != bool(vcc) or (not vcc and (int(hi or one) < r or int(lo or one) > r + 1))}
                if value:
                    masks[int(lo)] = value[1] == "-1"
                if new is not None:
                    masks["vcc"] = new == (test[1] == "and")
            elif re.match(r"v_cmp|v_\w+_co_", ins):         # (vcc without being named first)
                masks.pop("vcc", None)
        if branch in ("vccz", "vccnz") and "vcc" in masks:
            ways = ways[:1] if masks["vcc"] == (branch == "vccnz") else ways[1:]
        state = tuple(sorted((r, v) for r, v in masks.items() if r != "vcc"))
        for n in ways:
            if n in blocks and (n, flying, state) not in seen:
                seen.add((n, flying, state))
                todo.append((n, flying, state))
    return found


def test_path_search_sees_a_missing_wait():
    """The search itself: a transfer on one of two paths, with and without a wait behind it."""
    in_flight = lambda code: list(_transfers_at_barriers(code).values())
    code = ["s_cbranch_scc1 .L1", "global_load_lds_dwordx4 v[0:1], off", ".L1:", "s_waitcnt lgkmcnt(0)", "s_barrier", "s_endpgm"]
    assert in_flight(code) == [1]
    assert in_flight(code[:3] + ["s_waitcnt vmcnt(0)"] + code[3:]) == []
    loop = [".L0:", "s_barrier", "global_load_lds_dwordx4 v[0:1], off", "s_cbranch_scc1 .L0", "s_endpgm"]
    assert in_flight(loop) == [MANY]


def test_path_search_sees_a_wait_that_leaves_too_many():
    """A loop that asks for the tile after the next behind its barrier, two transfers a tile, and waits for all but the next tile's, or where there is none for all: with either wait
    left out, or one that leaves more, transfers of the tile that the barrier publishes may be under way."""
    load = "global_load_lds_dwordx4 v0, s[0:1]"

    def loop(next_one, last, clear="s_mov_b64 s[8:9], 0"):
        code = [load] * 4 + [".L0:", "s_mov_b64 s[8:9], -1", "s_and_b64 vcc, exec, s[40:41]", "s_cbranch_vccz .L1", *last, clear, ".L1:", "s_andn2_b64 vcc, exec, s[8:9]", "s_cbranch_vccnz .L2", *next_one,
                             ".L2:", "s_waitcnt lgkmcnt(0)", "s_barrier", "s_cbranch_scc1 .L3", load, load, ".L3:", "s_cbranch_scc1 .L0", "s_endpgm"]
        return list(_transfers_at_barriers(code).values())

    assert loop(["s_waitcnt vmcnt(2)"], ["s_waitcnt vmcnt(0)"]) == [2]
    assert loop(["s_waitcnt vmcnt(3)"], ["s_waitcnt vmcnt(0)"]) == [3]
    assert loop([], ["s_waitcnt vmcnt(0)"]) == [MANY]
    assert loop(["s_waitcnt vmcnt(2)"], []) == [MANY]
    assert loop(["s_waitcnt vmcnt(2)"], [], "s_mov_b64 s[8:9], s[10:11]") == [MANY]            # nothing is known of the mask: both ways
    assert loop(["s_waitcnt vmcnt(2)"], [], "s_mov_b64 s[10:11], 0") == [2]                    # not cleared: the second part always


# source: kernels, by the beginning of their names, their instances, and for each barrier that leaves transfers under way on purpose how many a wave may have there.  Those of stats_kernel and
# lines_kernel are of the next chunk of query rows, at a barrier that orders LDS which no transfer fills (the slab of diagonals, the rows' reduction): any number.  Those of
# range_stats_kernel are of the next tile of keys (64 rows, 1 KB a transfer, four waves), at the barrier that publishes the tile before it: what was asked for earlier has landed.
KERNELS = {
    "ls_decode.hip": [("decode_kernelI", 4, [])],
    "ls_prefill.hip": [("prefill_bf16_kernelI", 4, [])],
    "ls_score.hip": [("range_stats_kernelILi128E", 2, [4]), ("range_stats_kernelILi64E", 2, [2]), ("stats_kernelI", 4, [MANY]), ("retain_kernelI", 2, []), (r"lines_kernelI\w+Li[04]ELb", 16, [MANY]),
                     (r"lines_kernelI\w+Li[123]ELb", 24, [])],
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
            there = list(_transfers_at_barriers(lines).values())
            assert len(there) == len(in_flight) and all(n <= most for n, most in zip(there, in_flight)), (k, there)
        seen |= set(found)
    # no other kernel of the source has transfers
    assert not [k for k, lines in kernels.items() if k not in seen and any("_load_lds_" in x for x in lines)]
