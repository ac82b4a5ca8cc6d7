"""ls_select of long lists whose largest entries are negative or no number in a part of the list that nobody needs in order: no run of picks is taken
unseen there, whatever the workspace held before.  The oracle's selection exactly."""
import numpy as np
import pytest
import torch

from paper_2507_13681_amd import binding

pytestmark = pytest.mark.gpu

from tests.gpu_util import dev_scores, host  # noqa: E402
from tests.test_gpu_configs import check_selection_exact  # noqa: E402

KINDS = ["clean", "falls", "late", "nan", "falls in columns"]


def _head(kind, n, rng):
    """slash, vert, smax, vmax, total of a head; alpha is 1.  Its heaviest lines lie in the last half of the list, and half of them reach the target
    where overlaps do not fall; the first of them rules the columns out."""
    half = n // 2
    slash = np.full(n, 1e-4, np.float32)
    slash[half:] = 1 + 0.016 * rng.permutation(n - half) / (n - half)
    slash[half] = 2
    smax = np.zeros(n, np.float32)
    smax[half] = 1
    if kind.startswith("falls"):
        smax[half + 1:] = -0.01
    elif kind == "late":
        # only in the last part of the list, a few thousand picks from the first
        last = n - n // 32
        slash[last:] = np.float32(1.012) + (slash[last:] - 1) / 64
        smax[last:] = np.float32(-8.0 / (n // 32))
    elif kind == "nan":
        at = n - n // 5
        slash[at], smax[at] = 1.012, np.nan
    vert, vmax = np.zeros(n, np.float32), np.zeros(n, np.float32)
    vert[0] = 0.5
    total = np.float32(0.488 * half)
    return (vert, slash, vmax, smax, total) if kind.endswith("columns") else (slash, vert, smax, vmax, total)


@pytest.mark.parametrize("n", [9000, 16384, 32768, 65536])
def test_maxima_of_lines_that_are_not_put_in_order(oracle, n, H=32):
    print(f"late maxima n={n}", flush=True)
    rng = np.random.default_rng(n)
    clean = [_head("clean", n, rng) for _ in range(H)]
    heads = [_head(KINDS[h % len(KINDS)], n, rng) for h in range(H)]
    pack = lambda hs: {k: np.ascontiguousarray(np.stack([np.asarray(h[i]) for h in hs])[None], dtype=np.float32)
                       for i, k in enumerate(("slash", "vert", "smax", "vmax", "total"))}
    first, sc = pack(clean), pack(heads)
    ref_first, ref = oracle.select(first, 1, 1.0), oracle.select(sc, 1, 1.0)
    # runs that are taken unseen would come to other counts
    for h in range(1, 5):
        assert (ref["v_cnt"][0, h], ref["s_cnt"][0, h]) != (ref_first["v_cnt"][0, 0], ref_first["s_cnt"][0, 0]), KINDS[h]
    shape = binding.make_shape(1, H, 1, 64, n, 1, 1, "f32", 0.0)
    dev, dev_first = dev_scores(sc), dev_scores(first)
    ctx = binding.Context(shape)

    def select(s):
        out = binding.alloc_select(shape, accounted=False)
        ctx.ls_select(shape, 1.0, s["vert"], s["slash"], s["vmax"], s["smax"], s["total"], out["v_idx"], out["v_cnt"], out["s_idx"], out["s_cnt"])
        assert ctx.ls_poll_status() == 0
        return host({k: x for k, x in out.items() if x is not None})

    for fill in (0, 1, -1, None):
        if fill is None:                                   # ... and what a call on clean lists leaves there
            check_selection_exact(select(dev_first), ref_first)
        else:
            ctx.debug_fill_workspace(fill)
        check_selection_exact(select(dev), ref)
    ranges, left, again = ctx.debug_select_order(shape)
    assert 0 < left[0, 0] < ranges and again[0] == 0       # "clean": the tests' premise
