"""ls_select where the lists are put in order only as far as a walk can be expected to come: walks that go further, walks that end
on the last line in order, maxima that do not let long runs through, and contexts with room for the first lines' weights only.  The
oracle's selection exactly."""
import numpy as np
import pytest
import torch

from paper_2507_13681_amd import binding


def _head(kind, n, rng):
    """slash, vert, smax, vmax, total of a head; alpha is 1."""
    slash = (1.0 + rng.random(n) * 2.0 ** -6).astype(np.float32)
    vert, smax, vmax = np.zeros(n, np.float32), np.full(n, 1e-6, np.float32), np.zeros(n, np.float32)
    vert[: n // 7] = 1e-3
    if kind == "further":
        # a column is taken first, and every diagonal then adds half of its weight: twice as many are needed as weigh enough together
        vert[7], vmax[7], total = 5.0, 0.5, 0.44 * n
    elif kind == "all":
        # the same, and all diagonals do not reach the target: everything is selected
        vert[7], vmax[7], total = 5.0, 0.5, 0.7 * n
    elif kind == "columns":
        vert, slash = slash.copy(), np.full(n, 1e-4, np.float32)
        vmax, smax, total = np.full(n, 1e-6, np.float32), np.zeros(n, np.float32), 0.3 * n
    elif kind == "heavy":
        # a few lines weigh nearly everything
        slash = (slash * 1e-4).astype(np.float32)
        slash[rng.choice(n, 40, replace=False)] += 1.0
        total = 39.0
    elif kind == "negative":
        # overlaps that fall: no run is taken unseen
        smax = np.where(rng.random(n) < 0.5, -1e-3, 1e-3).astype(np.float32)
        vert[: n // 7], total = 0.9, 0.4 * n
    elif kind == "signs":
        # more lines below zero than above
        slash = (rng.random(n).astype(np.float32) - np.float32(0.7)) * 2
        vert = slash[::-1].copy()
        total = float(slash[slash > 0].sum()) * 0.9
    else:
        total = 0.5 * n                                    # "plain"
    return slash, vert, smax, vmax, np.float32(total)


HEADS = ["further", "plain", "all", "columns", "heavy", "negative", "signs"]


@pytest.mark.gpu
@pytest.mark.parametrize("n,room", [(8192, "usual"), (8193, "usual"), (12347, "usual"), (16384, "usual"), (40000, "usual"), (65537, "usual"), (131072, "usual"),
                                    (9001, "first lines"), (4097, "first lines"), (900, "first lines"), (20000, "one short")])
def test_walks_and_the_lines_in_order(n, room):
    from oracle import ref as oracle
    from tests.gpu_util import host
    from tests.test_gpu_configs import check_selection_exact
    print(f"lines in order n={n} room={room}", flush=True)
    rng = np.random.default_rng(n)
    heads = [_head(k, n, rng) for k in HEADS]
    H = len(heads)
    sc = {k: np.ascontiguousarray(np.stack([np.asarray(h[i]) for h in heads])[None], dtype=np.float32) for i, k in enumerate(("slash", "vert", "smax", "vmax", "total"))}
    n_hat = max(1, n // 3)
    ref = oracle.select(sc, n_hat, 1.0)
    further = int(ref["s_cnt"][0, 0])                      # the first head's walk does go beyond the lines that weigh enough
    assert np.sort(sc["slash"][0, 0])[::-1][:further * 3 // 4].sum(dtype=np.float64) > 1.01 * sc["total"][0, 0]
    shape = binding.make_shape(1, H, 1, 64, n, n_hat, 1, "f32", 0.0)
    up = lambda x: (x + 255) // 256 * 256
    first = up(8 * H * n) + 2 * up(8 * H * 1024)           # the lists' order and the first lines' weights and maxima: the least that ls_select takes
    size = {"usual": None, "first lines": first, "one short": 3 * up(8 * H * n) - 256}[room]
    ctx = binding.Context(shape) if size is None else binding.Context(workspace=size)
    dev = {k: torch.from_numpy(x).cuda() for k, x in sc.items()}
    for accounted in (False, True, False):
        out = binding.alloc_select(shape, accounted=accounted)
        ctx.ls_select(shape, 1.0, dev["vert"], dev["slash"], dev["vmax"], dev["smax"], dev["total"], out["v_idx"], out["v_cnt"],
                      out["s_idx"], out["s_cnt"], out["accounted"])
        assert ctx.ls_poll_status() == 0
        gpu = host({k: x for k, x in out.items() if x is not None})
        if accounted:
            np.testing.assert_array_equal(gpu["accounted"], ref["accounted"])
        check_selection_exact(gpu, ref)
