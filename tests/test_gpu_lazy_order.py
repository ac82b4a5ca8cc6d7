"""ls_select where the lists are put in order only as far as a walk can be expected to come: walks that go further, walks that end
on the last line in order, maxima that do not let long runs through, and contexts with room for the first lines' weights only.  The
oracle's selection exactly, and that ranges were left out and heads walked again where a test is for that."""
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
    ranges, left, again = ctx.debug_select_order(shape)
    if n < 8193 or room != "usual":
        assert ranges == 0                                 # everything was put in order
    else:
        assert again[0] > 0 and left[0, 0] == 0           # "further"
        assert again[1] == 0 and 0 < left[0, 1] < ranges   # "plain"


@pytest.mark.gpu
@pytest.mark.parametrize("H,n,further", [(8, 12347, 8), (32, 20000, 3), (96, 9000, 40), (128, 8200, 128), (129, 8200, 1), (200, 8193, 200), (300, 8300, 257), (1030, 8200, 7)])
def test_heads_walked_again(oracle, H, n, further):
    """Few heads and many, of which some or all need lines that were left out: workgroups that share a head, one a head, more heads than CUs and than threads."""
    from tests.gpu_util import dev_scores, host
    from tests.test_gpu_configs import check_selection_exact
    print(f"heads walked again H={H} n={n}", flush=True)
    rng = np.random.default_rng(H)
    kinds = np.full(H, "plain", dtype=object)
    kinds[rng.choice(H, further, replace=False)] = "further"
    kinds[rng.choice(np.flatnonzero(kinds == "further"), further // 3, replace=False)] = "all"
    two = {k: [_head(k, n, rng) for _ in range(2)] for k in ("plain", "further", "all")}
    heads = [two[k][h % 2] for h, k in enumerate(kinds)]
    pack = lambda hs: {k: np.ascontiguousarray(np.stack([np.asarray(h[i]) for h in hs])[None], dtype=np.float32) for i, k in enumerate(("slash", "vert", "smax", "vmax", "total"))}
    n_hat = n // 3
    some = oracle.select(pack(two["plain"] + two["further"] + two["all"]), n_hat, 1.0)
    which = [2 * ["plain", "further", "all"].index(k) + h % 2 for h, k in enumerate(kinds)]
    ref = {k: np.ascontiguousarray(x[:, which]) for k, x in some.items()}
    shape = binding.make_shape(1, H, 1, 64, n, n_hat, 1, "f32", 0.0)
    ctx, dev = binding.Context(shape), dev_scores(pack(heads))
    for _ in range(2):                                     # the second call finds what the first has counted
        out = binding.alloc_select(shape, accounted=False)
        ctx.ls_select(shape, 1.0, dev["vert"], dev["slash"], dev["vmax"], dev["smax"], dev["total"], out["v_idx"], out["v_cnt"], out["s_idx"], out["s_cnt"])
        assert ctx.ls_poll_status() == 0
        check_selection_exact(host({k: x for k, x in out.items() if x is not None}), ref)
    ranges, left, again = ctx.debug_select_order(shape)
    assert ranges > 0
    np.testing.assert_array_equal(again > 0, kinds != "plain")
    assert (left[0, kinds == "plain"] > 0).all() and (left[:, kinds != "plain"] == 0).all()
