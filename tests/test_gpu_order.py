"""Desc_Sort inside ls_select, where a list is put in order in several ranges of weights: the lengths at which their number
changes, and weights that miss the ranges' usual course or fill single bins.  The oracle's selection exactly; `accounted` is a running sum
over the picks, so it shows their order."""
import numpy as np
import pytest
import torch

from paper_2507_13681_amd import binding


def _sampled(n):
    """The lines from which the ranges' bounds are taken."""
    i = np.arange(2048)
    return i * n // 2048 + ((i * 0x9E3779B1 % 2 ** 32 >> 16) * (n // 2048) >> 16)


KINDS = {
    # distinct weights over ten binades
    "spread": lambda rng, n: np.exp2(rng.uniform(-10, 0, n)),
    # two thirds of one weight, more than a workgroup holds; the others few-valued
    "equal": lambda rng, n: np.where(rng.random(n) < 0.67, 0.25, rng.integers(1, 60, n) / 64.0),
    # all but a handful within 2^12 numbers: the bins of the outliers' ranges hold hundreds of lines each
    "crowd": lambda rng, n: np.where(rng.random(n) < 10 / n, np.exp2(rng.uniform(-60, 20, n)), 0.5 + rng.integers(0, 4096, n) * 2.0 ** -24),
    # few weights, each of hundreds of lines and more; two fifths of the lines at zero, in runs
    "few": lambda rng, n: rng.integers(1, 60, n) / 64.0,
    "zeros": lambda rng, n: np.where(np.arange(n) // 997 % 5 < 2, 0.0, np.exp2(rng.uniform(-20, 0, n))),
    # clusters inside clusters: each eighth of the lines lies within a 2^-6 of the span that is left
    "nested": lambda rng, n: 0.5 + np.ldexp(rng.integers(1, 1 << 6, n).astype(float), -np.minimum(6 * (1 + rng.geometric(0.4, n) % 4), 24)),
    # one weight; two; one beside a single other
    "one": lambda rng, n: np.full(n, 0.125),
    "two": lambda rng, n: np.where(rng.random(n) < 0.5, 0.125, 0.25),
    "but_one": lambda rng, n: np.where(np.arange(n) == n // 2, 3.0, 0.125),
    # every sampled line far above the others: the ranges found for them hold nearly nothing or nearly everything
    "unseen": lambda rng, n: np.where(np.isin(np.arange(n), _sampled(n)), rng.uniform(1, 2, n), rng.uniform(0.01, 0.02, n)),
}


@pytest.mark.gpu
@pytest.mark.parametrize("n,kind", [(4096, "crowd"), (4096, "spread"), (4097, "spread"), (4097, "crowd"), (8193, "equal"), (30011, "spread"),
                                    (30011, "equal"), (30011, "crowd"), (65536, "spread"), (65537, "unseen"), (65537, "spread"), (20000, "unseen"),
                                    (2049, "spread"), (16383, "spread"), (16384, "equal"),
                                    (33, "one"), (700, "crowd"), (1024, "few"), (1000, "two"), (1024, "nested"), (4096, "few"), (4096, "zeros"), (4095, "but_one"),
                                    (4096, "nested"), (8192, "zeros"), (8192, "few"), (8191, "two"), (10240, "nested"), (30011, "few"), (30011, "zeros"),
                                    (30011, "two"), (30011, "one"), (30011, "but_one"), (30011, "nested"), (131071, "few"), (131071, "equal"),
                                    (65537, "zeros"), (65537, "crowd"),
                                    (80862, "few"), (131072, "two"), (262144, "few"), (262143, "crowd"), (200001, "nested")])
def test_lists_in_ranges(oracle, n, kind, H=3):
    from tests.gpu_util import host
    from tests.test_gpu_configs import check_selection_exact
    print(f"lists in ranges n={n} {kind}", flush=True)
    rng = np.random.default_rng(n)
    v, s = (np.stack([KINDS[kind](rng, n) for _ in range(H)])[None] for _ in range(2))
    v = v.copy(); s = s.copy()
    s[:, 1] *= 1e-3; v[:, 0] *= 1e-3                                  # one head of columns, one of diagonals, one of both
    sc = dict(vert=v, slash=s, vmax=v * 1e-7, smax=s * 1e-7, total=np.maximum(v.sum(-1), s.sum(-1)))
    sc = {k: np.ascontiguousarray(x, dtype=np.float32) for k, x in sc.items()}
    for alpha in (0.3, 0.97):
        ref = oracle.select(sc, max(1, n // 3), alpha)
        shape = binding.make_shape(1, H, 1, 64, n, max(1, n // 3), 1, "f32", 0.0)
        ctx = binding.Context(shape)
        out = binding.alloc_select(shape, accounted=True)
        dev = {k: torch.from_numpy(x).cuda() for k, x in sc.items()}
        ctx.ls_select(shape, alpha, dev["vert"], dev["slash"], dev["vmax"], dev["smax"], dev["total"], out["v_idx"], out["v_cnt"],
                      out["s_idx"], out["s_cnt"], out["accounted"])
        assert ctx.ls_poll_status() == 0
        gpu = host(out)
        check_selection_exact(gpu, ref)
        np.testing.assert_array_equal(gpu["accounted"], ref["accounted"])


# so many heads that there is one range a list, beyond the length that always is
@pytest.mark.gpu
@pytest.mark.parametrize("n,kind", [(4097, "spread"), (5003, "few"), (6000, "zeros"), (8192, "crowd"), (8192, "equal")])
def test_long_lists_of_many_heads(oracle, n, kind):
    test_lists_in_ranges(oracle, n, kind, H=130)


# the longest lists in one range and the shortest in several: any number of heads, three ranges a list, two
@pytest.mark.gpu
@pytest.mark.parametrize("n,kind,H", [(5120, "spread", 3), (5120, "crowd", 5), (5121, "few", 3), (6144, "zeros", 42), (6145, "zeros", 42), (8192, "nested", 60), (8191, "spread", 64), (8193, "spread", 64)])
def test_one_range_or_several(oracle, n, kind, H):
    test_lists_in_ranges(oracle, n, kind, H=H)


# lines without weight, up to as many as are still ranked against each other at the end of a list in one range, and more; beside others of the last bin
@pytest.mark.gpu
@pytest.mark.parametrize("n,none", [(1024, 33), (2000, 127), (4096, 128), (5003, 129), (5120, 128), (5121, 128)])
def test_lines_without_weight(oracle, monkeypatch, n, none):
    def weights(rng, n):
        w = np.exp2(rng.uniform(-20, 0, n))
        w[rng.choice(n, none, replace=False)] = 0
        w[rng.choice(n, 3, replace=False)] = 2.0 ** -30                    # of the zeros' bin, but not zero
        return w
    monkeypatch.setitem(KINDS, "no weight", weights)
    test_lists_in_ranges(oracle, n, "no weight", H=4)
