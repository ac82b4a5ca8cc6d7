"""The greedy walk over lists whose picks come in runs of chosen lengths: single picks back and forth, runs that just fill or just miss
the entries a wave looks at, and changes from one kind to the other.  Every line has the same length, so that the weights
alone decide.  Against the oracle exactly."""
import numpy as np
import pytest
import torch

from paper_2507_13681_amd import binding

SHORT = [1] * 40
RUNS = SHORT + [255, 256, 257] + [1, 2, 3, 1] + [127, 128, 129, 1] + SHORT + [1023, 1, 1024, 1, 1025, 64, 65, 63] + [3] * 30 + [511, 512, 513, 256, 256, 2]


def _weights(n, first):
    """Two lists of n lines whose merged descending order takes RUNS lines from one and the other in turn."""
    take = np.concatenate([np.full(r, (i + first) % 2) for i, r in enumerate(RUNS * (2 * n // sum(RUNS) + 1))])
    rng = np.random.default_rng(n + first)
    out = []
    for which in (0, 1):
        at = np.flatnonzero(take == which)[:n]
        w = np.concatenate([1.0 - 0.9 * at / len(take), np.linspace(0.01, 0.001, n - len(at))])
        out.append(rng.permutation(w).astype(np.float32))
    return out


@pytest.mark.gpu
@pytest.mark.parametrize("n", [1500, 2049, 8192, 16383, 16384, 30011])
def test_walk_in_runs(oracle, n):
    from tests.gpu_util import host
    from tests.test_gpu_configs import check_selection_exact
    print(f"walk in runs n={n}", flush=True)
    v, s = (np.stack(x)[None] for x in zip(_weights(n, 0), _weights(n, 1)))
    sc = dict(vert=v, slash=s, vmax=v * np.float32(1e-10), smax=s * np.float32(1e-10), total=v.sum(-1) + s.sum(-1))
    dev = {k: torch.from_numpy(np.ascontiguousarray(x)).cuda() for k, x in sc.items()}
    for alpha, accounted in ((0.4, True), (0.97, True), (0.97, False)):
        ref = oracle.select(sc, 1, alpha)
        shape = binding.make_shape(1, 2, 1, 64, n, 1, 1, "f32", 0.0)
        ctx = binding.Context(shape)
        out = binding.alloc_select(shape, accounted=accounted)
        ctx.ls_select(shape, alpha, dev["vert"], dev["slash"], dev["vmax"], dev["smax"], dev["total"], out["v_idx"], out["v_cnt"],
                      out["s_idx"], out["s_cnt"], out["accounted"])
        assert ctx.ls_poll_status() == 0
        gpu = host({k: x for k, x in out.items() if x is not None})
        check_selection_exact(gpu, ref)
        if accounted:
            np.testing.assert_array_equal(gpu["accounted"], ref["accounted"])
