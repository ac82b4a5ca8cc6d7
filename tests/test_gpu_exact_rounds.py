"""walk_exact_kernel at the edges of its rounds, exactly as the oracle takes the lines: windows that are not whole quarters of 16 rows and longer than 64, lists
shorter than a first round, blocks of the sorted lists that are loaded again, scored rows at repeated positions, and walks that go on where gains are rounding errors of either sign."""
import numpy as np
import pytest
import torch

from paper_2507_13681_amd import binding, inputs

pytestmark = pytest.mark.gpu

from tests.gpu_util import Pipeline, dev_scores, host  # noqa: E402
from tests.test_gpu_configs import check_selection_exact  # noqa: E402


def _check(oracle, cfg, alpha, pos=None):
    q, k, v, _ = inputs.make_inputs(cfg)
    rows = slice(cfg.n_hat - cfg.w, cfg.n_hat) if pos is None else pos - (cfg.n - cfg.n_hat)
    qw = q[:, :, rows]
    kw = {} if pos is None else dict(q_pos=pos)
    sc, a = oracle.score(qw, k, **kw), oracle.window(qw, k, **kw)
    ref = oracle.select_exact(a, sc, cfg.n_hat, alpha, **kw)
    print(f"n {cfg.n} w {cfg.w} alpha {alpha}: oracle counts v {ref['v_cnt'].ravel().tolist()} s {ref['s_cnt'].ravel().tolist()}", flush=True)
    pipe = Pipeline(q, k, v, cfg.w, cfg.dtype)
    out = binding.alloc_select(pipe.shape, accounted=True)
    qp = None if pos is None else torch.from_numpy(np.asarray(pos, np.int64)).cuda()
    dev = dev_scores(sc)
    pipe.ctx.ls_select_exact(pipe.shape, alpha, torch.from_numpy(a).cuda(), dev["vert"], dev["slash"], dev["total"],
                             out["v_idx"], out["v_cnt"], out["s_idx"], out["s_cnt"], out["accounted"], qp)
    assert pipe.ctx.ls_poll_status() == 0
    got = host(out)
    check_selection_exact(got, ref)
    np.testing.assert_array_equal(got["accounted"], ref["accounted"])
    return ref


def _cfg(n, w, n_hat=None, **kw):
    return inputs.scaled(inputs.CONFIGS["llama8b_8k"], n=n, w=w, n_hat=n_hat or max(w, n // 2), Hq=4, Hkv=2, heavy_lo=4, heavy_hi=max(5, min(48, n // 40)), span=min(64, n // 4), **kw)


@pytest.mark.parametrize("n,w,alpha", [(40, 17, 0.9), (63, 32, 0.95), (200, 33, 0.95), (1100, 65, 0.98), (2500, 127, 0.95), (3000, 256, 0.9), (9000, 64, 0.99), (4097, 100, 0.98)])
def test_rounds_of_a_window(oracle, n, w, alpha):
    _check(oracle, _cfg(n, w), alpha)


@pytest.mark.parametrize("n,w", [(900, 20), (2600, 130)])
def test_rounds_of_repeated_positions(oracle, n, w):
    cfg = _cfg(n, w)
    pos = np.sort(np.random.default_rng(n).integers(n - cfg.n_hat, n, w))
    pos[w // 2] = pos[w // 2 + 1]
    assert len(np.unique(pos)) < w
    _check(oracle, cfg, 0.95, pos)


@pytest.mark.parametrize("n,w,alpha", [(1500, 32, 0.9999), (6000, 64, 0.9999)])
def test_rounds_of_nearly_covered_lines(oracle, n, w, alpha):
    """Most of the lines taken last add nothing but rounding errors, of either sign."""
    ref = _check(oracle, _cfg(n, w), alpha)
    assert (ref["v_cnt"] + ref["s_cnt"]).max() > 300
