"""Edges of the kernels' tiles, splits and dispatch rules, against the oracle."""
import numpy as np
import pytest
import torch

from paper_2507_13681_amd import binding, inputs
from tests.test_gpu_decode import _case, _check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,Hq,Hkv,cap,T,d,ragged", [
    (1, 2, 2, 31, 1, 128, False),      # a partial tile and a one-row tail tile
    (1, 16, 1, 32, 32, 64, False),     # whole tiles only; a full block of 16 heads
    (1, 17, 1, 33, 0, 128, True),      # a second block of heads with one head
    (2, 12, 2, 545, 33, 64, True),     # 20 tiles: two or three a wave and several splits; the tail's tiles move with the count
    (1, 32, 8, 575, 1, 128, True),     # 19 tiles: beyond one workgroup's share, splits of unequal length
    (1, 24, 1, 9000, 40, 128, True),   # many splits, two blocks of heads
])
def test_decode_tiles_and_splits(oracle, B, Hq, Hkv, cap, T, d, ragged):
    print(f"decode edge B={B} Hq={Hq} Hkv={Hkv} cap={cap} T={T} d={d}", flush=True)
    _check(oracle, _case(B, Hq, Hkv, cap, T, d, seed=3 * cap + T, ragged=ragged))


@pytest.mark.parametrize("dtype,d,n,n_hat", [
    ("bf16", 128, 9001, 67),       # two row blocks, 141 key blocks: items in many parts
    ("bf16", 64, 6400, 128),       # one whole row block
    ("f32", 64, 3000, 130),
    ("f32", 128, 2049, 1),         # one row
])
def test_prefill_parts_of_long_items(oracle, dtype, d, n, n_hat):
    """Few row blocks over a long context: items are cut into parts and put together again; in a workspace without room
    for parts they are not, with the same result."""
    from tests.gpu_util import Pipeline, dev_lists
    from tests.test_gpu_random_shapes import _selection
    print(f"parts {dtype} d={d} n={n} n_hat={n_hat}", flush=True)
    rng = np.random.default_rng(n)
    B, Hq, Hkv = 1, 4, 2
    q, k, v = inputs.make_plain(B, Hq, Hkv, n, n_hat, d, dtype=dtype, seed=n, q_scale=1.5)
    v_idx, v_cnt, s_idx, s_cnt = _selection(rng, B, Hq, n)
    s_idx[0, 0] = np.arange(n); s_cnt[0, 0] = n                       # one dense head
    rows = np.unique(rng.integers(0, Hq * n_hat, 60))
    ref, ref_lse = oracle.attend(q, k, v, v_idx, v_cnt, s_idx, s_cnt, rows=rows, mode=1)
    pipe = Pipeline(q, k, v, 1, dtype)
    small = binding.Context(workspace=2 << 20)
    tol = (2e-2, 5e-3, 2e-3) if dtype == "bf16" else (1e-4, 1e-5, 1e-4)
    for ctx in (pipe.ctx, small):
        pipe.ctx = ctx
        out, lse = pipe.prefill(dev_lists(v_idx, v_cnt, s_idx, s_cnt), sentinel=True)
        torch.cuda.synchronize()
        assert ctx.ls_poll_status() == 0
        assert not torch.isnan(out.float()).any() and not torch.isnan(lse).any()
        o = out.float().cpu().numpy().reshape(-1, d)[rows]
        l = lse.cpu().numpy().reshape(-1)[rows]
        err = np.abs(o - ref)
        assert err.max() <= tol[0] and err.mean() <= tol[1], (err.max(), err.mean())
        alive = np.isfinite(ref_lse)
        np.testing.assert_array_equal(np.isfinite(l), alive)
        assert np.abs(l[alive] - ref_lse[alive]).max(initial=0) <= tol[2]
