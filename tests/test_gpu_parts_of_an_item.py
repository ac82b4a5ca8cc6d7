"""Short turns of few heads, whose row blocks are cut into many parts: up to 48 of a block, in fp32 of one tile each, with cuts that fall into one tile.
Against the oracle, and with a workspace that has room for a dozen parts of a block."""
import numpy as np
import pytest
import torch

from paper_2507_13681_amd import binding, inputs
from tests.gpu_util import Pipeline, dev_lists
from tests.test_gpu_work_split import _lists

pytestmark = pytest.mark.gpu


# few row blocks: 48 workgroups each; fp32 up to 256 (5 blocks: 240, 6: 256), from 22 blocks on 12 each; bf16 up to what 15 MB of parts hold (d = 128: 4 blocks 192, 5 to 18 about 220), then up to every place (19: 512)
@pytest.mark.parametrize("Hq,Hkv,n,n_hat,d,dtype", [
    (1, 1, 16384, 16, 64, "f32"), (4, 1, 1024, 256, 64, "f32"), (8, 2, 300, 40, 64, "f32"), (5, 1, 4097, 60, 128, "f32"), (6, 2, 6001, 3, 64, "f32"),
    (11, 1, 2001, 129, 64, "f32"), (3, 1, 64, 64, 64, "f32"), (2, 1, 1, 1, 128, "f32"),
    (1, 1, 16384, 64, 64, "bf16"), (2, 1, 30011, 20, 128, "bf16"), (10, 2, 9001, 33, 128, "bf16"), (11, 1, 9000, 1, 128, "bf16"), (18, 2, 5001, 70, 128, "bf16"), (19, 1, 7000, 9, 128, "bf16"), (15, 5, 6000, 100, 64, "bf16")])
def test_many_parts_of_an_item(oracle, Hq, Hkv, n, n_hat, d, dtype):
    print(f"many parts Hq={Hq} n={n} n_hat={n_hat} d={d} {dtype}", flush=True)
    q, k, v = inputs.make_plain(1, Hq, Hkv, n, n_hat, d, dtype=dtype, seed=n, q_scale=1.5)
    lists = _lists(np.random.default_rng(n), 1, Hq, n)
    ref, rlse = oracle.attend(q, k, v, *lists, mode=0)
    pipe = Pipeline(q, k, v, 1, dtype)
    items = Hq * ((n - (n - n_hat) // 128 * 128 + 127) // 128)
    tables = Hq * ((n + 31) // 32 * 4 + 64 + (n // 64 + 5) * 3) + items * 20 + 16384
    # bf16 as everywhere; fp32: sums of at most n terms in another order and the hardware's exp2, as between queues and pieces
    tol = 2e-2 if dtype == "bf16" else 1e-5 * float(np.abs(v).max())
    for ctx in (pipe.ctx, binding.Context(workspace=tables + 13 * items * (128 * d * 4 + 1024 + 24))):
        pipe.ctx = ctx
        for _ in range(2):
            out, lse = pipe.prefill(dev_lists(*lists), sentinel=True)
            assert ctx.ls_poll_status() == 0
            o, l = out.float().cpu().numpy().reshape(ref.shape), lse.cpu().numpy().reshape(rlse.shape)
            assert not np.isnan(o).any() and not np.isnan(l).any()
            assert np.abs(o - ref).max() <= tol, np.abs(o - ref).max()
            alive = np.isfinite(rlse)
            np.testing.assert_array_equal(np.isfinite(l), alive)
            assert np.abs(l[alive] - rlse[alive]).max(initial=0.0) <= (2e-3 if dtype == "bf16" else 1e-4)
