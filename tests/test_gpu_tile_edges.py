"""The tile loops of the bf16 attention at their edges, with the work in pieces and in queues: runs of contiguous tiles of every length up to a few
and around 64 and 128 (a wave keeps 64 key blocks at a time), column lists that end at either half of a packed tile, contexts that end inside
either half of a key block."""
import numpy as np
import pytest
import torch

from paper_2507_13681_amd import binding, inputs
from tests.gpu_util import Pipeline, dev_lists

pytestmark = pytest.mark.gpu

COLUMNS = [0, 1, 31, 32, 33, 64, 65, 96, 97, 129]
DIAGONALS = [0, 1, 2, 66, 130, 64 * 61 + 1, 64 * 62 + 1, 64 * 63 + 1, 64 * 64 + 1, 64 * 65 + 1, 64 * 126 + 1, 64 * 128 + 1]      # 0 .. that many - 1


@pytest.mark.parametrize("d,n,n_hat", [(128, 8448, 130), (128, 8400, 97), (128, 8425, 3), (64, 8448, 130), (64, 8470, 40)])
def test_tile_loop_edges(oracle, d, n, n_hat):
    print(f"tile loop edges d={d} n={n} n_hat={n_hat}", flush=True)
    rng = np.random.default_rng(n)
    heads = [(COLUMNS[(i + j) % len(COLUMNS)], s) for i, s in enumerate(DIAGONALS) for j in (0, 3, 7)]
    Hq = len(heads)
    v_idx, s_idx = np.zeros((1, Hq, n), np.int32), np.zeros((1, Hq, n), np.int32)
    v_cnt, s_cnt = np.zeros((1, Hq), np.int32), np.zeros((1, Hq), np.int32)
    for h, (c, s) in enumerate(heads):
        s = min(s, n)
        v_idx[0, h, :c] = np.sort(rng.choice(n - n_hat, size=c, replace=False)); v_cnt[0, h] = c
        s_idx[0, h, :s] = np.arange(s); s_cnt[0, h] = s
    q, k, v = inputs.make_plain(1, Hq, 4, n, n_hat, d, dtype="bf16", seed=n + d, q_scale=1.5)
    ref, rlse = oracle.attend(q, k, v, v_idx, v_cnt, s_idx, s_cnt, mode=0)
    pipe = Pipeline(q, k, v, 1, "bf16")
    items = Hq * ((n - (n - n_hat) // 128 * 128 + 127) // 128)
    tables = Hq * ((n + 31) // 32 * 4 + 64 + (n // 64 + 5) * 3) + items * 20 + 4096        # no room for parts: queues of whole items
    for ctx, pieces in ((pipe.ctx, True), (binding.Context(workspace=tables), False)):
        pipe.ctx = ctx
        out, lse = pipe.prefill(dev_lists(v_idx, v_cnt, s_idx, s_cnt), sentinel=True)
        assert (ctx.debug_prefill_queues(pipe.shape)[2] > 0) == pieces
        assert ctx.ls_poll_status() == 0
        o, l = out.float().cpu().numpy().reshape(ref.shape), lse.cpu().numpy().reshape(rlse.shape)
        assert not np.isnan(o).any() and not np.isnan(l).any()
        err = np.abs(o - ref)
        assert err.max() <= 2e-2 and err.mean() <= 5e-3, (err.max(), err.mean())       # as everywhere for bf16
        alive = np.isfinite(rlse)
        np.testing.assert_array_equal(np.isfinite(l), alive)
        assert np.abs(l[alive] - rlse[alive]).max() <= 2e-3


@pytest.mark.parametrize("B,Hq,Hkv,n,n_hat,d", [(8, 16, 4, 8100, 3000, 128), (8, 16, 4, 8100, 6100, 64)])
def test_either_side_of_the_line(B, Hq, Hkv, n, n_hat, d):
    """One call beyond the line between pieces and queues against calls of four of its dialogues and of the rest, which lie below."""
    print(f"either side of the line B={B} n={n} n_hat={n_hat} d={d}", flush=True)
    in_pieces = lambda b: binding.prefill_in_pieces(binding.make_shape(b, Hq, Hkv, d, n, n_hat, 1, "bf16"))
    assert not in_pieces(B) and in_pieces(4) and in_pieces(B - 4)
    rng = np.random.default_rng(n_hat)
    v_idx, s_idx = np.zeros((B, Hq, n), np.int32), np.zeros((B, Hq, n), np.int32)
    v_cnt, s_cnt = np.zeros((B, Hq), np.int32), np.zeros((B, Hq), np.int32)
    for b in range(B):
        for h in range(Hq):
            kind = (b + h) % 4
            s = np.arange(n) if kind == 0 else np.zeros(0, int) if kind == 1 else np.flatnonzero(rng.random(n) < (0.02 if kind == 2 else 0.2))
            c = np.flatnonzero(rng.random(n) < (0.1 if kind == 1 else 0.01))
            v_idx[b, h, :len(c)] = c; v_cnt[b, h] = len(c)
            s_idx[b, h, :len(s)] = s; s_cnt[b, h] = len(s)
    q, k, v = inputs.make_plain(B, Hq, Hkv, n, n_hat, d, dtype="bf16", seed=n_hat, q_scale=1.5)
    whole = Pipeline(q, k, v, 1, "bf16")
    out, lse = whole.prefill(dev_lists(v_idx, v_cnt, s_idx, s_cnt), sentinel=True)
    tol = 4 * 2.0 ** -9 * float(np.abs(v).max())           # each side rounds every probability (2^-9 relative) and the result
    for b in (slice(0, 4), slice(4, B)):
        part, plse = Pipeline(q[b], k[b], v[b], 1, "bf16").prefill(dev_lists(v_idx[b], v_cnt[b], s_idx[b], s_cnt[b]), sentinel=True)
        assert not torch.isnan(out[b]).any() and not torch.isnan(part).any()
        assert (out[b].float() - part.float()).abs().max().item() <= tol
        some = torch.isfinite(plse)
        assert torch.equal(torch.isfinite(lse[b]), some)
        assert (lse[b][some] - plse[some]).abs().max().item() <= 1e-4


@pytest.mark.parametrize("Hq,Hkv,n,n_hat,d", [(1, 1, 64, 64, 64), (4, 1, 1024, 256, 64), (2, 1, 1000, 5, 128), (8, 8, 777, 300, 64), (16, 4, 2050, 131, 64)])
def test_fp32_single_tiles(oracle, Hq, Hkv, n, n_hat, d):
    """fp32 pieces of one tile: items of none, one and many tiles of either kind, cut after any of them."""
    print(f"fp32 single tiles Hq={Hq} n={n} n_hat={n_hat} d={d}", flush=True)
    rng = np.random.default_rng(n)
    v_idx, s_idx = np.zeros((1, Hq, n), np.int32), np.zeros((1, Hq, n), np.int32)
    v_cnt, s_cnt = np.zeros((1, Hq), np.int32), np.zeros((1, Hq), np.int32)
    for h in range(Hq):
        kind = (h + n) % 4                                 # some of both, columns only, one diagonal, all
        c = np.flatnonzero(rng.random(n) < (0.3 if kind < 2 else 0.0))
        s = np.arange(n) if kind == 3 else np.zeros(0, int) if kind == 1 else np.array([n // 2]) if kind == 2 else np.flatnonzero(rng.random(n) < 0.02)
        v_idx[0, h, :len(c)] = c; v_cnt[0, h] = len(c)
        s_idx[0, h, :len(s)] = s; s_cnt[0, h] = len(s)
    q, k, v = inputs.make_plain(1, Hq, Hkv, n, n_hat, d, dtype="f32", seed=n, q_scale=1.5)
    ref, rlse = oracle.attend(q, k, v, v_idx, v_cnt, s_idx, s_cnt, mode=0)
    pipe = Pipeline(q, k, v, 1, "f32")
    out, lse = pipe.prefill(dev_lists(v_idx, v_cnt, s_idx, s_cnt), sentinel=True)
    assert pipe.ctx.ls_poll_status() == 0
    o, l = out.cpu().numpy().reshape(ref.shape), lse.cpu().numpy().reshape(rlse.shape)
    assert not np.isnan(o).any() and not np.isnan(l).any()
    # sums of up to n products of fp32, exp2 of the hardware (2^-22): a few of those, times the largest value
    assert np.abs(o - ref).max() <= 64 * 2.0 ** -23 * np.abs(v).max()
    alive = np.isfinite(rlse)
    np.testing.assert_array_equal(np.isfinite(l), alive)
    assert np.abs(l[alive] - rlse[alive]).max() <= 1e-4


@pytest.mark.parametrize("Hq,Hkv,n,n_hat,d", [(64, 8, 2048, 2048, 128), (64, 64, 2500, 2101, 128), (64, 16, 3072, 3072, 64), (64, 8, 5003, 3050, 64)])
def test_parts_joined_by_the_last(Hq, Hkv, n, n_hat, d):
    """At least two items to a workgroup, heads of very unlike work (items of one part and of many, row blocks with few rows): against a call per
    16 heads, whose parts are put together by a kernel of its own, and against itself, whoever came last."""
    print(f"parts joined Hq={Hq} n={n} n_hat={n_hat} d={d}", flush=True)
    items = lambda heads: heads * ((n - (n - n_hat) // 128 * 128 + 127) // 128)
    grid = 512 if d == 128 else 768
    assert items(Hq) >= 2 * grid > 2 * items(16)
    rng = np.random.default_rng(n)
    v_idx, s_idx = np.zeros((1, Hq, n), np.int32), np.zeros((1, Hq, n), np.int32)
    v_cnt, s_cnt = np.zeros((1, Hq), np.int32), np.zeros((1, Hq), np.int32)
    for h in range(Hq):
        c = np.flatnonzero(rng.random(n) < (0.1, 0.0, 0.01, 0.5)[h % 4])
        s = np.arange(n) if h % 16 == 5 else np.zeros(0, int) if h % 4 == 3 else np.flatnonzero(rng.random(n) < 0.01)
        v_idx[0, h, :len(c)] = c; v_cnt[0, h] = len(c)
        s_idx[0, h, :len(s)] = s; s_cnt[0, h] = len(s)
    q, k, v = inputs.make_plain(1, Hq, Hkv, n, n_hat, d, dtype="bf16", seed=n, q_scale=1.5)
    whole = Pipeline(q, k, v, 1, "bf16")
    out, lse = whole.prefill(dev_lists(v_idx, v_cnt, s_idx, s_cnt), sentinel=True)
    assert whole.ctx.debug_prefill_queues(whole.shape)[2] > 0
    for _ in range(4):
        again, lagain = whole.prefill(dev_lists(v_idx, v_cnt, s_idx, s_cnt), sentinel=True)
        assert torch.equal(again, out) and torch.equal(lagain, lse)
    assert whole.ctx.ls_poll_status() == 0
    tol = 4 * 2.0 ** -9 * float(np.abs(v).max())           # each side rounds every probability (2^-9 relative) and the result
    for h0 in range(0, Hq, 16):
        h, g = slice(h0, h0 + 16), slice(h0 * Hkv // Hq, max(h0 * Hkv // Hq + 1, (h0 + 16) * Hkv // Hq))
        part, plse = Pipeline(q[:, h], k[:, g], v[:, g], 1, "bf16").prefill(dev_lists(v_idx[:, h], v_cnt[:, h], s_idx[:, h], s_cnt[:, h]), sentinel=True)
        assert not torch.isnan(out[:, h]).any() and not torch.isnan(part).any()
        assert (out[:, h].float() - part.float()).abs().max().item() <= tol
        some = torch.isfinite(plse)
        assert torch.equal(torch.isfinite(lse[:, h]), some)
        assert (lse[:, h][some] - plse[some]).abs().max().item() <= 1e-4
