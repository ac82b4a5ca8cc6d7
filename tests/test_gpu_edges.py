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


@pytest.mark.parametrize("Hkv,cap", [(8, 2000), (2, 4000)])     # eight tiles a split, a wave each; five: waves without a tile
@pytest.mark.parametrize("d,G", [(128, 4), (128, 17), (64, 3), (64, 24)])
def test_decode_splits_past_the_count(oracle, d, G, Hkv, cap):
    """Caches far from full: waves and whole splits whose first tile, asked for ahead of the count, lies past it.  The rows
    there are poison."""
    B, T = 4, 5
    print(f"decode past the count d={d} G={G} Hkv={Hkv} cap={cap}", flush=True)
    q, kc, vc, cnt, kt, vt = _case(B, G * Hkv, Hkv, cap, T, d, seed=d + G + cap)
    cnt[:, 0::2] = [[1], [33], [0], [cap // 5]]
    for b in range(B):
        for g in range(Hkv):
            kc[b, g, cnt[b, g]:] = float("nan"); vc[b, g, cnt[b, g]:] = float("nan")
    _check(oracle, (q, kc, vc, cnt, kt, vt))


@pytest.mark.parametrize("dtype,d,n,n_hat", [
    ("bf16", 128, 9001, 67),       # two row blocks, 141 key blocks: items in many parts
    ("bf16", 64, 6400, 128),       # one whole row block
    ("f32", 64, 3000, 130),
    ("f32", 128, 2049, 1),         # one row
])
def test_prefill_parts_of_long_items(oracle, dtype, d, n, n_hat):
    """Few row blocks over a long context: items are cut into parts and put together again; into fewer in a workspace with
    less room for them, into none in one without, with the same result."""
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
    # the parts' results take (4 d + 8) * 128 bytes each, at least a dozen at a time; everything else less than 64 KB
    some, none = binding.Context(workspace=2 << 20), binding.Context(workspace=1 << 18)
    tol = (2e-2, 5e-3, 2e-3) if dtype == "bf16" else (1e-4, 1e-5, 1e-4)
    for ctx in (pipe.ctx, some, none):
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


@pytest.mark.parametrize("B,Hq,Hkv,n,n_hat", [(1, 1, 1, 1, 1), (2, 8, 2, 900, 900), (1, 40, 5, 300, 129), (1, 24, 8, 2000, 1)])
def test_prefill_in_the_smallest_workspace(oracle, B, Hq, Hkv, n, n_hat):
    """The eight work queues lie one behind the other: the call needs 20 bytes per item (row block of a head) beside the
    bitmap and tables of each head, and says so where they are not there."""
    from tests.gpu_util import Pipeline, dev_lists
    from tests.test_gpu_random_shapes import _selection
    print(f"smallest workspace B={B} Hq={Hq} Hkv={Hkv} n={n} n_hat={n_hat}", flush=True)
    q, k, v = inputs.make_plain(B, Hq, Hkv, n, n_hat, 64, dtype="bf16", seed=n, q_scale=1.5)
    lists = _selection(np.random.default_rng(n), B, Hq, n)
    ref, _ = oracle.attend(q, k, v, *lists)
    pipe = Pipeline(q, k, v, 1, "bf16")
    up = lambda x: (x + 255) // 256 * 256
    heads, blocks = B * Hq, (n - (n - n_hat) // 128 * 128 + 127) // 128
    table = n // 64 + 4
    need = up(heads * ((n + 31) // 32 + 12) * 4) + up(heads * 4) + up(heads * (table + 1) * 2) + up(heads * blocks * 4) + 256 + up(heads * table) + up(heads * blocks * 16)
    pipe.ctx = binding.Context(workspace=need)
    out, _ = pipe.prefill(dev_lists(*lists), sentinel=True)
    queues, nqb, cuts = pipe.ctx.debug_prefill_queues(pipe.shape)
    assert nqb == blocks and cuts == 0
    items = np.sort(np.concatenate(queues))
    np.testing.assert_array_equal(items, np.sort([h << 16 | b for h in range(heads) for b in range(blocks)]))
    err = np.abs(out.float().cpu().numpy().reshape(-1, 64) - ref)
    assert err.max() <= 2e-2 and err.mean() <= 5e-3
    pipe.ctx = binding.Context(workspace=need - 256)
    with pytest.raises(binding.LoopServeError):
        pipe.prefill(dev_lists(*lists))


@pytest.mark.parametrize("d,splits", [(128, 7), (64, 2), (128, 1)])
def test_decode_with_room_for_fewer_splits(oracle, d, splits):
    """ls_decode_attend cuts the keys into as many splits as the workspace has room for."""
    B, Hkv, G, cap, T = 1, 4, 4, 3000, 9
    print(f"decode splits d={d} splits={splits}", flush=True)
    q, kc, vc, cnt, kt, vt = _case(B, G * Hkv, Hkv, cap, T, d, seed=splits)
    shape = binding.make_shape(B, G * Hkv, Hkv, d, cap + T, 1, 1, "bf16")
    room = B * G * Hkv * splits * (d + 4) * 4
    assert room + 256 < binding.decode_workspace_bytes(shape, cap, T)
    ctx = binding.Context(workspace=room)
    out = torch.full((B, G * Hkv, d), float("nan"), dtype=torch.bfloat16, device="cuda")
    ctx.ls_decode_attend(shape, q.cuda(), kc.cuda(), vc.cuda(), torch.from_numpy(cnt).cuda(), kt.cuda(), vt.cuda(), out, None)
    ref, _ = oracle.decode(q.float().numpy(), kc.float().numpy(), vc.float().numpy(), cnt, kt.float().numpy(), vt.float().numpy())
    assert np.abs(out.float().cpu().numpy() - ref).max() <= 2e-2


@pytest.mark.parametrize("B,Hq,Hkv,n,w,d,dtype", [
    (1, 8, 1, 127, 1, 128, "bf16"),        # one row, less than a key block; heads shared out over eight workgroups
    (1, 6, 2, 128, 33, 64, "bf16"),        # exactly one key block; a chunk of one row; three heads a KV head: no sharing
    (2, 8, 2, 257, 31, 128, "bf16"),       # one key in the last block; rows that do not exist in every chunk
    (1, 12, 2, 385, 128, 64, "f32"),       # heads shared by two only (6 = 2 x 3); longest window with diagonals in LDS
    (1, 2, 2, 640, 129, 128, "bf16"),      # shortest window whose diagonals come from the written matrix
    (8, 16, 8, 3000, 16, 64, "bf16"),      # more than 1024 workgroups: no sharing
    (1, 1, 1, 33000, 40, 64, "bf16"),      # more key blocks than a thread of the merge keeps
])
def test_score_chunks_and_shares(oracle, B, Hq, Hkv, n, w, d, dtype):
    from tests.gpu_util import Pipeline, host
    from tests.test_gpu_parity import _score_close
    print(f"score edge B={B} Hq={Hq} Hkv={Hkv} n={n} w={w} d={d} {dtype}", flush=True)
    q, k, v = inputs.make_plain(B, Hq, Hkv, n, w, d, dtype=dtype, seed=n + w, q_scale=2.0)
    pipe = Pipeline(q, k, v, w, dtype)
    _score_close(host(pipe.score()), oracle.score(q, k), w)


@pytest.mark.parametrize("w,dtype", [(1, "bf16"), (40, "bf16"), (200, "f32")])
def test_score_positions_in_head_groups(oracle, w, dtype):
    """Scoring positions given: the window matrix passes through the workspace for as many KV heads as it takes."""
    from tests.gpu_util import Pipeline, host
    from tests.test_gpu_parity import _score_close
    B, Hq, Hkv, n, d = 2, 6, 3, 700, 64
    q, k, v = inputs.make_plain(B, Hq, Hkv, n, w, d, dtype=dtype, seed=w, q_scale=2.0)
    pos = np.sort(np.random.default_rng(w).choice(n, size=w, replace=False))
    ref = oracle.score(q, k, q_pos=pos)
    pipe = Pipeline(q, k, v, w, dtype)
    whole = host(pipe.score(q_pos=pos))
    _score_close(whole, ref, w)
    one = Hq // Hkv * w * n * 4
    part = B * Hkv * ((n + 127) // 128) * (Hq // Hkv) * w * 8 + B * Hq * w * 8 + 4096
    print(f"head groups w={w} matrix {one} bytes a KV head", flush=True)
    pipe.ctx = binding.Context(workspace=part + 4 * one + one // 2)      # four of six KV heads at a time
    some = host(pipe.score(q_pos=pos))
    for name in whole:
        np.testing.assert_array_equal(whole[name], some[name])


@pytest.mark.parametrize("B,Hq,Hkv,n,w,rows,given", [
    (1, 2, 1, 700, 40, 1, True),           # a row at a time: every chunk passed once for each of its rows
    (1, 2, 1, 700, 40, 4, True),           # what the diagonals of the last rows take at one KV head
    (2, 6, 3, 700, 100, 33, True),         # one chunk of one KV head at a time
    (1, 6, 2, 900, 100, 70, True),         # one of them in two bands, rather than both chunk by chunk
    (1, 8, 4, 385, 70, 100, True),         # three KV heads chunk by chunk, then one
    (1, 4, 2, 600, 256, 31, True),         # parts of chunks that differ in length
    (2, 4, 2, 640, 129, 64, False),        # the last 129 rows: two chunks a band, the last of one row
])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_score_matrix_in_bands(oracle, B, Hq, Hkv, n, w, rows, given, dtype):
    """The window matrix passes through the workspace in bands of as many rows of KV heads as it takes, with the same sums."""
    from tests.gpu_util import Pipeline, host
    from tests.test_gpu_parity import _score_close
    print(f"bands B={B} Hq={Hq} Hkv={Hkv} n={n} w={w} rows={rows} {dtype}", flush=True)
    d = 64
    q, k, v = inputs.make_plain(B, Hq, Hkv, n, w, d, dtype=dtype, seed=w + n, q_scale=2.0)
    pos = np.sort(np.random.default_rng(w).choice(n, size=w, replace=False)) if given else None
    pipe = Pipeline(q, k, v, w, dtype)
    up = lambda x: (x + 255) // 256 * 256
    front = up(B * Hq * w * ((n + 127) // 128) * 8) + up(B * Hq * w * 8)
    row = Hq // Hkv * n * 4
    pipe.ctx = binding.Context(workspace=front + B * Hkv * w * row)
    whole = host(pipe.score(q_pos=pos))
    _score_close(whole, oracle.score(q, k, q_pos=pos), w)
    pipe.ctx = binding.Context(workspace=front + rows * row)
    bands = host(pipe.score(q_pos=pos))
    for name in whole:
        np.testing.assert_array_equal(whole[name], bands[name])
    pipe.ctx = binding.Context(workspace=front + row - 1)
    with pytest.raises(binding.LoopServeError):
        pipe.score(q_pos=pos)


@pytest.mark.parametrize("Hq,Hkv,ln,n_obs,d,dtype", [
    (4, 4, 129, 8, 64, "bf16"),            # one head a KV head: a chunk of eight rows
    (10, 2, 300, 8, 128, "bf16"),          # forty rows: a whole chunk and one of eight
    (6, 2, 257, 16, 64, "f32"),            # forty-eight rows: a whole chunk and half of one
    (16, 1, 1000, 16, 128, "bf16"),        # eight whole chunks
    (4, 2, 200, 5, 64, "bf16"),            # no divisor of 32: a chunk per head
    (4, 2, 500, 40, 128, "f32"),           # two chunks per head
])
def test_retention_score_chunks(oracle, Hq, Hkv, ln, n_obs, d, dtype):
    from tests.gpu_util import Pipeline
    print(f"retention edge Hq={Hq} Hkv={Hkv} len={ln} n_obs={n_obs} d={d} {dtype}", flush=True)
    q, k, v = inputs.make_plain(1, Hq, Hkv, ln, n_obs, d, dtype=dtype, seed=ln, q_scale=2.0)
    budget = 32
    ref = oracle.compress(q, k, budget)
    pipe = Pipeline(q, k, v, n_obs, dtype, budget=budget)
    keep_idx = torch.full((1, Hkv, budget), -1, dtype=torch.int32, device="cuda")
    keep_cnt = torch.zeros((1, Hkv), dtype=torch.int32, device="cuda")
    k_out = torch.zeros((1, Hkv, budget, d), dtype=pipe.k.dtype, device="cuda")
    pipe.ctx.ls_kv_compress(pipe.shape, budget, pipe.q, pipe.k, pipe.v, keep_idx, keep_cnt, k_out, torch.zeros_like(k_out))
    score = torch.empty((1, Hkv, ln), dtype=torch.float32, device="cuda")
    pipe.ctx.debug_compress_score(pipe.shape, score)
    np.testing.assert_allclose(score.cpu().numpy(), ref["score"], rtol=1e-3, atol=1e-6 * n_obs)


@pytest.mark.parametrize("n,w,alpha,kind", [
    (1, 1, 0.9, "spiky"),
    (65, 64, 0.95, "spiky"),               # the window is almost the context
    (1024, 33, 1.0, "flat"),               # one block of candidates, every line taken
    (1025, 256, 0.95, "flat"),             # a block of one candidate; longest window
    (3000, 97, 0.95, "spiky"),             # picks change lists all the time
    (5000, 64, 0.98, "ties"),              # few distinct weights: sums with ties in rounding, long runs
    (2500, 40, 0.9, "repeated"),           # scoring positions given, some of them twice
    (262144, 2, 0.3, "flat"),              # longest context: largest bitmaps
])
def test_exact_walk_rounds(oracle, n, w, alpha, kind):
    """ls_select_exact on synthetic window matrices against the oracle, to the last bit."""
    from tests.gpu_util import host
    from tests.test_gpu_configs import check_selection_exact
    print(f"exact walk n={n} w={w} alpha={alpha} {kind}", flush=True)
    rng = np.random.default_rng(n + w)
    H = 2
    pos = None
    if kind == "repeated":
        pos = np.sort(rng.integers(n // 2, n, w)); pos[1] = pos[0]
    p = np.arange(n - w, n) if pos is None else pos
    a = rng.exponential(size=(1, H, w, n)) ** (4 if kind == "spiky" else 1)
    if kind == "ties":
        a = np.round(a * 2) / 8 + 0.125
    a[0, :, np.arange(n)[None, :] > p[:, None]] = 0
    a = np.ascontiguousarray((a if kind == "ties" else a / a.sum(-1, keepdims=True)).astype(np.float32))
    vert = a.sum(2, dtype=np.float64)
    slash = np.zeros((1, H, n))
    for t in range(w):
        slash[0, :, :p[t] + 1] += a[0, :, t, p[t]::-1] if p[t] < n else 0
    sc = dict(vert=vert.astype(np.float32), slash=slash.astype(np.float32), total=vert.sum(-1).astype(np.float32))
    n_hat = max(w, n // 3)
    ref = oracle.select_exact(a, sc, n_hat, alpha, q_pos=pos)
    shape = binding.make_shape(1, H, 1, 64, n, n_hat, w, "f32", 0.0)
    ctx = binding.Context(shape)
    out = binding.alloc_select(shape, accounted=True)
    dev = {k: torch.from_numpy(v).cuda() for k, v in sc.items()}
    ctx.ls_select_exact(shape, alpha, torch.from_numpy(a).cuda(), dev["vert"], dev["slash"], dev["total"], out["v_idx"],
                        out["v_cnt"], out["s_idx"], out["s_cnt"], out["accounted"],
                        None if pos is None else torch.from_numpy(pos.astype(np.int64)).cuda())
    assert ctx.ls_poll_status() == 0
    gpu = host(out)
    print("  picks", ref["v_cnt"].ravel().tolist(), ref["s_cnt"].ravel().tolist(), flush=True)
    check_selection_exact(gpu, ref)
    np.testing.assert_array_equal(gpu["accounted"], ref["accounted"])


@pytest.mark.parametrize("n,alpha,kind", [
    (511, 1.0, "ties"), (513, 1.0, "ties"),      # a run of one entry less / more than the waves look at
    (5000, 1.0, "ties"),                         # multiples of 1/8 on sums of 2^20 and more: every other addition is a tie
    (4097, 1.0, "wide"),                         # weights over sixty binades: sums that leave theirs all the time
    (9000, 1.0, "halves"),                       # long runs of equal gains that are half the spacing of the sum
    (2100, 0.95, "alternate"),                   # picks that change lists all the time
])
def test_walk_sums(oracle, n, alpha, kind):
    """ls_select on synthetic line weights against the oracle, to the last bit, with and without the sum."""
    from tests.gpu_util import host
    from tests.test_gpu_configs import check_selection_exact
    print(f"walk sums n={n} alpha={alpha} {kind}", flush=True)
    rng = np.random.default_rng(n)
    H = 4
    v, s = rng.exponential(size=(2, 1, H, n))
    if kind == "ties":
        v, s = v * 1e-6, np.round(s * 8) / 8 + 0.125         # (all picks are diagonals: their gains are the weights)
        s[..., 0] = 2.0 ** 20 * (1 + np.arange(H))
    elif kind == "wide":
        v, s = np.exp2(60 * rng.random((2, 1, H, n)) - 50)
    elif kind == "halves":
        v, s = v * 1e-6, np.full((1, H, n), 2.0 ** -12); s[..., 0] = 2.0 ** 12 + 2.0 ** -11 * np.arange(H); s[..., 5] = 0.75
    elif kind == "alternate":
        v = np.arange(n, 0, -1)[None, None] + 0.25 * rng.random((1, H, n)); s = np.arange(n, 0, -1)[None, None] + 0.25 * rng.random((1, H, n))
    m = 1e-3 if kind in ("halves", "alternate") else 0.05
    sc = dict(vert=v, slash=s, vmax=v * m * rng.random((1, H, n)), smax=s * m * rng.random((1, H, n)), total=np.maximum(v.sum(-1), s.sum(-1)))
    sc = {k: np.ascontiguousarray(x, dtype=np.float32) for k, x in sc.items()}
    n_hat = n // 2
    ref = oracle.select(sc, n_hat, alpha)
    shape = binding.make_shape(1, H, 1, 64, n, n_hat, 1, "f32", 0.0)
    ctx = binding.Context(shape)
    dev = {k: torch.from_numpy(x).cuda() for k, x in sc.items()}
    for accounted in (True, False):
        out = binding.alloc_select(shape, accounted=accounted)
        ctx.ls_select(shape, alpha, dev["vert"], dev["slash"], dev["vmax"], dev["smax"], dev["total"], out["v_idx"], out["v_cnt"],
                      out["s_idx"], out["s_cnt"], out["accounted"])
        assert ctx.ls_poll_status() == 0
        print("  picks", ref["v_cnt"].ravel().tolist(), ref["s_cnt"].ravel().tolist(), flush=True)
        gpu = {k: x for k, x in out.items() if x is not None}
        gpu = host(gpu)
        check_selection_exact(gpu, ref)
        if accounted:
            np.testing.assert_array_equal(gpu["accounted"], ref["accounted"])


@pytest.mark.parametrize("n", [1, 63, 64, 65, 1023, 1024, 1025, 2047, 2048, 2049, 8191, 8192, 8193])
def test_sorted_and_emitted_lists(oracle, n):
    """Lengths around the waves' shares of a list, the lists in one range and those that the walk writes out itself; few distinct
    weights, so that the order of equal ones shows."""
    from tests.gpu_util import host
    from tests.test_gpu_configs import check_selection_exact
    print(f"sorted lists n={n}", flush=True)
    rng = np.random.default_rng(n)
    H = 3
    v, s = rng.integers(1, 40, size=(2, 1, H, n)) / 8.0
    s[:, 1] *= 1e-3; v[:, 0] *= 1e-3                                  # one head of columns, one of diagonals, one of both
    sc = dict(vert=v, slash=s, vmax=v * 1e-7, smax=s * 1e-7, total=np.maximum(v.sum(-1), s.sum(-1)))
    sc = {k: np.ascontiguousarray(x, dtype=np.float32) for k, x in sc.items()}
    ref = oracle.select(sc, max(1, n // 3), 0.7)
    shape = binding.make_shape(1, H, 1, 64, n, max(1, n // 3), 1, "f32", 0.0)
    ctx = binding.Context(shape)
    out = binding.alloc_select(shape, accounted=True)
    dev = {k: torch.from_numpy(x).cuda() for k, x in sc.items()}
    ctx.ls_select(shape, 0.7, dev["vert"], dev["slash"], dev["vmax"], dev["smax"], dev["total"], out["v_idx"], out["v_cnt"],
                  out["s_idx"], out["s_cnt"], out["accounted"])
    assert ctx.ls_poll_status() == 0
    gpu = host(out)
    check_selection_exact(gpu, ref)
    np.testing.assert_array_equal(gpu["accounted"], ref["accounted"])


@pytest.mark.parametrize("n,w,G", [(2048, 64, 4), (2049, 64, 4), (700, 100, 8), (900, 1, 1), (300, 33, 17)])
def test_score_merges_row_statistics_itself(oracle, n, w, G):
    """Up to sixteen key blocks and 32 chunks of rows the line sums' kernel merges the row statistics; with more of either a
    kernel of its own does."""
    from tests.gpu_util import Pipeline, host
    from tests.test_gpu_parity import _score_close
    print(f"row statistics n={n} w={w} G={G}", flush=True)
    q, k, v = inputs.make_plain(1, 2 * G, 2, n, w, 64, dtype="bf16", seed=n + w, q_scale=2.0)
    _score_close(host(Pipeline(q, k, v, w, "bf16").score()), oracle.score(q, k), w)


@pytest.mark.parametrize("ln,budget,d,dtype", [
    (4096, 1, 64, "bf16"), (4097, 4096, 64, "bf16"),                  # keys per thread: 4 -> 16; all but one kept
    (16384, 700, 128, "f32"), (16385, 16001, 64, "bf16"),             # 16 -> 32
    (32768, 65, 128, "bf16"), (32769, 2000, 64, "bf16"),              # one workgroup a head -> many
    (50, 50, 64, "f32"),                                              # all kept
])
def test_retention_sizes(oracle, ln, budget, d, dtype):
    """Lengths around the forms of the top-B selection, budgets around a workgroup's rows of the gather; repeated key rows, so
    that the threshold falls among equal scores."""
    from tests.gpu_util import Pipeline
    print(f"retention sizes len={ln} budget={budget} d={d} {dtype}", flush=True)
    q, k, v = inputs.make_plain(1, 4, 2, ln, 8, d, dtype=dtype, seed=ln, q_scale=2.0)
    k = np.ascontiguousarray(k[:, :, np.arange(ln) % 97])
    pipe = Pipeline(q, k, v, 8, dtype, budget=budget)
    keep_idx = torch.full((1, 2, budget), -1, dtype=torch.int32, device="cuda")
    keep_cnt = torch.zeros((1, 2), dtype=torch.int32, device="cuda")
    k_out = torch.zeros((1, 2, budget, d), dtype=pipe.k.dtype, device="cuda")
    v_out = torch.zeros_like(k_out)
    pipe.ctx.ls_kv_compress(pipe.shape, budget, pipe.q, pipe.k, pipe.v, keep_idx, keep_cnt, k_out, v_out)
    score = torch.empty((1, 2, ln), dtype=torch.float32, device="cuda")
    pipe.ctx.debug_compress_score(pipe.shape, score)
    assert keep_cnt.cpu().tolist() == [[min(budget, ln)] * 2]
    for h in range(2):
        got = keep_idx[0, h].cpu().numpy()
        np.testing.assert_array_equal(got, oracle.topb(score[0, h].cpu().numpy(), budget))
        at = torch.from_numpy(got.astype(np.int64)).cuda()
        assert torch.equal(k_out[0, h], pipe.k[0, h, at]) and torch.equal(v_out[0, h], pipe.v[0, h, at])


@pytest.mark.parametrize("B,Hkv,ln,budget", [
    (4, 8, 16385, 16384), (4, 8, 32768, 300),                         # heads enough for one workgroup each, 32 keys a thread
    (4, 8, 32769, 300), (31, 1, 32768, 5000),                         # too long for one; a head too few
])
def test_retention_of_many_heads(oracle, B, Hkv, ln, budget):
    """Where one workgroup per head ends and the launches spread over the chip begin, by length and by heads."""
    print(f"retention of many heads B={B} Hkv={Hkv} len={ln} budget={budget}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(ln)
    k = torch.randn(B, Hkv, 97, 64, device="cuda", generator=g).to(torch.bfloat16)[:, :, torch.arange(ln, device="cuda") % 97].contiguous()
    q = torch.randn(B, Hkv, 8, 64, device="cuda", generator=g).to(torch.bfloat16)
    shape = binding.make_shape(B, Hkv, Hkv, 64, ln, 1, 8, "bf16")
    ctx = binding.Context(shape, budget)
    keep_idx = torch.full((B, Hkv, budget), -1, dtype=torch.int32, device="cuda")
    keep_cnt = torch.zeros((B, Hkv), dtype=torch.int32, device="cuda")
    ctx.ls_kv_compress(shape, budget, q, k, None, keep_idx, keep_cnt)
    score = torch.empty((B, Hkv, ln), dtype=torch.float32, device="cuda")
    ctx.debug_compress_score(shape, score)
    assert (keep_cnt == budget).all()
    for b in range(B):
        for h in range(Hkv):
            np.testing.assert_array_equal(keep_idx[b, h].cpu().numpy(), oracle.topb(score[b, h].cpu().numpy(), budget))


def test_profile_covers_the_parts():
    """ls_profile_* with and without room for parts: every call counted, the time of its kernels below the calls' own."""
    from tests.gpu_util import Pipeline, dev_lists
    n, n_hat, H = 9000, 100, 8
    q, k, v = inputs.make_plain(1, H, 2, n, n_hat, 128, dtype="bf16", seed=1)
    every = np.broadcast_to(np.arange(n, dtype=np.int32), (1, H, n))
    lists = dev_lists(every, np.full((1, H), n), every, np.full((1, H), n))       # dense heads: 141 tiles an item
    pipe = Pipeline(q, k, v, 1, "bf16")
    times = []
    for ctx in (pipe.ctx, binding.Context(workspace=1 << 18)):
        pipe.ctx = ctx
        pipe.prefill(lists)
        ctx.profile_enable(True)
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        for _ in range(10):
            pipe.prefill(lists)
        e1.record()
        torch.cuda.synchronize()
        ms, calls = ctx.profile_prefill_kernel_ms()
        ctx.profile_enable(False)
        assert calls == 10 and 0 < ms < e0.elapsed_time(e1) / 10
        times.append(ms)
    print("attention kernels in parts and whole, ms:", times, flush=True)
    assert times[0] < times[1]                             # sixteen items on 256 compute units: parts win, combining included
