"""The scoring passes over ranges of keys at their edges: few rows a workgroup, two waves on one chunk and one wave on two, contexts that end inside a tile, one tile in
all, rows of long contexts that see little of it, and logits whose reference has to move late.  Against float64."""
import math

import numpy as np
import pytest
import torch

from paper_2507_13681_amd import binding, inputs
from tests.gpu_util import Pipeline, host

pytestmark = pytest.mark.gpu


def _window(q, k, pos, scale):
    """[B, Hq, w, n] causal probabilities in float64."""
    B, Hq, w, d = q.shape
    n, G = k.shape[2], Hq // k.shape[1]
    x = np.einsum("bhtd,bhnd->bhtn", q.astype(np.float64), np.repeat(k, G, axis=1).astype(np.float64)) * scale
    x[:, :, np.arange(n)[None, :] > np.asarray(pos)[:, None]] = -np.inf
    x = np.exp(x - x.max(-1, keepdims=True))
    return x / x.sum(-1, keepdims=True)


@pytest.mark.parametrize("B,Hq,Hkv,n,w,d", [(1, 4, 4, 63, 5, 128), (1, 4, 4, 65, 33, 64), (1, 8, 2, 129, 16, 128), (2, 6, 2, 1000, 40, 64), (1, 4, 1, 2177, 64, 128),
                                          (1, 8, 1, 3001, 100, 128), (1, 16, 2, 4100, 128, 64), (1, 2, 1, 5003, 256, 128), (1, 8, 8, 9001, 8, 128)])
@pytest.mark.parametrize("rising", [False, True])
def test_scores_over_ranges(B, Hq, Hkv, n, w, d, rising):
    print(f"score ranges B={B} Hq={Hq} Hkv={Hkv} n={n} w={w} d={d} rising={rising}", flush=True)
    q, k, v = inputs.make_plain(B, Hq, Hkv, n, w, d, dtype="bf16", seed=n + w, q_scale=1.5)
    if rising:                                             # the largest logits come last, by far: 2^60 and more above the first
        q[..., 0], k[..., 0] = 4.0, np.round(np.linspace(-16, 16, n)).astype(np.float32)
    rng = np.random.default_rng(n)
    for pos in (None, np.sort(rng.choice(n, size=w, replace=False)).astype(np.int64)):
        pipe = Pipeline(q, k, v, w, "bf16")
        got = host(pipe.score(q_pos=pos))
        at = np.arange(n - w, n) if pos is None else pos
        A = _window(q, k, at, 1 / math.sqrt(d))
        slash, smax = np.zeros((B, Hq, n)), np.zeros((B, Hq, n))
        for t, p in enumerate(at):
            diag = A[:, :, t, :p + 1][..., ::-1]
            slash[..., :p + 1] += diag
            smax[..., :p + 1] = np.maximum(smax[..., :p + 1], diag)
        for name, want in (("vert", A.sum(2)), ("vmax", A.max(2)), ("slash", slash), ("smax", smax), ("total", A.sum((2, 3)))):
            # exact products, sums of at most n terms, hardware exp2 of arguments of up to 2^7: as everywhere for ls_score
            np.testing.assert_allclose(got[name].reshape(want.shape), want, rtol=1e-3, atol=1e-6 * w, err_msg=name)


@pytest.mark.parametrize("Hq,Hkv,n,w,d", [(8, 8, 25600, 8, 64), (8, 8, 25601, 8, 64), (4, 1, 4096, 128, 128), (8, 2, 2049, 1, 64), (4, 2, 129, 128, 64), (12, 4, 6000, 97, 128)])
def test_key_blocks_that_join_their_results(Hq, Hkv, n, w, d):
    """As many workgroups as still add shared diagonals and totals themselves, and one row of blocks more; several groups of blocks, one, a block of one
    key; no shared diagonals.  Again and again on one context: the same bits, whoever comes last."""
    print(f"joined blocks Hq={Hq} Hkv={Hkv} n={n} w={w} d={d}", flush=True)
    q, k, v = inputs.make_plain(1, Hq, Hkv, n, w, d, dtype="bf16", seed=n + w, q_scale=1.5)
    pipe = Pipeline(q, k, v, w, "bf16")
    got = host(pipe.score())
    A = _window(q, k, np.arange(n - w, n), 1 / math.sqrt(d))
    slash, smax = np.zeros((1, Hq, n)), np.zeros((1, Hq, n))
    for t in range(w):
        p = n - w + t
        diag = A[:, :, t, :p + 1][..., ::-1]
        slash[..., :p + 1] += diag
        smax[..., :p + 1] = np.maximum(smax[..., :p + 1], diag)
    for name, want in (("vert", A.sum(2)), ("vmax", A.max(2)), ("slash", slash), ("smax", smax), ("total", A.sum((2, 3)))):
        np.testing.assert_allclose(got[name].reshape(want.shape), want, rtol=1e-3, atol=1e-6 * w, err_msg=name)      # as above
    for _ in range(3):
        again = host(pipe.score())
        for name in got:
            np.testing.assert_array_equal(again[name], got[name], err_msg=name)


@pytest.mark.parametrize("Hq,Hkv,n,w,packed", [(24, 8, 44001, 32, False), (7, 1, 150003, 32, False), (48, 8, 17002, 16, True), (11, 1, 140003, 8, True)])
def test_three_chunks_of_rows_for_four_waves(Hq, Hkv, n, w, packed):
    """A workgroup of the statistics pass with three chunks of 32 rows, or of up to 32: its fourth wave has none, and no rows to read (in the last
    KV head there are none behind).  `packed`: windows that share chunks, as the retention score has them."""
    print(f"three chunks Hq={Hq} Hkv={Hkv} n={n} w={w}", flush=True)
    G, d = Hq // Hkv, 64
    chunks = -(-G * w // 32)
    assert chunks % 4 == 3 and Hkv * -(-n // 128) * chunks >= (3072 if packed else 8192)       # four chunks a workgroup, ranges of keys
    q, k, v = inputs.make_plain(1, Hq, Hkv, n, w, d, dtype="bf16", seed=n, q_scale=1.5)
    A = _window(q, k, np.arange(n - w, n), 1 / math.sqrt(d))
    if not packed:
        got = host(Pipeline(q, k, v, w, "bf16").score())
        for name, want in (("vert", A.sum(2)), ("vmax", A.max(2)), ("total", A.sum((2, 3)))):
            np.testing.assert_allclose(got[name].reshape(want.shape), want, rtol=1e-3, atol=1e-6 * w, err_msg=name)      # as above
        return
    dev = lambda x: torch.from_numpy(x).cuda().to(torch.bfloat16)
    shape, budget = binding.make_shape(1, Hq, Hkv, d, n, 1, w, "bf16"), 500
    idx, cnt = torch.empty(1, Hkv, budget, dtype=torch.int32, device="cuda"), torch.empty(1, Hkv, dtype=torch.int32, device="cuda")
    binding.Context(shape, budget).ls_kv_compress(shape, budget, dev(q), dev(k), dev(v), idx, cnt, None, None)
    score = A.reshape(Hkv, G * w, n).sum(1)
    for g in range(Hkv):
        assert cnt[0, g].item() == budget
        threshold = np.sort(score[g])[-budget]
        for i in set(np.argsort(-score[g], kind="stable")[:budget]).symmetric_difference(idx[0, g].tolist()):
            assert abs(score[g, i] - threshold) <= 1e-3 * threshold            # as below


@pytest.mark.parametrize("n,w,d", [(1, 1, 64), (32, 32, 128), (33, 31, 64), (100, 97, 128), (128, 128, 64), (129, 1, 128), (160, 128, 128), (255, 127, 64), (257, 33, 128), (300, 61, 64)])
def test_rows_that_see_a_part_of_a_block(n, w, d):
    """Newest rows that begin, end or lie inside a block of 128 keys, and chunks of fewer than 32 rows."""
    print(f"rows in a block n={n} w={w} d={d}", flush=True)
    q, k, v = inputs.make_plain(1, 4, 2, n, w, d, dtype="bf16", seed=n + w, q_scale=1.5)
    got = host(Pipeline(q, k, v, w, "bf16").score())
    A = _window(q, k, np.arange(n - w, n), 1 / math.sqrt(d))
    slash, smax = np.zeros((1, 4, n)), np.zeros((1, 4, n))
    for t in range(w):
        p = n - w + t
        diag = A[:, :, t, :p + 1][..., ::-1]
        slash[..., :p + 1] += diag
        smax[..., :p + 1] = np.maximum(smax[..., :p + 1], diag)
    for name, want in (("vert", A.sum(2)), ("vmax", A.max(2)), ("slash", slash), ("smax", smax), ("total", A.sum((2, 3)))):
        np.testing.assert_allclose(got[name].reshape(want.shape), want, rtol=1e-3, atol=1e-6 * w, err_msg=name)      # as above


@pytest.mark.parametrize("B,Hq,Hkv,n,n_obs,d,budget", [(1, 4, 1, 300, 8, 128, 100), (2, 8, 1, 1025, 16, 64, 1000), (1, 8, 2, 4097, 32, 128, 64), (1, 3, 3, 8191, 5, 64, 77), (1, 8, 1, 2049, 16, 128, 512),
                                                      (1, 8, 1, 2050, 32, 128, 512)])
def test_retention_with_few_rows(B, Hq, Hkv, n, n_obs, d, budget):
    """Kept entries against float64 scores: the same, up to entries within 1e-3 of the threshold."""
    print(f"retention B={B} Hq={Hq} n={n} n_obs={n_obs} d={d}", flush=True)
    q, k, v = inputs.make_plain(B, Hq, Hkv, n, n_obs, d, dtype="bf16", seed=n, q_scale=1.5)
    dev = lambda x: torch.from_numpy(x).cuda().to(torch.bfloat16)
    shape = binding.make_shape(B, Hq, Hkv, d, n, 1, n_obs, "bf16")
    idx, cnt = torch.empty(B, Hkv, budget, dtype=torch.int32, device="cuda"), torch.empty(B, Hkv, dtype=torch.int32, device="cuda")
    binding.Context(shape, budget).ls_kv_compress(shape, budget, dev(q), dev(k), dev(v), idx, cnt, None, None)
    score = _window(q, k, np.arange(n - n_obs, n), 1 / math.sqrt(d)).reshape(B, Hkv, Hq // Hkv, n_obs, n).sum((2, 3))
    for b in range(B):
        for g in range(Hkv):
            assert cnt[b, g].item() == budget
            kept = idx[b, g].cpu().numpy()
            assert np.all(np.diff(kept) > 0)
            threshold = np.sort(score[b, g])[-budget]
            want = set(np.argsort(-score[b, g], kind="stable")[:budget])
            for i in want.symmetric_difference(kept.tolist()):
                assert abs(score[b, g, i] - threshold) <= 1e-3 * threshold
