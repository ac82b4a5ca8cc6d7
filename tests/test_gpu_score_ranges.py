"""The scoring passes at their edges, against float64: statistics by a workgroup per 128 keys and by ranges of keys (few rows a workgroup, two waves on one chunk and one
wave on two, contexts that end inside a tile, ranges of one tile, logits whose reference has to move late), key blocks that join their results, the retention's second pass.  Which
kernels a shape takes is asserted: the library says so itself."""
import math

import numpy as np
import pytest
import torch

from paper_2507_13681_amd import binding, inputs
from tests.gpu_util import Pipeline, host

pytestmark = pytest.mark.gpu


def _reference(q, k, at):
    """The line sums and maxima of rows at positions `at` (bf16 tensors q [B, Hq, w, d], k [B, Hkv, n, d] on the GPU) in float64, head by head."""
    B, Hq, w, d = q.shape
    n, G = k.shape[2], Hq // k.shape[1]
    out = {name: np.zeros((B, Hq, n)) for name in ("vert", "vmax", "slash", "smax")}
    hidden = torch.arange(n, device="cuda")[None, :] > torch.from_numpy(np.asarray(at)).cuda()[:, None]
    for b in range(B):
        for h in range(Hq):
            x = (q[b, h].double() @ k[b, h // G].double().T.contiguous()) / math.sqrt(d)
            A = torch.softmax(x.masked_fill(hidden, -math.inf), dim=-1)
            slash, smax = torch.zeros(n, device="cuda", dtype=torch.float64), torch.zeros(n, device="cuda", dtype=torch.float64)
            for t, p in enumerate(at):
                diag = A[t, :p + 1].flip(-1)
                slash[:p + 1] += diag
                smax[:p + 1] = torch.maximum(smax[:p + 1], diag)
            for name, x in (("vert", A.sum(0)), ("vmax", A.amax(0)), ("slash", slash), ("smax", smax)):
                out[name][b, h] = x.cpu().numpy()
    out["total"] = out["vert"].sum(-1)
    return out


def _check(got, want, w):
    for name in want:                                      # exact products, sums of at most n terms, hardware exp2: as everywhere for ls_score
        np.testing.assert_allclose(got[name].reshape(want[name].shape), want[name], rtol=1e-3, atol=1e-6 * w, err_msg=name)


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
def test_scores_of_little_work(B, Hq, Hkv, n, w, d, rising):
    """Statistics by a workgroup per 128 keys."""
    print(f"scores of little work B={B} Hq={Hq} Hkv={Hkv} n={n} w={w} d={d} rising={rising}", flush=True)
    assert binding.score_route(binding.make_shape(B, Hq, Hkv, d, n, w, w, "bf16"), 0 if w <= 128 else 1)["ranges"] == 0
    q, k, v = inputs.make_plain(B, Hq, Hkv, n, w, d, dtype="bf16", seed=n + w, q_scale=1.5)
    if rising:                                             # the largest logits come last, 2^16 (d = 128) or 2^23 above the first
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


@pytest.mark.parametrize("B,Hq,Hkv,n,w,d,chunks,explicit", [
    (2, 40, 8, 13185, 32, 128, 4, False), (2, 32, 8, 8191, 64, 64, 4, False), (4, 64, 8, 6209, 64, 128, 8, False), (4, 40, 8, 9857, 64, 64, 8, False), (2, 16, 8, 4735, 200, 128, 4, False),
    (2, 32, 8, 8191, 64, 128, 4, True), (1, 32, 8, 8321, 100, 128, 4, True), (2, 16, 8, 4735, 200, 128, 4, True)])
def test_scores_over_ranges(B, Hq, Hkv, n, w, d, chunks, explicit):
    """Statistics by ranges of keys: five chunks of rows for workgroups of four, eight, sixteen and ten for workgroups of eight, a ragged window beyond 128 rows, and explicit
    positions; contexts that end one key into a tile and one key before its end."""
    print(f"score ranges B={B} Hq={Hq} Hkv={Hkv} n={n} w={w} d={d} explicit={explicit}", flush=True)
    route = binding.score_route(binding.make_shape(B, Hq, Hkv, d, n, w, w, "bf16"), 0 if w <= 128 and not explicit else 1, explicit)
    assert route["ranges"] > 1 and route["chunks"] == chunks and n % 64 in (1, 63)
    q, k, v = inputs.make_plain(B, Hq, Hkv, n, w, d, dtype="bf16", seed=n + w, q_scale=1.5)
    pos = np.sort(np.random.default_rng(n).choice(n, size=w, replace=False)).astype(np.int64) if explicit else None
    pipe = Pipeline(q, k, v, w, "bf16")
    _check(host(pipe.score(q_pos=pos)), _reference(pipe.q, pipe.k, np.arange(n - w, n) if pos is None else pos), w)


@pytest.mark.parametrize("B,n,d,explicit,joins", [(4, 5003, 64, False, True), (4, 5003, 128, False, True), (6, 5003, 128, False, False), (8, 2001, 64, False, True), (4, 5003, 128, True, False)])
def test_a_batch_has_the_bits_of_its_dialogues(B, n, d, explicit, joins):
    """A batch whose statistics come by ranges, its dialogues one by one by a workgroup per 128 keys (and their blocks joined, or merged in the second pass): another order of the
    sums would move the line at which a head's selection stops."""
    Hq, Hkv, w = 32, 8, 40
    print(f"batch and dialogues B={B} n={n} d={d} explicit={explicit}", flush=True)
    q, k, v = inputs.make_plain(B, Hq, Hkv, n, w, d, dtype="bf16", seed=n + B, q_scale=1.5)
    pos = np.sort(np.random.default_rng(n).choice(n, size=w, replace=False)).astype(np.int64) if explicit else None
    batch, one = (binding.score_route(binding.make_shape(b, Hq, Hkv, d, n, w, w, "bf16"), int(explicit), explicit) for b in (B, 1))
    assert batch["ranges"] > 1 and one["ranges"] == 0 and batch["joins"] == joins and one["joins"] != explicit and batch["folds"] == (n <= 2048)
    got = host(Pipeline(q, k, v, w, "bf16").score(q_pos=pos))
    for b in range(B):
        alone = host(Pipeline(q[b:b + 1], k[b:b + 1], v[b:b + 1], w, "bf16").score(q_pos=pos))
        for name in alone:
            np.testing.assert_array_equal(got[name].reshape(B, -1)[b], alone[name].reshape(-1), err_msg=name)


@pytest.mark.parametrize("Hq,Hkv,n,w,d,joins", [(8, 8, 25600, 8, 64, False), (8, 8, 25601, 8, 64, False), (4, 1, 4096, 128, 128, True), (8, 2, 2049, 1, 64, True), (4, 2, 129, 128, 64, True), (12, 4, 6000, 97, 128, True),
                                          (4, 4, 16384, 8, 64, True), (4, 4, 16385, 8, 64, False), (16, 16, 12800, 8, 64, True), (16, 16, 12801, 8, 64, False), (8, 2, 8193, 64, 128, True)])
def test_key_blocks_that_join_their_results(Hq, Hkv, n, w, d, joins):
    """Up to 1600 workgroups and 16384 keys, and one row of blocks or one key more; several groups of blocks, one, a block of one
    key; shares of the total of 1024 and of 2048 keys; no shared diagonals.  Again and again on one context: the same bits, whoever comes last."""
    print(f"joined blocks Hq={Hq} Hkv={Hkv} n={n} w={w} d={d}", flush=True)
    assert binding.score_route(binding.make_shape(1, Hq, Hkv, d, n, w, w, "bf16"), 0)["joins"] == joins
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
def test_retention_of_short_caches(B, Hq, Hkv, n, n_obs, d, budget):
    """Statistics by a workgroup per 128 keys, merged by the second pass.  Kept entries against float64 scores: the same, up to entries within 1e-3 of the threshold."""
    print(f"retention B={B} Hq={Hq} n={n} n_obs={n_obs} d={d}", flush=True)
    route = binding.score_route(binding.make_shape(B, Hq, Hkv, d, n, 1, n_obs, "bf16"), 2)
    assert route["ranges"] == 0 and route["folds"] and not route["streams"]
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


@pytest.mark.parametrize("B,Hq,Hkv,n,n_obs,d,ranges,chunks,streams", [
    (4, 8, 8, 12225, 32, 128, 24, 4, True), (2, 32, 8, 12287, 16, 64, 48, 4, True), (1, 40, 8, 9793, 32, 128, 48, 4, False), (1, 64, 8, 6143, 32, 64, 48, 4, False),
    (4, 64, 8, 12417, 32, 128, 24, 8, False), (3, 64, 8, 3998, 16, 128, 32, 4, True), (1, 4, 1, 196671, 16, 64, 256, 4, True), (2, 6, 2, 70017, 20, 128, 128, 4, True)])
@pytest.mark.parametrize("rising", [False, True])
def test_retention_over_ranges(B, Hq, Hkv, n, n_obs, d, ranges, chunks, streams, rising):
    """Statistics by ranges of keys: one chunk of rows and two (two waves share one), five for workgroups of four (the second has one), eight for workgroups of four and of eight,
    ranges of one tile, 256 ranges of one KV head; the second pass with all rows in LDS, and without.  `rising`: logits that climb by 2^65 (d = 128) or 2^92 every 288 keys, so that a
    range's reference moves many times."""
    print(f"retention ranges B={B} Hq={Hq} Hkv={Hkv} n={n} n_obs={n_obs} d={d} rising={rising}", flush=True)
    shape, budget = binding.make_shape(B, Hq, Hkv, d, n, 1, n_obs, "bf16"), 300
    route = binding.score_route(shape, 2)
    assert (route["ranges"], route["chunks"], route["streams"]) == (ranges, chunks, streams) and not route["folds"]
    if n == 3998:
        assert 64 in np.diff(route["begins"])              # a range of one tile
    q, k, v = inputs.make_plain(B, Hq, Hkv, n, n_obs, d, dtype="bf16", seed=n, q_scale=1.5)
    if rising:
        q[..., 0], k[..., 0] = 16.0, 4.0 * (np.arange(n) // 32 % 9)
    dev = lambda x: torch.from_numpy(x).cuda().to(torch.bfloat16)
    qd, kd = dev(q), dev(k)
    idx, cnt = torch.empty(B, Hkv, budget, dtype=torch.int32, device="cuda"), torch.empty(B, Hkv, dtype=torch.int32, device="cuda")
    score, ctx = torch.empty(B, Hkv, n, device="cuda"), binding.Context(shape, budget)
    ctx.ls_kv_compress(shape, budget, qd, kd, None, idx, cnt, None, None)
    ctx.debug_compress_score(shape, score)
    G, hidden = Hq // Hkv, torch.arange(n, device="cuda")[None, :] > torch.arange(n - n_obs, n, device="cuda")[:, None]
    for b in range(B):
        for g in range(Hkv):
            want, keys = torch.zeros(n, device="cuda", dtype=torch.float64), kd[b, g].double().T.contiguous()
            for h in range(g * G, g * G + G):
                want += torch.softmax(((qd[b, h].double() @ keys) / math.sqrt(d)).masked_fill(hidden, -math.inf), dim=-1).sum(0)
            want = want.cpu().numpy()
            np.testing.assert_allclose(score[b, g].cpu().numpy(), want, rtol=1e-3, atol=1e-6 * n_obs * G)        # as for ls_score, whose sums are of n_obs rows
            assert cnt[b, g].item() == budget
            threshold = np.sort(want)[-budget]
            for i in set(np.argsort(-want, kind="stable")[:budget]).symmetric_difference(idx[b, g].tolist()):
                assert abs(want[i] - threshold) <= 1e-3 * threshold


@pytest.mark.parametrize("B,Hq,Hkv,n,w,d", [(1, 64, 8, 6200, 16, 128), (4, 32, 8, 6300, 32, 64), (2, 48, 8, 8100, 16, 64)])
def test_retention_sums_chunk_by_chunk(B, Hq, Hkv, n, w, d):
    """Rows of zeros: a key's score is the sum of 1 / L over the rows, L whole numbers, to the last bit as 32 rows at a time are added (eight by eight and four of them in a
    lane, then the halves): through all rows at once the rounding errors are those of a sum four times as long."""
    print(f"chunk by chunk B={B} Hq={Hq} n={n} w={w} d={d}", flush=True)
    shape, budget = binding.make_shape(B, Hq, Hkv, d, n, 1, w, "bf16"), 100
    assert binding.score_route(shape, 2)["streams"]
    q, k = torch.zeros(B, Hq, w, d, device="cuda", dtype=torch.bfloat16), torch.randn(B, Hkv, n, d, device="cuda").to(torch.bfloat16)
    idx, cnt = torch.empty(B, Hkv, budget, dtype=torch.int32, device="cuda"), torch.empty(B, Hkv, dtype=torch.int32, device="cuda")
    score, ctx = torch.empty(B, Hkv, n, device="cuda"), binding.Context(shape, budget)
    ctx.ls_kv_compress(shape, budget, q, k, None, idx, cnt, None, None)
    ctx.debug_compress_score(shape, score)
    rows, one = Hq // Hkv * w, np.float32(1)
    il = [one / np.float32(n - w + r % w + 1) for r in range(rows)]
    halves, through = [np.float32(0)] * 2, [np.float32(0)] * 2
    for c in range(0, rows, 32):
        for g in range(2):
            ps = np.float32(0)
            for r in range(16):                            # register r of a lane of half g
                x = il[c + 8 * (r // 4) + 4 * g + r % 4]
                ps, through[g] = ps + x, through[g] + x
            halves[g] = halves[g] + ps
    want = halves[0] + halves[1]
    assert want != through[0] + through[1]                 # (these shapes tell the two orders apart)
    assert (score[..., :n - w - 127] == float(want)).all()
