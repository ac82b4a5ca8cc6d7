"""How ls_sparse_prefill shares its work among the workgroups: in pieces of about equal work, and by work queues where the turn is larger.  One call over a batch
that lies beyond the line is compared with calls over its parts, which lie below: the same cells summed in another order of tiles and parts."""
import numpy as np
import pytest
import torch

from paper_2507_13681_amd import binding, inputs


def _in_pieces(B, Hq, Hkv, n, n_hat, d, dtype="bf16"):
    return binding.prefill_in_pieces(binding.make_shape(B, Hq, Hkv, d, n, n_hat, 1, dtype))


# tiles of 64 keys as if every head were dense, half at d = 64; items; of a turn that is all of the context, the tiles that it sees
@pytest.mark.parametrize("B,Hq,Hkv,n,n_hat,d,dtype,pieces", [
    (1, 4, 1, 131072, 4096, 128, "bf16", True), (1, 4, 1, 131072, 4097, 128, "bf16", False),                                                   # 262144 tiles, few items
    (4, 32, 8, 4096, 4096, 128, "bf16", True), (4, 32, 8, 8192, 4096, 128, "bf16", False), (2, 64, 8, 12288, 2560, 128, "bf16", True), (2, 64, 8, 12288, 2561, 128, "bf16", False),      # many
    (1, 11, 1, 47616, 8192, 128, "bf16", True), (1, 11, 1, 47616, 8064, 128, "bf16", False),                                                   # 704 items, 693
    (1, 32, 8, 32768, 4096, 128, "bf16", True), (1, 32, 8, 32768, 4097, 128, "bf16", False),                                                   # 524288 tiles
    (1, 4, 1, 32768, 32768, 128, "f32", True), (1, 4, 1, 32832, 32832, 128, "f32", False),
    (1, 64, 8, 115957, 547, 64, "bf16", True), (1, 32, 8, 131072, 2048, 64, "bf16", True), (1, 32, 8, 131072, 2049, 64, "bf16", False),
    (1, 64, 8, 12800, 10240, 64, "bf16", True), (1, 64, 8, 12800, 10241, 64, "bf16", False),                                                   # 5120 items
    (1, 64, 8, 6000, 6000, 128, "bf16", True), (1, 32, 8, 10000, 10000, 128, "bf16", True), (1, 32, 8, 12000, 12000, 128, "bf16", False),      # 204800 seen
    (2, 64, 8, 8192, 8192, 64, "bf16", False), (1, 32, 8, 32768, 10923, 64, "bf16", False)])
def test_where_the_line_lies(B, Hq, Hkv, n, n_hat, d, dtype, pieces):
    assert _in_pieces(B, Hq, Hkv, n, n_hat, d, dtype) == pieces


def _lists(rng, B, H, n):
    """Heads of very unequal work: every diagonal; none; a few; the newest alone with many columns; random ones."""
    v, s = [], []
    for i in range(B * H):
        kind = i % 5
        s.append(np.arange(n) if kind == 0 else np.zeros(0, int) if kind == 1 else np.unique(rng.integers(0, n, 3)) if kind == 2
                 else np.zeros(1, int) if kind == 3 else np.flatnonzero(rng.random(n) < rng.choice([0.01, 0.2])))
        v.append(np.zeros(0, int) if kind == 0 and i % 2 else np.flatnonzero(rng.random(n) < (0.3 if kind == 3 else 0.02)))
    def pack(x):
        out = np.zeros((B * H, n), np.int32)
        for i, e in enumerate(x):
            out[i, :len(e)] = e
        return out.reshape(B, H, n), np.array([len(e) for e in x], np.int32).reshape(B, H)
    vi, vc = pack(v)
    si, sc = pack(s)
    return vi, vc, si, sc


# the turn is the end of the context or all of it; n and n_hat have no relation to any tile size
@pytest.mark.gpu
@pytest.mark.parametrize("B,Hq,Hkv,n,n_hat,d,dtype", [
    (22, 16, 4, 3999, 3000, 128, "bf16"), (5, 4, 2, 21001, 21001, 64, "bf16"), (5, 4, 1, 20001, 12000, 128, "bf16"),
    (5, 4, 1, 21001, 21001, 64, "f32"), (5, 4, 2, 20003, 12001, 128, "f32")])
def test_queues_and_pieces_agree(B, Hq, Hkv, n, n_hat, d, dtype):
    from tests.gpu_util import Pipeline, dev_lists
    print(f"queues and pieces B={B} Hq={Hq} n={n} n_hat={n_hat} d={d} {dtype}", flush=True)
    cut = max(b for b in range(1, B) if _in_pieces(b, Hq, Hkv, n, n_hat, d, dtype))
    assert not _in_pieces(B, Hq, Hkv, n, n_hat, d, dtype)
    q, k, v = inputs.make_plain(B, Hq, Hkv, n, n_hat, d, dtype=dtype, seed=n, q_scale=1.5)
    lists = _lists(np.random.default_rng(n), B, Hq, n)
    out, lse = Pipeline(q, k, v, 1, dtype).prefill(dev_lists(*lists), sentinel=True)
    # In bf16 each side rounds every probability (2^-9 relative, against references that differ) and the result: 4 * 2^-9 of
    # the largest value.  fp32: sums of at most n terms in another order, sqrt(n) * 2^-24 * 8 and room for exp's argument.
    tol = (4 * 2.0 ** -9 if dtype == "bf16" else 1e-5) * float(np.abs(v).max())
    for b in (slice(b0, b0 + cut) for b0 in range(0, B, cut)):
        part, plse = Pipeline(q[b], k[b], v[b], 1, dtype).prefill(dev_lists(*(x[b] for x in lists)), sentinel=True)
        assert not torch.isnan(out[b]).any() and not torch.isnan(part).any()
        assert (out[b].float() - part.float()).abs().max().item() <= tol
        some = torch.isfinite(plse)
        assert torch.equal(torch.isfinite(lse[b]), some)
        assert (lse[b][some] - plse[some]).abs().max().item() <= 1e-4


@pytest.mark.gpu
@pytest.mark.parametrize("B,Hq,Hkv,n,n_hat,d", [(1, 1, 1, 5000, 100, 128), (1, 4, 2, 3001, 3001, 64), (5, 4, 1, 20001, 12000, 128)])
def test_items_are_shared_as_the_device_says(B, Hq, Hkv, n, n_hat, d):
    """Pieces and queues as the kernels left them: every item once, items of the one dense head cut; no cut without room for parts."""
    from tests.gpu_util import Pipeline, dev_lists
    print(f"items as shared B={B} Hq={Hq} n={n} n_hat={n_hat} d={d}", flush=True)
    q, k, v = inputs.make_plain(B, Hq, Hkv, n, n_hat, d, dtype="bf16", seed=n)
    every = np.broadcast_to(np.arange(n, dtype=np.int32), (B, Hq, n)).copy()
    lists = np.zeros((B, Hq, n), np.int32), np.zeros((B, Hq), np.int32), every, np.full((B, Hq), 5, np.int32)
    lists[3][0, 0] = n
    pipe = Pipeline(q, k, v, 1, "bf16")
    blocks = (n - (n - n_hat) // 128 * 128 + 127) // 128
    want = np.sort([h << 16 | b for h in range(B * Hq) for b in range(blocks)])
    tables = B * Hq * ((n + 31) // 32 * 4 + 64 + (n // 64 + 5) * 3) + B * Hq * blocks * 20 + 4096
    for ctx, cut in ((pipe.ctx, True), (binding.Context(workspace=tables), False)):
        pipe.ctx = ctx
        pipe.prefill(dev_lists(*lists), sentinel=True)
        queues, nqb, cuts = ctx.debug_prefill_queues(pipe.shape)
        assert nqb == blocks and (cuts > 0) == cut, cuts
        np.testing.assert_array_equal(np.sort(np.concatenate(queues)), want)


@pytest.mark.gpu
@pytest.mark.parametrize("Hq,Hkv,n,n_hat,d", [(16, 4, 3001, 3001, 64), (8, 2, 4096, 4096, 128), (32, 8, 5003, 300, 128), (32, 8, 4099, 4099, 128),
                                                (32, 8, 131001, 1100, 64), (20, 4, 130001, 3300, 64)])      # few long items; queues whatever the room: beyond the line
def test_room_for_some_parts(Hq, Hkv, n, n_hat, d):
    """A workspace with room for some of the parts: items are still cut, in fewer pieces or by the queues, to the same result."""
    from tests.gpu_util import Pipeline, dev_lists
    print(f"room for some parts Hq={Hq} n={n} n_hat={n_hat} d={d}", flush=True)
    q, k, v = inputs.make_plain(1, Hq, Hkv, n, n_hat, d, dtype="bf16", seed=n, q_scale=1.5)
    lists = dev_lists(*_lists(np.random.default_rng(n), 1, Hq, n))
    pipe = Pipeline(q, k, v, 1, "bf16")
    ref, rlse = pipe.prefill(lists, sentinel=True)
    items = Hq * ((n - (n - n_hat) // 128 * 128 + 127) // 128)
    places = 512 if d == 128 else 768
    slots, fewest = places - 1 + min(items, places - 1), 0.3          # fewest: share of them with which items are still cut
    if not _in_pieces(1, Hq, Hkv, n, n_hat, d):                           # (the longest part grows by half until all parts fit)
        slots, fewest = 1024, 0.5
    tables = Hq * ((n + 31) // 32 * 4 + 64 + (n // 64 + 5) * 3) + items * 20 + 16384
    tol = 4 * 2.0 ** -9 * float(np.abs(v).max())                      # as between queues and pieces
    for share in (1.0, 0.99, 0.9, 0.7, 0.667, 0.5, 0.3, 0.1, 0.02):
        ctx = pipe.ctx = binding.Context(workspace=tables + int(share * slots) * (128 * d * 4 + 1024 + 24))
        ctx.profile_enable(True)
        out, lse = pipe.prefill(lists, sentinel=True)
        torch.cuda.synchronize()
        assert ctx.profile_prefill_kernel_ms()[1] == 1
        queues, _, cuts = ctx.debug_prefill_queues(pipe.shape)
        assert (cuts > 0 or share < fewest) and len(np.unique(np.concatenate(queues))) == sum(map(len, queues)) == items, (share, cuts)
        assert not torch.isnan(out).any()
        assert (out.float() - ref.float()).abs().max().item() <= tol
        some = torch.isfinite(rlse)
        assert torch.equal(torch.isfinite(lse), some)
        assert (lse[some] - rlse[some]).abs().max().item() <= 1e-4


# row blocks a head, and heads, at which pieces and items come out in each other (512 and 768 pieces) or just do not
@pytest.mark.gpu
@pytest.mark.parametrize("B,Hq,Hkv,n,n_hat,d", [(2, 32, 8, 6001, 3, 128), (4, 64, 8, 1200, 130, 128), (2, 64, 8, 3001, 5, 64), (3, 64, 8, 2999, 129, 64),
                                               (2, 33, 3, 3001, 1, 128), (4, 64, 8, 1200, 300, 128)])
def test_short_turns_of_many_heads(B, Hq, Hkv, n, n_hat, d):
    """Against the same call without room for parts: queues of whole items."""
    from tests.gpu_util import Pipeline, dev_lists
    print(f"short turns of many heads B={B} Hq={Hq} n={n} n_hat={n_hat} d={d}", flush=True)
    q, k, v = inputs.make_plain(B, Hq, Hkv, n, n_hat, d, dtype="bf16", seed=n, q_scale=1.5)
    lists = dev_lists(*_lists(np.random.default_rng(n), B, Hq, n))
    pipe = Pipeline(q, k, v, 1, "bf16")
    out, lse = pipe.prefill(lists, sentinel=True)
    queues, blocks, _ = pipe.ctx.debug_prefill_queues(pipe.shape)
    items = B * Hq * blocks
    assert len(np.unique(np.concatenate(queues))) == sum(map(len, queues)) == items
    pipe.ctx = binding.Context(workspace=B * Hq * ((n + 31) // 32 * 4 + 64 + (n // 64 + 5) * 3) + items * 20 + 4096)
    ref, rlse = pipe.prefill(lists, sentinel=True)
    assert pipe.ctx.debug_prefill_queues(pipe.shape)[2] == 0
    assert not torch.isnan(out).any()
    tol = 4 * 2.0 ** -9 * float(np.abs(v).max())                      # as between queues and pieces
    assert (out.float() - ref.float()).abs().max().item() <= tol
    some = torch.isfinite(rlse)
    assert torch.equal(torch.isfinite(lse), some)
    assert (lse[some] - rlse[some]).abs().max().item() <= 1e-4
