"""ls_sparse_prefill where a row's logits rise along the keys, so that the softmax reference has to move all the time, or fall.  Against the
same attention in 64 bits."""
import math

import pytest
import torch

from paper_2507_13681_amd import binding

SLOPES = [0.0, 1.0, 2.0, 4.0, 16.0, 32.0, 80.0, -8.0]      # of the query heads: base-2 logits in 64 keys


@pytest.mark.gpu
@pytest.mark.parametrize("kind", ["dense", "band", "band and columns", "columns"])
@pytest.mark.parametrize("B,n,n_hat,d", [(1, 6000, 300, 128), (1, 3001, 3001, 64), (1, 5000, 1, 64), (6, 24000, 9000, 128)])      # the last: work queues
def test_rising_logits(B, n, n_hat, d, kind):
    print(f"rising logits B={B} n={n} n_hat={n_hat} d={d} {kind}", flush=True)
    Hq, Hkv = len(SLOPES), 2
    g = torch.Generator(device="cuda").manual_seed(n + d)
    q, k, v = (torch.randn(B, h, m, d, device="cuda", generator=g) for h, m in ((Hq, n_hat), (Hkv, n), (Hkv, n)))
    pos = torch.arange(n, device="cuda")
    per = torch.tensor(SLOPES, device="cuda").view(1, Hq, 1) / 64 * math.log(2) * math.sqrt(d)
    q[..., 0], q[..., 1] = 128 * per, per                  # the position in two coordinates of K, exact in bf16
    k[..., 0], k[..., 1] = (pos // 128 - n // 256).float(), (pos % 128).float()
    q, k, v = q.bfloat16(), k.bfloat16(), v.bfloat16()
    diagonals = {"dense": n, "columns": 0}.get(kind, 1024)
    cols = torch.randperm(n, device="cuda", generator=g)[:300].sort()[0].int() if "columns" in kind else torch.zeros(0, dtype=torch.int32, device="cuda")
    v_idx, s_idx = torch.zeros(B, Hq, n, dtype=torch.int32, device="cuda"), torch.zeros(B, Hq, n, dtype=torch.int32, device="cuda")
    v_idx[..., :len(cols)] = cols
    s_idx[..., :diagonals] = pos[:diagonals].int()
    v_cnt, s_cnt = (torch.full((B, Hq), c, dtype=torch.int32, device="cuda") for c in (len(cols), diagonals))
    shape = binding.make_shape(B, Hq, Hkv, d, n, n_hat, 1, "bf16")
    ctx = binding.Context(shape)
    out, lse = torch.full_like(q, float("nan")), torch.full((B, Hq, n_hat), float("nan"), device="cuda")
    ctx.ls_sparse_prefill(shape, q, k, v, v_idx, v_cnt, s_idx, s_cnt, out, lse)
    assert ctx.ls_poll_status() == 0 and not torch.isnan(out).any() and not torch.isnan(lse).any()
    rows = torch.arange(n_hat - 1, -1, -max(1, n_hat // 150), device="cuda")
    p = n - n_hat + rows
    off = p[:, None] - pos[None]
    picked = torch.zeros(n, dtype=torch.bool, device="cuda")
    picked[cols.long()] = True
    allowed = (off >= 0) & ((off < diagonals) | picked[None])
    for b in (0, B - 1):
        for h in range(Hq):
            kk, vv = k[b, h // (Hq // Hkv)].double(), v[b, h // (Hq // Hkv)].double()
            x = (q[b, h, rows].double() @ kk.T.contiguous() / math.sqrt(d)).masked_fill(~allowed, -math.inf)
            ref_lse = torch.logsumexp(x, -1)
            some = torch.isfinite(ref_lse)
            ref = torch.softmax(x[some], -1) @ vv
            got = out[b, h, rows].double()
            assert (got[~some] == 0).all() and torch.equal(torch.isfinite(lse[b, h, rows]), some)
            # probabilities and the result are rounded to bf16, 2^-9 each at most
            assert (got[some] - ref).norm() <= 2.0 ** -8 * ref.norm(), (h, ((got[some] - ref).norm() / ref.norm()).item())
            # fp32 logits: some roundings of the largest (sums of d terms of that size, and the reference's own)
            top = (q[b, h, rows].double().abs() @ kk.abs().T.contiguous()).max().item() / math.sqrt(d)
            assert (lse[b, h, rows][some].double() - ref_lse[some]).abs().max().item() <= 8 * 2.0 ** -24 * top + 1e-5
