"""What the library is timed on: one attention layer's work in a multi-turn dialogue, through the public calls.

Four kinds of case, each a stage of a dialogue as a serving program drives it (binding.Context, one context kept):

  turn      a new turn arrives: ls_score -> ls_select -> ls_sparse_prefill over the grown context.  `sampled` scores
            random rows of the turn instead of its last ones; `carried` adds the lines kept from earlier turns with
            ls_merge_lines before the attention.
  select    the selection alone from given line weights; `exact` counts overlaps cell by cell (ls_select_exact),
            `accounted` asks for the accounted mass as well.
  compress  decode-time retention of one cache: ls_kv_compress, with the kept rows copied out.
  decode    one generated token: ls_decode_attend over the retained rows and the tokens since.

Inputs have the structure of paper_2507_13681_amd.inputs (sinks, heavy columns per query head, a local band, a relevant
span), drawn on the GPU because they are large.
"""
import math

import numpy as np
import torch

from paper_2507_13681_amd import binding


def _turn(name, **kw):
    c = dict(name=name, kind="turn", B=1, Hq=32, Hkv=8, d=128, n=32768, n_hat=10923, w=64, dtype="bf16", alpha=0.95,
             sampled=False, carried=False)
    c.update(kw)
    return c


def listed():
    return [
        # the third turn of a 32k dialogue, 8B-class heads: the workload bench.py reports
        _turn("turn_32k"),
        # the opening turn of a dialogue: every position is a new row
        _turn("first_turn_8k", n=8192, n_hat=8192),
        # the longest context: the last of eight turns at 131072 tokens, a window of 128 rows
        _turn("turn_131k", n=131072, n_hat=16384, w=128),
        # four dialogues at once, 64 query heads on 8 KV heads (70B-class)
        _turn("turn_16k_b4", B=4, Hq=64, n=16384, n_hat=5462),
        # a one-line follow-up question deep in a dialogue: few new rows, odd lengths
        _turn("follow_up", n=12347, n_hat=61, w=61, alpha=0.90),
        # a short prompt of a small fp32 model
        _turn("turn_1k_fp32", Hq=4, Hkv=1, d=64, n=1024, n_hat=256, w=32, dtype="f32", alpha=0.90),
        # d = 64 heads, rows scored at random positions of the turn, lines of earlier turns carried along; ragged
        _turn("carried_d64", Hq=16, Hkv=4, d=64, n=5003, n_hat=1777, w=48, sampled=True, carried=True),
        # the selection by itself, as when the line weights are kept and another coverage target is asked for
        dict(name="select_32k", kind="select", B=1, Hq=32, Hkv=8, d=128, n=32768, n_hat=10923, w=64, alpha=0.95,
             exact=False, accounted=False),
        # the opt-in selection with exact overlaps
        dict(name="select_exact_8k", kind="select", B=1, Hq=32, Hkv=8, d=128, n=8192, n_hat=4096, w=64, alpha=0.95,
             exact=True, accounted=True),
        # retention while decoding a batch: the last 16 tokens' queries rank a 16k cache, 2048 rows are kept
        dict(name="compress_16k_b4", kind="compress", B=4, Hq=64, Hkv=8, d=128, n=16384, n_obs=16, budget=2048, gather=True),
        # one token for that batch over the retained rows
        dict(name="decode_b4", kind="decode", B=4, Hq=64, Hkv=8, d=128, cap=2048, T=16, ragged=False),
        # one token of a single dialogue with a small retained set: the smallest call there is
        dict(name="decode_b1", kind="decode", B=1, Hq=32, Hkv=8, d=128, cap=512, T=7, ragged=True),
    ]


HEADS = [(32, 8), (64, 8), (16, 4), (8, 2), (8, 8), (4, 1)]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["turn", "turn", "turn", "select", "compress", "decode", "decode"])
    hq, hkv = rng.choice(HEADS)
    B, d = rng.choice([1, 1, 2, 4]), rng.choice([64, 128, 128])
    if kind == "turn":
        f32 = rng.random() < 0.2
        if f32:
            B, hq, hkv, d = 1, *rng.choice([(4, 1), (8, 2)]), 64
        n = _log(rng, 256, 4096 if f32 else 131072)
        n_hat = _log(rng, 16, n)
        # no more than about an eighth of turn_131k's causal cells: a drawn context may come out much denser
        while B * hq * n_hat * (n - n_hat // 2) > 8e9:
            n_hat = max(16, n_hat * 3 // 4)
        w = min(n_hat, rng.choice([32, 64, 64, 128, rng.randint(17, 127)]))
        return dict(kind=kind, B=B, Hq=hq, Hkv=hkv, d=d, n=n, n_hat=n_hat, w=w, dtype="f32" if f32 else "bf16",
                    alpha=rng.choice([0.90, 0.95, 0.95, 0.98]), sampled=not f32 and rng.random() < 0.25, carried=rng.random() < 0.25)
    if kind == "select":
        exact = rng.random() < 0.4
        n = _log(rng, 256, 8192 if exact else 65536)
        return dict(kind=kind, B=1, Hq=hq, Hkv=hkv, d=d, n=n, n_hat=_log(rng, 64, n), w=rng.choice([32, 64, rng.randint(17, 127)]),
                    alpha=rng.choice([0.90, 0.95]), exact=exact, accounted=rng.random() < 0.3)
    if kind == "compress":
        n = _log(rng, 512, 131072 // B)
        return dict(kind=kind, B=B, Hq=hq, Hkv=hkv, d=d, n=n, n_obs=rng.choice([8, 16, 16, 32]),
                    budget=min(n, _log(rng, 128, 8192)), gather=rng.random() < 0.7)
    return dict(kind=kind, B=rng.choice([1, 2, 4, 8]), Hq=hq, Hkv=hkv, d=d, cap=_log(rng, 64, 16384), T=rng.randint(0, 64),
                ragged=rng.random() < 0.5)


# ---- inputs ------------------------------------------------------------------------------------------

def _structured(case, n_hat, seed, dtype):
    """q [B,Hq,n_hat,d], k, v [B,Hkv,n,d] with the planted structure of inputs.make_inputs."""
    B, Hq, Hkv, d, n = case["B"], case["Hq"], case["Hkv"], case["d"], case["n"]
    G, m, sq = Hq // Hkv, max(d // 4, 8), math.sqrt(d)
    host = np.random.Generator(np.random.PCG64(seed))
    g = torch.Generator(device="cuda").manual_seed(int(host.integers(1 << 40)))
    rnd = lambda *s: torch.randn(*s, device="cuda", generator=g)
    tau = max(3.0, 3.8 + 0.2 * (math.log2(n) - 15))      # 3.0 at 1k, 3.4 at 8k, 3.8 at 32k, 4.2 at 131k
    band, beta, rho = min(256, max(8, n // 32)), 6.0, 0.5
    gk = math.sqrt(beta / m)
    span = min(1024, n // 16) if n >= 4096 else 0
    heavy_lo, heavy_hi = max(2, min(16, n // 128)), max(3, min(256, n // 64))
    cols_below = max(n - n_hat, n // 2)                  # heavy columns lie in the history
    q = torch.empty(B, Hq, n_hat, d, dtype=dtype, device="cuda")
    k = torch.empty(B, Hkv, n, d, dtype=dtype, device="cuda")
    v = rnd(B, Hkv, n, d).to(dtype)
    a = math.exp(-1.0 / band)
    for b in range(B):
        for j in range(Hkv):
            E = torch.from_numpy(np.linalg.qr(host.standard_normal((d, 2 + G + m)))[0].astype(np.float32)).cuda()
            u, u_span, Uh, Ep = E[:, 0], E[:, 1], E[:, 2:2 + G], E[:, 2 + G:]
            r = rnd(n, m)                                # AR(1) path: 1/(1 - aL) = (1 + aL)(1 + a^2 L^2)(1 + a^4 L^4)...
            r[1:] *= math.sqrt(1.0 - a * a)
            s = 1
            while s < n:
                r[s:] += (a ** s) * r[:-s].clone()
                s *= 2
            K = rnd(n, d)
            K -= (K @ E) @ E.T.contiguous()
            K += gk * (r @ Ep.T.contiguous())
            K[:4] += 3.0 * u
            if span:
                lo = int(host.integers(0, n - span))
                K[lo:lo + span] += 2.0 * u_span
            for gq in range(G):
                cnt = int(host.integers(heavy_lo, heavy_hi + 1))
                cols = torch.from_numpy(np.sort(4 + host.choice(cols_below - 4, size=cnt, replace=False))).cuda()
                K[cols] += 2.0 * Uh[:, gq]
                Q = rho * rnd(n_hat, d) + (sq * tau) * (u + Uh[:, gq]) + (sq * gk) * (r[n - n_hat:] @ Ep.T.contiguous())
                if span:
                    qb = min(64, n_hat)
                    at = [0, (n_hat - qb) // 2, n_hat - qb][(j * G + gq) % 3]
                    Q[at:at + qb] += (sq * tau) * u_span
                q[b, j * G + gq] = Q.to(dtype)
            k[b, j] = K.to(dtype)
    return q, k, v


def _window(case, q_win, k):
    """The scored rows' causal softmax and its line sums and maxima, as a program that kept them holds them."""
    B, Hq, Hkv, d, n, w = case["B"], case["Hq"], case["Hkv"], case["d"], case["n"], case["w"]
    G = Hq // Hkv
    A = torch.zeros(B, Hq, w, n, device="cuda")
    rows = torch.arange(n - w, n, device="cuda")
    hidden = torch.arange(n, device="cuda")[None, :] > rows[:, None]
    for b in range(B):
        for h in range(Hq):
            x = (q_win[b, h].float() @ k[b, h // G].float().T.contiguous()) / math.sqrt(d)
            A[b, h] = torch.softmax(x.masked_fill(hidden, -math.inf), dim=-1)
    slash, smax = torch.zeros(B, Hq, n, device="cuda"), torch.zeros(B, Hq, n, device="cuda")
    for t in range(w):
        p = n - w + t
        diag = A[:, :, t, :p + 1].flip(-1)
        slash[:, :, :p + 1] += diag
        smax[:, :, :p + 1] = torch.maximum(smax[:, :, :p + 1], diag)
    vert = A.sum(2)
    return dict(a_win=A, vert=vert, slash=slash, vmax=A.amax(2), smax=smax, total=vert.sum(-1))


def _lists(case, host, cap, lo, hi):
    """Ascending index lists of a few hundred lines per head: what an earlier turn left behind."""
    B, Hq, n = case["B"], case["Hq"], case["n"]
    idx, cnt = np.zeros((B, Hq, cap), np.int32), np.zeros((B, Hq), np.int32)
    for b in range(B):
        for h in range(Hq):
            x = np.unique(np.concatenate([np.arange(lo), host.integers(0, n, hi)]))[:cap]
            idx[b, h, :len(x)], cnt[b, h] = x, len(x)
    return torch.from_numpy(idx).cuda(), torch.from_numpy(cnt).cuda()


def _select_outputs(shape, accounted=False):
    """ls_select's outputs; entries past a list's count stay what they are here."""
    sel = binding.alloc_select(shape, accounted=accounted)
    for t in sel.values():
        if t is not None:
            t.fill_(-1)
    return sel


def prepare(case, seed):
    c, kind = case, case["kind"]
    B, Hq, Hkv, d = c["B"], c["Hq"], c["Hkv"], c["d"]
    host = np.random.Generator(np.random.PCG64([seed, 17]))
    s = dict(case=c)
    if kind == "turn":
        dt = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32
        n, n_hat, w = c["n"], c["n_hat"], c["w"]
        s["q"], s["k"], s["v"] = _structured(c, n_hat, seed, dt)
        s["shape"] = binding.make_shape(B, Hq, Hkv, d, n, n_hat, w, c["dtype"])
        s["q_pos"] = None
        s["q_win"] = s["q"][:, :, -w:].contiguous()
        if c["sampled"]:
            at = torch.from_numpy(np.sort(host.choice(n_hat, size=w, replace=False)).astype(np.int64)).cuda()
            s["q_win"], s["q_pos"] = s["q"][:, :, at].contiguous(), n - n_hat + at
        s["score"] = binding.alloc_score(s["shape"])
        s["sel"] = _select_outputs(s["shape"])
        if c["carried"]:
            cap = min(n, 512)
            vi, vc = _lists(c, host, cap, 4, min(200, n // 8))
            si, sc = _lists(c, host, cap, min(128, n // 8), min(100, n // 8))
            s["old"] = dict(v_idx=vi, v_cnt=vc, s_idx=si, s_cnt=sc)
            s["merged"] = _select_outputs(s["shape"])
        s["out"] = torch.empty_like(s["q"])
        s["lse"] = torch.empty(B, Hq, n_hat, device="cuda")
        s["ctx"] = binding.Context(s["shape"])
    elif kind == "select":
        q, k, _ = _structured(c, c["n_hat"], seed, torch.bfloat16)
        w = c["w"] = min(c["w"], c["n_hat"])
        s["shape"] = binding.make_shape(B, Hq, Hkv, d, c["n"], c["n_hat"], w, "bf16")
        s["score"] = _window(c, q[:, :, -w:], k)
        if not c["exact"]:
            del s["score"]["a_win"]
        s["sel"] = _select_outputs(s["shape"], c["accounted"])
        s["ctx"] = binding.Context(s["shape"])
    elif kind == "compress":
        q, s["k"], s["v"] = _structured(c, c["n_obs"], seed, torch.bfloat16)
        s["q_obs"] = q
        s["shape"] = binding.make_shape(B, Hq, Hkv, d, c["n"], 1, c["n_obs"], "bf16")
        s["keep_idx"] = torch.empty(B, Hkv, c["budget"], dtype=torch.int32, device="cuda")
        s["keep_cnt"] = torch.empty(B, Hkv, dtype=torch.int32, device="cuda")
        rows = (B, Hkv, c["budget"], d)
        s["k_out"] = torch.empty(rows, dtype=torch.bfloat16, device="cuda") if c["gather"] else None
        s["v_out"] = torch.empty(rows, dtype=torch.bfloat16, device="cuda") if c["gather"] else None
        s["ctx"] = binding.Context(s["shape"], c["budget"])
    else:
        g = torch.Generator(device="cuda").manual_seed(seed)
        rnd = lambda *z: torch.randn(*z, device="cuda", generator=g).to(torch.bfloat16)
        cap, T = c["cap"], c["T"]
        s["q"] = rnd(B, Hq, d)
        s["k_c"], s["v_c"] = rnd(B, Hkv, cap, d), rnd(B, Hkv, cap, d)
        s["k_t"], s["v_t"] = (rnd(B, Hkv, T, d), rnd(B, Hkv, T, d)) if T else (None, None)
        cnt = host.integers(cap // 2, cap + 1, (B, Hkv)) if c["ragged"] else np.full((B, Hkv), cap)
        s["cnt"] = torch.from_numpy(cnt.astype(np.int32)).cuda()
        s["out"] = torch.empty(B, Hq, d, dtype=torch.bfloat16, device="cuda")
        s["lse"] = torch.empty(B, Hq, device="cuda")
        s["shape"] = binding.make_shape(B, Hq, Hkv, d, cap + T, 1, 1, "bf16")
        s["ctx"] = binding.Context(workspace=binding.decode_workspace_bytes(s["shape"], cap, T))
    return s


def run(s):
    c, ctx, shape = s["case"], s["ctx"], s["shape"]
    if c["kind"] == "turn":
        sc, sel = s["score"], s["sel"]
        ctx.ls_score(shape, s["q_win"], s["k"], sc["vert"], sc["slash"], sc["vmax"], sc["smax"], sc["total"], s["q_pos"])
        ctx.ls_select(shape, c["alpha"], sc["vert"], sc["slash"], sc["vmax"], sc["smax"], sc["total"],
                      sel["v_idx"], sel["v_cnt"], sel["s_idx"], sel["s_cnt"], None)
        if c["carried"]:
            ctx.ls_merge_lines(shape, s["old"], sel, s["merged"])
            sel = s["merged"]
        ctx.ls_sparse_prefill(shape, s["q"], s["k"], s["v"], sel["v_idx"], sel["v_cnt"], sel["s_idx"], sel["s_cnt"],
                              s["out"], s["lse"])
        # the index lists only feed the attention; whether they are the right ones shows in `out`, and `select` has them exactly
        return dict(out=s["out"], lse=s["lse"], **sc)
    if c["kind"] == "select":
        sc, sel = s["score"], s["sel"]
        if c["exact"]:
            ctx.ls_select_exact(shape, c["alpha"], sc["a_win"], sc["vert"], sc["slash"], sc["total"],
                                sel["v_idx"], sel["v_cnt"], sel["s_idx"], sel["s_cnt"], sel["accounted"])
        else:
            ctx.ls_select(shape, c["alpha"], sc["vert"], sc["slash"], sc["vmax"], sc["smax"], sc["total"],
                          sel["v_idx"], sel["v_cnt"], sel["s_idx"], sel["s_cnt"], sel["accounted"])
        return sel
    if c["kind"] == "compress":
        ctx.ls_kv_compress(shape, c["budget"], s["q_obs"], s["k"], s["v"] if c["gather"] else None, s["keep_idx"],
                           s["keep_cnt"], s["k_out"], s["v_out"])
        return dict(keep_idx=s["keep_idx"], keep_cnt=s["keep_cnt"], k_out=s["k_out"], v_out=s["v_out"])
    ctx.ls_decode_attend(shape, s["q"], s["k_c"], s["v_c"], s["cnt"], s["k_t"], s["v_t"], s["out"], s["lse"])
    return dict(out=s["out"], lse=s["lse"])


# A selection of these inputs keeps about this share of the causal cells (the benchmark's workload: 0.207).
SHARE = 0.2


def work(case):
    c, kind = case, case["kind"]
    B, Hq, Hkv, d = c["B"], c["Hq"], c["Hkv"], c["d"]
    if kind == "turn":
        e, n, n_hat, w = (2 if c["dtype"] == "bf16" else 4), c["n"], c["n_hat"], c["w"]
        cells = B * Hq * (n_hat * (n - n_hat) + n_hat * (n_hat + 1) // 2)
        return dict(bytes=e * d * B * (2 * Hq * n_hat + Hq * w + 2 * Hkv * n) + 4 * B * Hq * (4 * n + n_hat),
                    flops=2.0 * d * B * Hq * w * n + SHARE * 4.0 * d * cells)
    if kind == "select":
        # the weights (and maxima, or the window matrix) in; of the lists about an eighth is written
        read = 2 + c["w"] if c["exact"] else 4
        return dict(bytes=4 * B * Hq * c["n"] * (read + 0.25), flops=0)
    if kind == "compress":
        kept = 4 * d * c["budget"] * 2 if c["gather"] else 0      # K and V rows in and out
        return dict(bytes=2 * d * B * (Hkv * c["n"] + Hq * c["n_obs"]) + B * Hkv * (4 * c["budget"] + kept),
                    flops=2.0 * d * B * Hq * c["n_obs"] * c["n"])
    L = (0.75 if c["ragged"] else 1.0) * c["cap"] + c["T"]
    return dict(bytes=4 * d * B * (Hkv * L + Hq), flops=4.0 * d * B * Hq * L)


def tolerance(case):
    if case["kind"] == "select":
        return "exact"                          # defined to the last bit: binary32 with single roundings, ties by index
    if case["kind"] == "compress":
        return {"rel": 1e-2, "differ": 0.01}    # two scores within rounding of each other may change places at the cut
    if case.get("dtype") == "f32":
        return {"rel": 1e-4}                    # fp32 throughout; the hardware's exp2
    return {"rel": 1e-2, "max": 0.5}            # probabilities and results rounded to bf16
