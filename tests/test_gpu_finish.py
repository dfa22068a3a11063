"""The one call of a layer (restkv_evict) against its four stages: every output bit for bit, on the one-launch finish of
short layers and on either side of each rule that leads there."""
import pytest
import torch

import paper_2605_08840_amd as rk

pytestmark = pytest.mark.gpu


def _layer(p, seed, dup=0, bad=False, token_major=False, shift=0):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    dt = torch.float32 if p.dtype == rk.RESTKV_F32 else torch.bfloat16
    hq, hkv, L, W, d = p.n_q_heads, p.n_kv_heads, p.seq_len, p.window, p.head_dim
    q = torch.randn((hq, W, d), generator=gen, device="cuda").to(dt)

    def cache():
        x = torch.randn((hkv, L, d), generator=gen, device="cuda").to(dt)
        if dup:                                  # equal scores in runs of whole rows: ties are cut by position
            x = x[:, torch.arange(L, device="cuda") % dup]
        if bad:
            x[0, L // 3] = float("inf")
        if token_major:
            x = x.transpose(0, 1).contiguous().transpose(0, 1)
        out = torch.empty(x.numel() + 8, dtype=dt, device="cuda")[shift:shift + x.numel()].view(-1)
        out.copy_((x.transpose(0, 1) if token_major else x).reshape(-1))
        return out

    gram = torch.randn((hq, d, d), generator=gen, device="cuda") / d ** 0.5
    return q, cache(), cache(), torch.matmul(gram, gram.transpose(1, 2).contiguous())


CASES = [
    # (P, W, kept prefix tokens, heads, launches of the box stage, more)
    (1, 1, 1, (1, 1), 0, {}),                                              # everything is kept
    (63, 2, 5, (4, 2), 0, {}),
    (2047, 64, 1900, (8, 2), 0, {}),
    (2048, 64, 1984, (32, 8), 0, dict(dtype="bf16", head_dim=128)),        # largest row of 256 x 8
    (2049, 33, 1, (8, 2), 0, dict(ema_alpha=1.0)),
    (4097, 16, 300, (4, 4), 0, dict(dtype="bf16", token_major=True)),
    (8193, 16, 8193, (4, 1), 0, {}),                                       # everything is kept
    (16384, 8, 700, (4, 2), 0, dict(dtype="bf16")),                        # largest row of all
    (16385, 8, 700, (4, 2), 1, dict(dtype="bf16")),
    (1000, 8, 257, (4, 2), 0, dict(dup=7)),
    (5000, 8, 257, (4, 2), 0, dict(dup=7)),
    (900, 8, 100, (4, 2), 0, dict(bad=True)),
    (900, 8, 100, (4, 2), 0, dict(variant="pmax", base_window=9)),
    (900, 8, 100, (4, 2), 0, dict(adaptive=False, base_window=63)),
    (900, 8, 100, (4, 2), 1, dict(adaptive=False, base_window=65)),        # wider than the launch takes
    (900, 8, 100, (4, 2), 0, dict(beta=31.0)),
    (900, 8, 100, (4, 2), 1, dict(beta=30.0)),
    (900, 8, 100, (4, 2), 0, dict(ld_score=903)),
    (900, 8, 100, (4, 2), 1, dict(shift=1)),                               # rows that are not 16-byte aligned
    (2048, 64, 1984, (64, 64), 0, dict(head_dim=64, dtype="bf16")),        # most workgroups of a row of 2048 ...
    (2048, 64, 1985, (64, 64), 1, dict(head_dim=64, dtype="bf16")),        # ... and one more of each head
]


@pytest.mark.parametrize("P,W,kept,heads,boxes,more", CASES)
def test_evict_matches_its_stages(P, W, kept, heads, boxes, more):
    more = dict(more)
    data = {k: more.pop(k) for k in ("dup", "bad", "token_major", "shift") if k in more}
    if more.get("variant") == "pmax":
        more["variant"] = rk.RESTKV_POOL_MAX
    kw = dict(n_q_heads=heads[0], n_kv_heads=heads[1], head_dim=64, seq_len=P + W, window=W, budget=kept + W, dtype="f32")
    kw.update(more)
    if data.get("token_major"):
        kw.update(kv_stride_h=kw["head_dim"], kv_stride_t=kw["n_kv_heads"] * kw["head_dim"])
    p = rk.make_params(**kw)
    q, k, v, gram = _layer(p, P + 31 * W + kept, **data)
    dt = k.dtype
    a, b = rk.alloc_layer_buffers(p, dt), rk.alloc_layer_buffers(p, dt)
    for buf in (a, b):
        for name in ("score", "ema", "final", "aws_info", "aws_d", "idx", "k_out", "v_out"):
            getattr(buf, name).fill_(-7)
    rk.restkv_score(p, q, k, v, gram, a.score, a.workspace)
    rk.restkv_smooth(p, a.score, a.ema, a.final, a.aws_info, a.aws_d, a.workspace)
    rk.restkv_select(p, a.final, a.idx, a.workspace)
    rk.restkv_compact(p, k, v, a.idx, a.k_out, a.v_out)
    rk.restkv_timing_enable(True)
    try:
        rk.evict_layer(p, q, k, v, gram, b)
        launches = {name: n for name, (_, n) in rk.restkv_timing_read().items()}
    finally:
        rk.restkv_timing_enable(False)
    torch.cuda.synchronize()
    assert launches["box"] == boxes and launches["compact"] == boxes, launches
    for name in ("score", "ema", "final", "aws_info", "aws_d", "idx", "k_out", "v_out"):
        x, y = getattr(a, name), getattr(b, name)
        assert torch.equal(x.view(torch.uint8), y.view(torch.uint8)), name


@pytest.mark.parametrize("P,boxes", [(2047, 0), (16385, 1)])
def test_evict_without_the_optional_outputs(P, boxes):
    """ema, aws_info and aws_d absent: the smoothed scores stay in the workspace, the other outputs are the same bits."""
    p = rk.make_params(n_q_heads=4, n_kv_heads=2, head_dim=64, seq_len=P + 16, window=16, budget=300, dtype="bf16", beta=100.0)
    q, k, v, gram = _layer(p, P)
    a, b = rk.alloc_layer_buffers(p, k.dtype), rk.alloc_layer_buffers(p, k.dtype)
    rk.restkv_score(p, q, k, v, gram, a.score, a.workspace)
    rk.restkv_smooth(p, a.score, a.ema, a.final, a.aws_info, a.aws_d, a.workspace)
    rk.restkv_select(p, a.final, a.idx, a.workspace)
    rk.restkv_compact(p, k, v, a.idx, a.k_out, a.v_out)
    kept = [x.fill_(-7) for x in (b.ema, b.aws_info, b.aws_d)]
    want = [x.clone() for x in kept]
    b.ema = b.aws_info = b.aws_d = None
    rk.restkv_timing_enable(True)
    try:
        rk.evict_layer(p, q, k, v, gram, b)
        launches = rk.restkv_timing_read()["box"][1]
    finally:
        rk.restkv_timing_enable(False)
    torch.cuda.synchronize()
    assert launches == boxes
    for name in ("score", "final", "idx", "k_out", "v_out"):
        assert torch.equal(getattr(a, name).view(torch.uint8), getattr(b, name).view(torch.uint8)), name
    assert all(torch.equal(x, y) for x, y in zip(kept, want))
