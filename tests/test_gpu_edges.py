"""GPU parity at the edges of the kernels' tiles and at the sizes where a launch rule changes side,
against the oracle with the tolerances of gpu_util.py."""
import numpy as np
import pytest
import torch

import workloads
from gpu_util import assert_score_close, attention_statistics, oracle_score, params_for, run_gpu_layer
from test_gpu_parity import _score_against_oracle_then_every_stage_exactly, _smooth_select_inputs, rk  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Hq,Hkv,d,L,W,B", [
    (2, 1, 64, 33, 1, 20),          # 32 keys of prefix: one block exactly, one query row
    (4, 2, 64, 32 + 65, 32, 40),    # 64 query rows per KV head: the last size with two wavefronts; prefix one past two blocks
    (6, 2, 64, 500, 22, 60),        # 66 query rows: four wavefronts, two of them nearly empty
    (8, 1, 128, 1031, 33, 90),      # window one past a 32-row block, prefix of 998
    (3, 3, 128, 32 * 171, 5, 90),   # 3 heads x 171 key blocks: just above the size up to which a score workgroup is one wavefront
    (40, 1, 64, 700, 12, 50),       # more heads per group than the bf16 path takes
])
def test_fp32_kernels_block_edges(rk, oracle_mod, Hq, Hkv, d, L, W, B):  # noqa: F811
    w = workloads.small_case(Hq=Hq, Hkv=Hkv, d=d, L=L, W=W, B=B, dtype="f32", D=2 * d, structure="sinks", seed=57)
    _score_against_oracle_then_every_stage_exactly(rk, oracle_mod, w, "fp32 block edges")


@pytest.mark.parametrize("Hq,Hkv,d,L,W,dtype", [
    (1, 1, 128, 31 + 33, 33, "f32"),      # one head; 31 keys of prefix; the second block of window rows holds one row
    (4, 2, 128, 300, 32, "f32"),          # two heads: one chunk of heads exactly, window rows fill their block
    (6, 2, 64, 289, 31, "f32"),           # three: the last chunk holds one; 258 keys, two past eight blocks
    (5, 1, 128, 1090, 66, "f32"),         # five, three blocks of window rows, 1024 keys
    (6, 2, 128, 300, 9, "bf16"),          # bf16 inputs (one plane) through the same kernels
])
def test_fp32_planes_head_and_row_remainders(rk, oracle_mod, Hq, Hkv, d, L, W, dtype):  # noqa: F811
    """Heads past the last chunk, window rows past the last block: what the workspace held before (ones in every bit,
    then zeros) must not show, bit for bit, and the scores lie within the tolerance of gpu_util.py."""
    w = workloads.small_case(Hq=Hq, Hkv=Hkv, d=d, L=L, W=W, B=W + 20, dtype=dtype, D=2 * d, seed=83)
    q, k, v = workloads.make_qkv(w)
    wo = workloads.make_wo(w)
    p = params_for(rk, w)
    gram = torch.empty((Hq, d, d), dtype=torch.float32, device="cuda")
    rk.restkv_prepare_wo(p, wo.cuda(), gram)
    buf = rk.alloc_layer_buffers(p, q.dtype, "cuda")
    got = []
    rk.restkv_debug_force_fp32(True)
    try:
        for fill in (255, 0):
            buf.workspace.view(torch.uint8).fill_(fill)
            rk.restkv_score(p, q.cuda(), k.cuda(), v.cuda(), gram, buf.score, buf.workspace)
            got.append(buf.score[..., :w.prefix].cpu().numpy())
    finally:
        rk.restkv_debug_force_fp32(False)
    assert np.array_equal(got[0], got[1])
    for g, (Ig, tol) in oracle_score(oracle_mod, w, q, k, v, wo).items():
        assert_score_close(got[0][g], Ig, tol, f"head {g}")


@pytest.mark.parametrize("dtype,pad", [("f32", 1), ("f32", 4), ("bf16", 3), ("bf16", 4)])
def test_fp32_kernels_row_alignment(rk, oracle_mod, dtype, pad):  # noqa: F811
    """Rows that start on no 4-element boundary (element-wise loads) and on one (4-element loads);
    bf16 rows that are not 16-byte aligned take the same kernels."""
    w = workloads.small_case(Hq=4, Hkv=2, d=64, L=210, W=9, B=40, dtype=dtype, D=96, seed=58)
    q, k, v = workloads.make_qkv(w)
    wo = workloads.make_wo(w)
    st = w.head_dim + pad
    kp, vp = (torch.zeros((w.n_kv_heads, w.seq_len, st), dtype=k.dtype, device="cuda") for _ in range(2))
    kp[..., :w.head_dim] = k.cuda()
    vp[..., :w.head_dim] = v.cuda()
    p = params_for(rk, w, kv_stride_t=st, kv_stride_h=w.seq_len * st)
    gram = torch.empty((w.n_q_heads, w.head_dim, w.head_dim), dtype=torch.float32, device="cuda")
    rk.restkv_prepare_wo(p, wo.cuda(), gram)
    buf = rk.alloc_layer_buffers(p, k.dtype, "cuda")
    rk.restkv_score(p, q.cuda(), kp, vp, gram, buf.score, buf.workspace)
    torch.cuda.synchronize()
    got = buf.score.cpu().numpy()
    ref = oracle_score(oracle_mod, w, q, k, v, wo)
    for g in range(w.n_kv_heads):
        Ig, tol = ref[g]
        assert np.isfinite(got[g]).all()
        assert_score_close(got[g], Ig, tol, f"row alignment head {g}")


@pytest.mark.parametrize("Hq,Hkv,d,W,dtype", [
    (256, 256, 64, 33, "bf16"),     # 64 rows per workgroup of the merge, second half nearly empty
    (256, 64, 128, 64, "bf16"),     # 64 rows, groups of 4
    (256, 256, 64, 32, "f32"),      # 32 rows
    (256, 128, 64, 17, "bf16"),     # 32 rows, 15 of them absent
    (64, 16, 128, 63, "bf16"),      # 16 rows, one of them absent
    (64, 8, 64, 60, "f32"),         # 16 rows
    (64, 16, 64, 57, "bf16"),       # 8 rows
    (12, 4, 128, 5, "bf16"),        # 4 rows
])
def test_merge_row_blocks(rk, oracle_mod, Hq, Hkv, d, W, dtype):  # noqa: F811
    """Every number of rows per workgroup of the merge kernel, with keys that hold most of a row's attention."""
    w = workloads.small_case(Hq=Hq, Hkv=Hkv, d=d, L=W + 135, W=W, B=W + 30, dtype=dtype, D=2 * d, structure="sinks", seed=59)
    _score_against_oracle_then_every_stage_exactly(rk, oracle_mod, w, "merge row blocks")


@pytest.mark.parametrize("Hq,Hkv,d,L,W,structure", [
    (32, 32, 64, 64 * 32 + 5, 16, "sinks"),       # score pass with its tiles split, 53 keys in the last one; one row block
    (64, 32, 128, 64 * 32 + 40, 33, "plain"),     # three row blocks; 7 keys in the last tile
    (64, 64, 64, 64 * 64 + 33, 32, "sinks"),      # attention pass too; one key in the second half of the last tile
    (128, 64, 128, 64 * 64 + 1, 9, "lowrank"),    # one key in the first half, none in the second, for the last splits
    (256, 64, 128, 64 * 65, 8, "sinks"),          # whole tiles; one row block, full
    (256, 64, 128, 64 * 64 + 50, 16, "sinks"),    # two, both full
    (256, 64, 128, 64 * 64 + 40, 20, "lowrank"),  # three, the last one half full
    (256, 64, 128, 64 * 66 + 3, 32, "sinks"),     # four
    (154, 22, 64, 64 * 62 + 31, 33, "drift"),     # nine row blocks in three workgroups of the score pass
    (150, 25, 64, 64 * 62 + 31, 33, "sinks"),     # ... in two that take whole tiles: three would be more than the chip holds
    (35, 7, 128, 64 * 73 - 11, 9, "drift"),       # value-Gram pass: five heads in three workgroups
])
def test_tiles_split_between_wavefronts(rk, oracle_mod, Hq, Hkv, d, L, W, structure):  # noqa: F811
    """Few rows per KV head: two wavefronts share a tile's keys and their sums meet, kept-out keys of both halves among them."""
    w = workloads.small_case(Hq=Hq, Hkv=Hkv, d=d, L=L, W=W, B=W + 200, dtype="bf16", D=2 * d, structure=structure, seed=61)
    _score_against_oracle_then_every_stage_exactly(rk, oracle_mod, w, "tiles split between wavefronts")


@pytest.mark.parametrize("P,W,Hkv,kind", [
    (2047, 5, 2, "ties"), (2049, 4, 1, "lognormal"), (4096, 3, 2, "constant"), (4097, 5, 2, "ties"),
    (8192, 2, 1, "lognormal"), (8193, 6, 1, "ties"), (16384, 3, 2, "ties"), (16387, 4, 2, "lognormal"),
    (32768, 2, 1, "ties"),          # the longest row that one workgroup holds
    (32769, 2, 1, "ties"),          # ... and one past it
    (16500, 64, 5, "lognormal"),    # more rows of this length than compute units: the streaming launches
    (40000, 7, 2, "outliers"),      # a few scores 60 octaves above the rest stretch the sample's bins
    (20000, 7, 2, "outliers"), (150001, 6, 2, "outliers"),
])
def test_row_statistics_and_selection_at_launch_rules(rk, oracle_mod, P, W, Hkv, kind):  # noqa: F811
    """Top-B index sums, window and selection, exactly, around the row lengths where another launch takes over,
    with many equal values and with values far above the rest."""
    B, L = W + min(P - 1, 700), P + W
    s = _smooth_select_inputs(77, Hkv, W, P, "lognormal" if kind == "outliers" else kind)
    if kind == "outliers":
        s[:, :, 5::P // 3] *= np.float32(2.0 ** 60)
    p = rk.make_params(n_q_heads=Hkv, n_kv_heads=Hkv, head_dim=64, seq_len=L, window=W, budget=B, dtype="bf16",
                       ema_alpha=0.25, base_window=3, beta=50.0)
    buf = rk.alloc_layer_buffers(p, torch.bfloat16, "cuda")
    buf.score[..., :P].copy_(torch.from_numpy(s))
    rk.restkv_smooth(p, buf.score, buf.ema, buf.final, buf.aws_info, buf.aws_d, buf.workspace)
    rk.restkv_select(p, buf.final, buf.idx, buf.workspace)
    torch.cuda.synchronize()
    fin, idx = buf.final.cpu().numpy(), buf.idx.cpu().numpy()
    info, dd = buf.aws_info.cpu().numpy(), buf.aws_d.cpu().numpy()
    for g in range(Hkv):
        sm = oracle_mod.smooth_head(s[g], 0.25, 50.0, 3, True, B)
        assert dd[g, 0] == sm["d_front"] and dd[g, 1] == sm["d_rear"]
        assert tuple(info[g]) == (sm["w_s"], sm["gamma"])
        np.testing.assert_allclose(fin[g, :P], sm["final"], rtol=2e-5, atol=1e-30)
        np.testing.assert_array_equal(idx[g], oracle_mod.select(fin[g, :P].astype(np.float64), W, B))


@pytest.mark.parametrize("W", [1, 5, 8, 16, 20, 33])
@pytest.mark.parametrize("P", [700, 17000, 40003])     # one launch for the statistics; the streaming launches, also unaligned
def test_infinite_scores_stay_infinite(rk, W, P):  # noqa: F811
    """A score of +-inf (a position that a caller forces in or out) in the newest, the oldest or a middle query
    makes the position's temporal and spatial sums +-inf and touches no other position: the rows
    that pad the window for the kernels add nothing.  Selection keeps the positions at +inf and drops those at -inf."""
    Hkv, B = 7, W + 300
    rng = np.random.default_rng(W * 7 + P)
    s = rng.lognormal(size=(Hkv, W, P)).astype(np.float32)
    hi, lo = [11, P // 2, P - 2], [3, P // 3, P - 30]
    s[:, W - 1, hi[0]] = s[:, 0, hi[1]] = s[:, W // 2, hi[2]] = np.inf
    s[:, W - 1, lo[0]] = s[:, 0, lo[1]] = s[:, W // 2, lo[2]] = -np.inf
    p = rk.make_params(n_q_heads=Hkv, n_kv_heads=Hkv, head_dim=64, seq_len=P + W, window=W, budget=B, dtype="bf16",
                       ema_alpha=0.25, base_window=1, adaptive=False)
    buf = rk.alloc_layer_buffers(p, torch.bfloat16, "cuda")
    buf.score.copy_(torch.from_numpy(s))
    rk.restkv_smooth(p, buf.score, buf.ema, buf.final, buf.aws_info, buf.aws_d, buf.workspace)
    rk.restkv_select(p, buf.final, buf.idx, buf.workspace)
    torch.cuda.synchronize()
    e = s[:, 0].astype(np.float64)
    for i in range(1, W):
        e = 0.25 * s[:, i] + 0.75 * e
    for got in (buf.ema.cpu().numpy(), buf.final.cpu().numpy()):
        np.testing.assert_allclose(got, e, rtol=2e-5)          # (also: infinities at the same places, no NaN)
    idx = buf.idx.cpu().numpy()
    assert all(set(hi) <= set(r.tolist()) and not set(lo) & set(r.tolist()) for r in idx)


@pytest.mark.parametrize("P", [700, 17000, 40003, 70001])     # one launch for the statistics; the streaming launches
def test_heads_of_one_layer_as_of_two(rk, P):  # noqa: F811
    """Eight heads and more are dealt to the workgroups eight at a time, fewer with their parts running fastest: 13 heads
    (eight and a remainder of five) give bit for bit what layers of 7 and 6 heads give."""
    Hkv, W = 13, 5
    s = torch.from_numpy(np.random.default_rng(P).lognormal(size=(Hkv, W, P)).astype(np.float32))

    def run(part):
        p = rk.make_params(n_q_heads=len(part), n_kv_heads=len(part), head_dim=64, seq_len=P + W, window=W, budget=W + 300,
                           dtype="bf16", ema_alpha=0.25, base_window=3, beta=50.0)
        b = rk.alloc_layer_buffers(p, torch.bfloat16, "cuda")
        b.score[..., :P].copy_(part)
        rk.restkv_smooth(p, b.score, b.ema, b.final, b.aws_info, b.aws_d, b.workspace)
        rk.restkv_select(p, b.final, b.idx, b.workspace)
        torch.cuda.synchronize()
        return [x.cpu() for x in (b.ema[:, :P], b.final[:, :P], b.aws_info, b.aws_d, b.idx)]

    for whole, a, b in zip(run(s), run(s[:7]), run(s[7:])):
        assert torch.equal(whole, torch.cat([a, b]))


def _keys(x):
    """The order the searches work in: larger float <=> larger key, -0 < +0, NaNs at the ends."""
    b = np.ascontiguousarray(x, dtype=np.float32).view(np.uint32)
    return np.maximum(np.where(b >> 31, ~b, b ^ np.uint32(0x80000000)), 1).astype(np.int64)


def _top_by_key(row, k):
    """Positions of the k largest entries (equal keys: lower position first), ascending."""
    return np.sort(np.argsort(-_keys(row), kind="stable")[:k])


def _statistics_and_selection_by_key(rk, s, fin, B):
    """Top-B position sums of the raw score s [Hkv, W, P] and selection on fin [Hkv, P], against the order of the keys."""
    Hkv, W, P = s.shape
    p = rk.make_params(n_q_heads=Hkv, n_kv_heads=Hkv, head_dim=64, seq_len=P + W, window=W, budget=B, dtype="bf16",
                       ema_alpha=0.25, base_window=1, beta=1e6)
    buf = rk.alloc_layer_buffers(p, torch.bfloat16, "cuda")
    buf.score.copy_(torch.from_numpy(s.view(np.int32)).cuda().view(torch.float32))
    rk.restkv_smooth(p, buf.score, buf.ema, buf.final, buf.aws_info, buf.aws_d, buf.workspace)
    buf.final.copy_(torch.from_numpy(fin.view(np.int32)).cuda().view(torch.float32))
    rk.restkv_select(p, buf.final, buf.idx, buf.workspace)
    torch.cuda.synchronize()
    dd, idx = buf.aws_d.cpu().numpy(), buf.idx.cpu().numpy()
    bt = min(B, P)
    for g in range(Hkv):
        sums = [int(_top_by_key(s[g, i], bt).sum()) for i in range(W)]
        assert dd[g, 0] == sum(sums[:W // 2]) / (float(bt) * (W // 2))
        assert dd[g, 1] == sum(sums[W // 2:]) / (float(bt) * (W - W // 2))
        np.testing.assert_array_equal(idx[g], np.r_[_top_by_key(fin[g], B - W), np.arange(P, P + W)])


@pytest.mark.parametrize("P", [90, 2048, 5000, 16385, 32768, 40001])
@pytest.mark.parametrize("finite", [0, 9, 70])
def test_rows_of_unset_memory(rk, P, finite):  # noqa: F811
    """Rows of all-ones words (memory filled with 0xFF: NaNs) with fewer ordinary values than are to be chosen:
    the ordinary values are taken, then the lowest positions."""
    Hkv, W, B = 2, 2, 82
    rng = np.random.default_rng(P + finite)
    s = np.full((Hkv, W, P), 0xFFFFFFFF, dtype=np.uint32).view(np.float32)
    for r in s.reshape(-1, P):
        r[rng.choice(P, finite, replace=False)] = rng.normal(size=finite).astype(np.float32)
    _statistics_and_selection_by_key(rk, s, np.ascontiguousarray(s[:, 0]), B)


@pytest.mark.parametrize("P", [40001, 90000])
@pytest.mark.parametrize("seen,unseen", [(-0.0, 0.0), (0.0, -0.0), (-0.0, -0.0)])
def test_zeros_of_both_signs_at_a_bracket_end(rk, P, seen, unseen):  # noqa: F811
    """The sampled searches bracket the threshold with an end at a zero, and zeros of the other sign lie where
    neither samples (positions 22 .. 28: runs of 16 from 0 on and hundreds apart, single ones at 19 | 29 and 21 | 43):
    entries counted by comparison (-0 = +0) and ranked by key (-0 < +0) are the same ones."""
    Hkv, W, zeros = 2, 2, 600 if P < 50000 else 1400
    B = W + zeros + 100
    rng = np.random.default_rng(P)
    row = -1.0 - rng.random(P).astype(np.float32)               # the zeros are the largest entries, the cut lies below them
    row[rng.choice(np.arange(200, P), zeros, replace=False)] = seen
    row[22:29] = unseen
    s = np.broadcast_to(row, (Hkv, W, P)).copy()
    _statistics_and_selection_by_key(rk, s, np.ascontiguousarray(s[:, 0]), B)


@pytest.mark.parametrize("d", [64, 128])
def test_fp32_scores_of_subnormal_weights(rk, oracle_mod, d):  # noqa: F811
    """Keys 87 to 103 nats below the largest have attention weights below the smallest normal FP32 number: their scores
    keep what FP32 holds of them.  A weight is off by half a unit of 2^-149, times the distance I/A, and its product with
    the distance by half a unit again; everything else is within the tolerance of gpu_util.py."""
    w = workloads.small_case(Hq=2, Hkv=2, d=d, L=400, W=9, B=60, dtype="f32", D=2 * d, seed=71)
    q, k, v = workloads.make_qkv(w)
    wo = workloads.make_wo(w)
    q[:], k[..., 0] = 0.0, -16.0 * torch.rand(k.shape[:2], generator=torch.Generator().manual_seed(5))
    q[..., 0] = float(d) ** 0.5                                  # logit of a key = its first component
    k[:, 7, 0] = 87.0
    got = run_gpu_layer(rk, w, q, k, v, wo)["score"]
    fac = oracle_mod.gram_factor(wo.double().numpy().reshape(w.n_q_heads, d, -1))
    for g in range(w.n_kv_heads):
        Ig, I, A, _ = oracle_mod.score_head(q[g:g + 1].numpy(), k[g].numpy(), v[g].numpy(), fac[g:g + 1], w.window,
                                             1.0 / np.sqrt(d), True, aux=True)
        sub = (Ig > 0) & (Ig < 2.0 ** -126)
        assert sub.mean() > 0.5
        tol = 1e-3 * Ig + 2.0 ** -149 * 0.5 * (I[0] / np.where(A[0] > 0, A[0], np.inf) + 1.0)
        bad = np.abs(got[g] - Ig) > tol
        assert not bad.any(), (got[g][bad][:3], Ig[bad][:3], tol[bad][:3])


@pytest.mark.parametrize("dtype,d,late", [("bf16", 64, False), ("bf16", 128, False), ("f32", 64, False), ("f32", 128, False),
                                          ("f32", 128, True)])
def test_largest_key_whose_value_lies_near_the_output(rk, oracle_mod, dtype, d, late):  # noqa: F811
    """A query's largest key holds 0.4 of its attention and its value differs from every other's, c, by 2^-7 c: in the
    expanded distance |z|^2 - 2 z.v + |v|^2 the terms cancel to 2^-14 of their size, the difference z_rest - v of
    the leave-one-out form (0 for the other keys, whose value is the output of the others) does not.  Weights of equal
    logits are equal, so the output of the other keys is c to FP32 rounding and the key's score to a few 2^-24 * 2^7.
    late: the key comes last and never held more than half of the mass (the matrix-core path keeps no such key)."""
    w = workloads.small_case(Hq=2, Hkv=2, d=d, L=606, W=6, B=60, dtype=dtype, D=2 * d, seed=73)
    q, k, v = workloads.make_qkv(w)
    wo = workloads.make_wo(w)
    n = w.prefix - 3 if late else 1
    q[:], k[:] = 0.0, 0.0
    q[..., 0] = float(d) ** 0.5 if d == 64 else 11.3125           # (a bf16 value near sqrt(128))
    k[:, n, 0] = 6.0
    c = torch.from_numpy(np.random.default_rng(3).choice([-1.0, 0.5, 2.0], size=d)).to(v.dtype)
    v[:] = c
    v[:, n] = (c.float() * (1 + 2.0 ** -7)).to(v.dtype)
    got = run_gpu_layer(rk, w, q, k, v, wo)["score"]
    ref = oracle_score(oracle_mod, w, q, k, v, wo, with_amax=True)
    for g in range(w.n_kv_heads):
        Ig, _, A = ref[g]
        assert ((A[:, n] > 0.3) & (A[:, n] < 0.5)).all()
        np.testing.assert_allclose(got[g][:, n], Ig[:, n], rtol=1e-3)


@pytest.mark.parametrize("P", [32769, 70001, 270000])
@pytest.mark.parametrize("kind", ["constant", "four values", "mostly zero", "lognormal", "one tie too many"])
def test_exact_search_of_long_rows(rk, P, kind):  # noqa: F811
    """Rows with more candidates than the streaming searches hold (many equal values; a bracket too wide at this
    length): the exact search of the row, with and without equal values at the cut."""
    Hkv, W, B = 2, 2, 2 + 4000
    rng = np.random.default_rng(P)
    s = rng.lognormal(size=(Hkv, W, P)).astype(np.float32)
    if kind == "constant":
        s[:] = 1.5
    elif kind == "four values":
        s = rng.integers(0, 4, size=s.shape).astype(np.float32)
    elif kind == "mostly zero":
        s[rng.random(s.shape) < 0.99] = 0.0
    elif kind == "one tie too many":                   # 4001 entries at the top value: the last is left out (select), none (statistics)
        s[:] = 0.25
        s[:, :, P - 4001:] = 8.0
    _statistics_and_selection_by_key(rk, s, np.ascontiguousarray(s[:, 0]), B)


@pytest.mark.parametrize("dtype,d", [("f32", 64), ("bf16", 64), ("bf16", 128)])
def test_gram_and_statistics_at_any_float_address(rk, dtype, d):  # noqa: F811
    """gram, attn_out and lse need no more than the alignment of their floats: same results as from aligned arrays."""
    w = workloads.small_case(Hq=4, Hkv=2, d=d, L=300, W=9, B=40, dtype=dtype, D=96, seed=79)
    q, k, v = (x.cuda() for x in workloads.make_qkv(w))
    p = params_for(rk, w)
    gram = torch.empty((4, d, d), dtype=torch.float32, device="cuda")
    rk.restkv_prepare_wo(p, workloads.make_wo(w).cuda(), gram)
    out, lse = attention_statistics(q.cpu(), k.cpu(), v.cpu(), w.window)

    def shifted(x):
        y = torch.empty(x.numel() + 1, dtype=x.dtype, device="cuda")[1:].view(x.shape)
        return y.copy_(x)

    got = []
    for move in (lambda x: x.cuda(), shifted):
        buf = rk.alloc_layer_buffers(p, q.dtype, "cuda")
        g, o, s = move(gram), move(out), move(lse)
        rk.restkv_score(p, q, k, v, g, buf.score, buf.workspace)
        one = buf.score.clone()
        rk.restkv_score_from_attention(p, q, k, v, g, o, s, buf.score, buf.workspace)
        torch.cuda.synchronize()
        got.append((one, buf.score.clone()))
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])


@pytest.mark.parametrize("Hq,Hkv,d,L,W,side,two", [
    (8, 8, 128, 64 * 3 + 1 + 16, 16, 1, 0),     # prefix of three tiles and a key: hardly more tiles than units to share
    (32, 8, 128, 64 * 33, 64, 1, 1),            # 33 tiles a head, prefix ends with a tile
    (32, 8, 128, 64 * 33 + 1, 64, 1, 1),        # one key in the last tile of the whole context
    (16, 4, 128, 1500, 40, 1, 0),               # four KV heads, five row blocks
    (28, 4, 128, 900, 33, 0, 0),                # nine row blocks: the second workgroup of a split is nearly empty, one pass after the other
    (64, 8, 128, 1200, 64, 1, 0),               # two full workgroups of rows, two of heads
    (8, 8, 64, 2300, 16, 0, 0),                 # splits of two tiles, half a row block
    (64, 8, 64, 1900, 33, 0, 0),                # ... and row blocks for all wavefronts
    (64, 8, 128, 2300, 64, 1, 0),               # three tiles, no second parts
    (8, 8, 128, 2300, 5, 1, 1),                 # three tiles, one wavefront with rows
])
def test_attention_and_value_gram_passes_share_the_chip(rk, oracle_mod, Hq, Hkv, d, L, W, side, two):  # noqa: F811
    """The two passes in one launch, side by side (`side`; heavy weights in two parts: `two`) or one after the other: first
    and last KV head against the oracle, and the same bits from a workspace full of ones (no sum is read that was not written)."""
    w = workloads.small_case(Hq=Hq, Hkv=Hkv, d=d, L=L, W=W, B=W + 20, dtype="bf16", D=2 * d, structure="sinks", seed=91)
    q, k, v = workloads.make_qkv(w)
    wo = workloads.make_wo(w)
    p = params_for(rk, w)
    assert rk.restkv_debug_score_plan(p)[2:] == (side, two)
    gram = torch.empty((Hq, d, d), dtype=torch.float32, device="cuda")
    rk.restkv_prepare_wo(p, wo.cuda(), gram)
    buf = rk.alloc_layer_buffers(p, q.dtype, "cuda")
    got = []
    for fill in (255, 0):
        buf.workspace.view(torch.uint8).fill_(fill)
        rk.restkv_score(p, q.cuda(), k.cuda(), v.cuda(), gram, buf.score, buf.workspace)
        got.append(buf.score[..., :w.prefix].cpu().numpy())
    assert np.array_equal(got[0], got[1])
    for g, (Ig, tol) in oracle_score(oracle_mod, w, q, k, v, wo, heads=[0, Hkv - 1]).items():
        assert_score_close(got[0][g], Ig, tol, f"head {g}")


def test_smoothing_of_more_rows_than_one_grid_dimension_holds(rk):  # noqa: F811
    """16.8 million (head, query) rows of 256 threads, 2^32 threads in all: accepted, and the same numbers as torch's."""
    Hkv, W, P = 8192, 2048, 16
    p = params_for(rk, workloads.small_case(Hq=Hkv, Hkv=Hkv, d=64, L=P + W, W=W, B=W + 5, dtype="f32", alpha=0.5, beta=1.0))
    score = torch.rand((Hkv, W, P), device="cuda", generator=torch.Generator("cuda").manual_seed(3))
    ema = torch.empty((Hkv, P), device="cuda")
    final = torch.empty_like(ema)
    info = torch.empty((Hkv, 2), dtype=torch.int32, device="cuda")
    drift = torch.empty((Hkv, 2), dtype=torch.float64, device="cuda")
    ws = torch.empty(3 << 30, dtype=torch.uint8, device="cuda")
    rk.restkv_smooth(p, score, ema, final, info, drift, ws)
    # the EMA's weights: 2^-(W-1) for the oldest query, then 2^-(W-i)
    wts = torch.tensor([0.5 ** (W - max(i, 1)) for i in range(W)], dtype=torch.float64, device="cuda")
    want = torch.einsum("gwp,w->gp", score[:, -40:].double(), wts[-40:])
    assert torch.allclose(ema.double(), want, rtol=1e-5, atol=1e-9)
    # (a budget above the window is above the prefix here: every position of a row is taken)
    assert bool((drift == (P - 1) / 2.0).all()) and bool((info[:, 0] == 5).all())
