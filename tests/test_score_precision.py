"""How far the scores may lie from 64 bits: bounds that a kernel with fewer bits in any of its products fails.

The bounds come from the same inputs on the CPU: the scores in float64, and once more with one quantity rounded as a kernel
would.  The CPU tests show that each planted loss of bits exceeds the bound that the GPU tests then apply."""
import numpy as np
import pytest
import torch

import workloads
from gpu_util import params_for
from test_gpu_parity import rk  # noqa: F401


def scores64(q, k, v, gram, W, weights=None, dot=None, gmax=False):
    """Indicator of one KV head (mean over its query heads, or the largest) [W, P] in float64; q [G,W,d], k, v [L,d], gram [G,d,d].  The key
    with a row's largest weight in leave-one-out form.  weights: what becomes of the weights of A V [G,W,L], relative to
    their row's largest; dot(a, b): the products a b^T."""
    q, k, v, gram = q.double(), k.double(), v.double(), gram.double()
    G, _, d = q.shape
    L = k.shape[0]
    P = L - W
    dot = dot or (lambda a, b: a @ b.T)
    hidden = torch.arange(L)[None, :] > (P + torch.arange(W))[:, None]
    logits = torch.stack([(dot(q[h], k) / d ** 0.5).masked_fill(hidden, float("-inf")) for h in range(G)])
    exact = torch.exp(logits - logits.amax(-1, keepdim=True))
    used = weights(exact) if weights else exact
    out = torch.zeros((W, P), dtype=torch.float64)
    for h in range(G):
        p, pr = exact[h], used[h]
        den = p.sum(-1, keepdim=True)
        top = p.argmax(-1, keepdim=True)
        rest = p.scatter(1, top, 0.0).sum(-1, keepdim=True)
        z = dot(pr, v.T) / den
        u = dot(z, gram[h])
        vv = (dot(v[:P], gram[h]) * v[:P]).sum(-1)
        x = ((u * z).sum(-1, keepdim=True) - 2.0 * dot(u, v[:P]) + vv[None]).clamp_min(0.0)
        omit = den - p
        omit.scatter_(1, top, rest)
        ind = p[:, :P] / omit[:, :P] * x.sqrt()
        y = dot(pr.scatter(1, top, 0.0), v.T) / rest - v[top[:, 0]]
        loo = (p.gather(1, top) / den)[:, 0] * (dot(y, gram[h]) * y).sum(-1).clamp_min(0.0).sqrt()
        rows = (top[:, 0] < P).nonzero()[:, 0]
        ind[rows, top[rows, 0]] = loo[rows]
        out = torch.maximum(out, ind) if gmax else out + ind
    return out if gmax else out / G


def distance(a, b):
    return float((a.double() - b).norm() / b.norm())


def heads_of(w, q, k, v, gram, g):
    G = w.group
    return q[g * G:(g + 1) * G], k[g], v[g], gram[g * G:(g + 1) * G], w.window


def gpu_scores(rk, w, q, k, v, wo, **over):  # noqa: F811
    p = params_for(rk, w, **over)
    gram = torch.empty((w.n_q_heads, w.head_dim, w.head_dim), dtype=torch.float32, device="cuda")
    rk.restkv_prepare_wo(p, wo.cuda(), gram)
    buf = rk.alloc_layer_buffers(p, q.dtype, "cuda")
    rk.restkv_score(p, q.cuda(), k.cuda(), v.cuda(), gram, buf.score, buf.workspace)
    return buf.score[..., :w.prefix].cpu(), gram.cpu()


def gram_of(w, wo):
    x = wo.double().reshape(w.n_q_heads, w.head_dim, -1)
    return x @ x.transpose(1, 2)


# ---- bf16: weights of the attention pass beside the value-Gram pass --------------------------

def in_bf16(p, seed=5):
    """Weights rounded to bf16 in a frame that is a random fraction of a power of two for every row."""
    c = 1.0 + torch.rand((*p.shape[:2], 1), generator=torch.Generator().manual_seed(seed), dtype=torch.float64)
    return (p * c).bfloat16().double() / c


def largest_exact(p, keys, share):
    """What one reference per tile gives: the largest weight of a 64-key tile stays as it is where it is more than `share` of
    its split's sum (`keys` keys), the others are rounded."""
    out = in_bf16(p)
    for k0 in range(0, p.shape[2], keys):
        total = p[..., k0:k0 + keys].sum(-1, keepdim=True)
        for t0 in range(k0, min(k0 + keys, p.shape[2]), 64):
            x, o = p[..., t0:t0 + 64], out[..., t0:t0 + 64]
            m = x.amax(-1, keepdim=True)
            o.copy_(torch.where((x == m) & (m > share * total), x, o))
    return out


def heavy_groups_exact(p, keys, share, iw):
    """What a second part of the weights gives: all weights of 16 keys stay as they are in the `iw` window positions of all
    heads where one of them is more than `share` of its split's sum."""
    out = in_bf16(p)
    for k0 in range(0, p.shape[2], keys):
        total = p[..., k0:k0 + keys].sum(-1, keepdim=True)
        for i0 in range(0, p.shape[1], iw):
            for t0 in range(k0, min(k0 + keys, p.shape[2]), 16):
                x = p[:, i0:i0 + iw, t0:t0 + 16]
                if bool((x > share * total[:, i0:i0 + iw]).any()):
                    out[:, i0:i0 + iw, t0:t0 + 16] = x
    return out


# key splits of few tiles beside the value-Gram pass: (Hq, Hkv, L, W)
CLUSTERED = [(16, 4, 4096, 16), (28, 4, 3000, 64), (32, 8, 3000, 64), (64, 8, 4096, 16)]


def clustered(Hq, Hkv, L, W, strength):
    """Keys and queries that share a rank-16 component: a few weights carry a row's sum."""
    w = workloads.small_case(Hq=Hq, Hkv=Hkv, d=128, L=L, W=W, B=W + 100, dtype="bf16", D=256, seed=29)
    gen = torch.Generator().manual_seed(31)
    q, k, v = (t.float() for t in workloads.make_qkv(w))
    f = torch.randn((Hkv, 16, 128), generator=gen) * 0.25 * strength
    k += torch.randn((Hkv, L, 16), generator=gen) @ f
    q += torch.randn((Hq, W, 16), generator=gen) @ f.repeat_interleave(w.group, dim=0)
    return w, q.bfloat16(), k.bfloat16(), v.bfloat16(), workloads.make_wo(w)


def weights_bound(w, plan, ref, args):
    """One and a half times what the weights' rounding gives with 16 keys exact wherever one is above 1/16 of its split's
    sum, and 1.2e-6 for everything else: u and Gram matrices enter their products as two bf16 parts, whose sum is up to
    2^-17 = 7.6e-6 of an entry off; over the 128 entries of a product that averages to some 7.6e-6 / sqrt(3 128) = 4e-7
    for each, and FP32 sums add as much."""
    gp = 1 << (w.group - 1).bit_length()
    sim = scores64(*args, weights=lambda p: heavy_groups_exact(p, 64 * plan[1], 1.0 / 16.0, 32 // gp))
    return 1.5 * distance(sim, ref) + 1.2e-6


@pytest.mark.parametrize("strength", [0.7, 1.0])
@pytest.mark.parametrize("Hq,Hkv,L,W", CLUSTERED)
def test_one_exact_weight_per_tile_would_exceed_the_bound(Hq, Hkv, L, W, strength):
    import paper_2605_08840_amd as lib
    w, q, k, v, wo = clustered(Hq, Hkv, L, W, strength)
    plan = lib.restkv_debug_score_plan(params_for(lib, w))
    assert plan[2:] == (1, 1)
    args = heads_of(w, q, k, v, gram_of(w, wo), 0)
    ref = scores64(*args)
    planted = scores64(*args, weights=lambda p: largest_exact(p, 64 * plan[1], 1.0 / 33.0))
    assert distance(planted, ref) > 2.0 * weights_bound(w, plan, ref, args)


@pytest.mark.gpu
@pytest.mark.parametrize("strength", [0.7, 1.0])
@pytest.mark.parametrize("Hq,Hkv,L,W", CLUSTERED)
def test_heavy_weights_beside_the_value_gram_pass(rk, Hq, Hkv, L, W, strength):  # noqa: F811
    """Few key splits: clustered scores stay as near to 64 bits as the weights that enter in two parts allow."""
    w, q, k, v, wo = clustered(Hq, Hkv, L, W, strength)
    plan = rk.restkv_debug_score_plan(params_for(rk, w))
    assert plan[2:] == (1, 1)
    got, gram = gpu_scores(rk, w, q, k, v, wo)
    for g in (0, Hkv - 1):
        args = heads_of(w, q, k, v, gram, g)
        ref = scores64(*args)
        assert distance(got[g], ref) <= weights_bound(w, plan, ref, args), f"head {g}"


# ---- FP32 ---------------------------------------------------------------------------------

@pytest.mark.gpu
@pytest.mark.parametrize("Hkv,d,P,W", [(1, 64, 700, 33), (2, 128, 1031, 40), (8, 64, 6001, 64)])
def test_fp32_division_and_square_root_round_correctly(rk, Hkv, d, P, W):  # noqa: F811
    """Queries of zeros: a row that sees n keys has weights of exactly 1 / n, and values of two whole numbers have exact
    squared norms.  The value-norm indicator is then fl(fl(1 / n) fl(sqrt(a^2 + b^2))), bit for bit."""
    w = workloads.small_case(Hq=Hkv, Hkv=Hkv, d=d, L=P + W, W=W, B=W + 40, dtype="f32")
    gen = torch.Generator().manual_seed(P)
    q = torch.zeros((Hkv, W, d))
    k = torch.randn((Hkv, w.seq_len, d), generator=gen)
    v = torch.zeros_like(k)
    v[..., 3] = torch.randint(1, 2048, v.shape[:2], generator=gen).float()
    v[..., d - 2] = torch.randint(1, 2048, v.shape[:2], generator=gen).float()
    p = params_for(rk, w, variant=rk.RESTKV_IND_VALUE_NORM)
    buf = rk.alloc_layer_buffers(p, q.dtype, "cuda")
    rk.restkv_score(p, q.cuda(), k.cuda(), v.cuda(), None, buf.score, buf.workspace)
    n = np.arange(P + 1, P + W + 1, dtype=np.float32)
    norms = np.sqrt((v[:, :P].numpy() ** 2).sum(-1))
    want = (np.float32(1.0) / n)[None, :, None] * norms[:, None, :]
    assert want.dtype == np.float32 and np.array_equal(buf.score[..., :P].cpu().numpy(), want)


def planes(x, n):
    """x as the sum of n bf16 numbers, each the nearest to what the others have left."""
    out, rest = [], x.float()
    for _ in range(n):
        h = rest.bfloat16().float()
        out.append(h.double())
        rest = rest - h
    return out


def plane_dot(n=3, without=()):
    """Products of values in planes: those of planes i and j with i + j < 3 (high, middle, low), less the ones in `without`."""
    def f(a, b):
        pa, pb = planes(a, n), planes(b, n)
        return sum(pa[i] @ pb[j].T for i in range(n) for j in range(n) if i + j < 3 and (i, j) not in without)
    return f


# plain and clustered logits, groups of one and several heads, both head dimensions; one and several key splits
FP32_LAYERS = [(1, 1, 64, 300, 5, 0.0), (4, 1, 128, 1500, 20, 0.5), (4, 2, 64, 2100, 33, 0.5), (2, 2, 128, 2100, 16, 0.0), (14, 2, 128, 1000, 9, 0.0)]


def fp32_layer(Hq, Hkv, d, L, W, strength):
    w = workloads.small_case(Hq=Hq, Hkv=Hkv, d=d, L=L, W=W, B=W + 60, dtype="f32", D=2 * d, seed=37)
    gen = torch.Generator().manual_seed(41)
    q, k, v = workloads.make_qkv(w)
    f = torch.randn((Hkv, 16, d), generator=gen) * 0.25 * strength
    k += torch.randn((Hkv, L, 16), generator=gen) @ f
    q += torch.randn((Hq, W, 16), generator=gen) @ f.repeat_interleave(w.group, dim=0)
    return w, q, k, v, workloads.make_wo(w)


def fp32_bound(w, ref, args, **kw):
    """Twice what products in float32 alone give (torch's, on the CPU), and 3e-7, five roundings of 2^-24, for the exponential, the quotient, the
    root and the sums outside of the products."""
    return 2.0 * distance(scores64(*args, dot=lambda a, b: (a.float() @ b.float().T).double(), **kw), ref) + 3e-7


@pytest.mark.parametrize("layer", FP32_LAYERS)
def test_planes_with_any_part_missing_would_exceed_the_bound(layer):
    w, q, k, v, wo = fp32_layer(*layer)
    args = heads_of(w, q, k, v, gram_of(w, wo).float(), 0)
    ref = scores64(*args)
    bound = fp32_bound(w, ref, args)
    assert distance(scores64(*args, dot=plane_dot()), ref) < 0.2 * bound
    for lost in (dict(n=2), dict(without={(0, 2)}), dict(without={(2, 0)}), dict(without={(1, 1)}), dict(without={(1, 0)})):
        assert distance(scores64(*args, dot=plane_dot(**lost)), ref) > 1.5 * bound, lost


@pytest.mark.gpu
@pytest.mark.parametrize("layer", FP32_LAYERS)
def test_fp32_scores_are_as_exact_as_fp32_products(rk, layer):  # noqa: F811
    w, q, k, v, wo = fp32_layer(*layer)
    got, gram = gpu_scores(rk, w, q, k, v, wo)
    for g in range(w.n_kv_heads):
        args = heads_of(w, q, k, v, gram, g)
        ref = scores64(*args)
        assert distance(got[g], ref) <= fp32_bound(w, ref, args), f"head {g}"


@pytest.mark.gpu
@pytest.mark.parametrize("d,W", [(64, 9), (128, 40)])
@pytest.mark.parametrize("value", [float("-inf"), -torch.finfo(torch.float32).max, -3.4e38, -1e30])
def test_fp32_keys_outside_of_the_planes(rk, d, W, value):  # noqa: F811
    """Keys whose logits are -inf or far below every other: weight and score zero, the rest of every row as if they were
    not there.  -FLT_MAX and -3.4e38 round to an infinite bf16."""
    w, q, k, v, wo = fp32_layer(4, 2, d, 777, W, 0.0)
    q[..., 5] = q[..., 5].abs() + 0.5
    gone = [0, 31, 300, 600]
    k[:, gone] = 0.0
    k[:, gone, 5] = value
    got, gram = gpu_scores(rk, w, q, k, v, wo)
    for g in range(2):
        args = heads_of(w, q, k.clamp_min(-1e30), v, gram, g)
        ref = scores64(*args)
        assert bool((got[g][:, gone] == 0).all()) and bool((ref[:, gone] == 0).all())
        assert distance(got[g], ref) <= fp32_bound(w, ref, args), f"head {g}"


@pytest.mark.gpu
@pytest.mark.parametrize("d,W", [(64, 9), (128, 40)])
@pytest.mark.parametrize("q2,k2,v2,m2", [
    (110, -110, 0, 0),          # keys whose low planes would be subnormal
    (-112, 112, 0, 0),          # queries likewise; keys whose products with a query's high plane are of ordinary size
    (0, 0, -114, 118),          # values, outputs and u rows; Gram entries near the end of the range
    (0, 0, 40, -70),            # Gram entries below the range, values inside it
    (0, 0, 61, -100),           # values above it
])
def test_fp32_operands_far_from_one(rk, d, W, q2, k2, v2, m2):  # noqa: F811
    """Powers of two that leave the logits as they are and scale the scores: as exact as with operands around one."""
    w, q, k, v, wo = fp32_layer(4, 2, d, 777, W, 0.3)
    p = params_for(rk, w)
    gram = gram_of(w, wo).float()
    buf = rk.alloc_layer_buffers(p, q.dtype, "cuda")
    up = lambda x, e: torch.ldexp(x, torch.tensor(e // 2)).ldexp(torch.tensor(e - e // 2))        # noqa: E731
    rk.restkv_score(p, up(q, q2).cuda(), up(k, k2).cuda(), up(v, v2).cuda(), up(gram, m2).cuda(), buf.score, buf.workspace)
    got = buf.score[..., :w.prefix].cpu().double() * 2.0 ** (-v2 - m2 / 2)
    for g in range(2):
        args = heads_of(w, q, k, v, gram, g)
        ref = scores64(*args)
        assert distance(got[g], ref) <= fp32_bound(w, ref, args), f"head {g}"


@pytest.mark.gpu
@pytest.mark.parametrize("Hq,Hkv,d,P,form,gmax", [
    (12, 4, 128, 4096, (4, 1), False), (12, 4, 128, 4097, (4, 0), False),       # 512 workgroups: the last size at which the heads of a group have wavefronts of their own
    (8, 4, 64, 6144, (2, 1), False), (8, 4, 64, 6145, (4, 0), False),           # the same for heads of 64, two wavefronts
    (20, 4, 64, 6144, (4, 1), False), (20, 4, 64, 6145, (4, 0), False),         # five heads on four wavefronts
    (8, 4, 64, 1000, (2, 1), True), (20, 4, 64, 1000, (4, 1), True),            # the group's largest: the wavefronts' results meet by maximum
    (4, 4, 128, 4096, (1, 0), False),                                           # one head: one wavefront
])
def test_fp32_heads_side_by_side_and_one_after_the_other(rk, Hq, Hkv, d, P, form, gmax):  # noqa: F811
    """Either side of the rule, with keys that planes do not hold.  form: wavefronts of a workgroup, whether they divide the heads."""
    w, q, k, v, wo = fp32_layer(Hq, Hkv, d, P + 3, 3, 0.3)
    over = dict(variant=rk.RESTKV_GROUP_MAX) if gmax else {}
    assert rk.restkv_debug_fp32_plan(params_for(rk, w, **over))[2:] == form
    q[..., 5] = q[..., 5].abs() + 0.5
    gone = [0, 31, 300, P - 1]
    k[:, gone] = 0.0
    k[:, gone, 5] = float("-inf")
    got, gram = gpu_scores(rk, w, q, k, v, wo, **over)
    for g in (0, Hkv - 1):
        args = heads_of(w, q, k.clamp_min(-1e30), v, gram, g)
        ref = scores64(*args, gmax=gmax)
        assert bool((got[g][:, gone] == 0).all())
        assert distance(got[g], ref) <= fp32_bound(w, ref, args, gmax=gmax), f"head {g}"
