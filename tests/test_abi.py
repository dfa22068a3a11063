"""Host-side checks of the C ABI: the library loads, exports what the header declares,
and turns bad arguments into error codes before anything is enqueued (no GPU needed)."""
import ctypes
import os
import re

import pytest
import torch

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def rk():
    import paper_2605_08840_amd as r
    if not os.path.exists(r.LIB_PATH):
        import __graft_entry__
        __graft_entry__.build()
    return r


def good(rk, **kw):
    base = dict(n_q_heads=4, n_kv_heads=2, head_dim=64, seq_len=1024, window=32, budget=128, dtype="f32")
    base.update(kw)
    return rk.make_params(**base)


def test_exports_every_declared_symbol(rk):
    text = open(os.path.join(ROOT, "include", "restkv.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    names = sorted(set(re.findall(r"\b(restkv_[a-z_]+)\s*\(", text)))
    assert {"restkv_score", "restkv_score_smooth", "restkv_smooth", "restkv_smooth_b", "restkv_select_b", "restkv_select", "restkv_compact", "restkv_prepare_wo",
            "restkv_workspace_bytes", "restkv_strerror", "restkv_version"} <= set(names)
    L = rk.lib()
    for n in names:
        assert hasattr(L, n), n
    assert rk.restkv_version() >= 100


def test_param_block_layout_matches_header(rk):
    # 14 four-byte fields then 5 eight-byte fields, no padding
    assert ctypes.sizeof(rk.RestkvParams) == 14 * 4 + 5 * 8


def test_workspace_bytes(rk):
    assert rk.restkv_workspace_bytes(good(rk)) > 0
    big = good(rk, n_q_heads=32, n_kv_heads=8, head_dim=128, seq_len=131072, window=64, budget=2048, dtype="bf16")
    assert rk.restkv_workspace_bytes(big) > 32 * 131008 * 4      # holds v M v^T for every head
    for bad in (dict(budget=32), dict(budget=2000), dict(n_q_heads=5), dict(window=0),
                dict(window=1024), dict(base_window=4), dict(ema_alpha=1.5), dict(beta=0.0),
                dict(beta=1e-7),           # floor(|x| / beta) would leave the 32-bit range
                dict(variant=3), dict(variant=0x30), dict(variant=0x80), dict(variant=8)):
        assert rk.restkv_workspace_bytes(good(rk, **bad)) == 0, bad


def test_error_codes_without_launch(rk):
    L = rk.lib()
    p = good(rk)
    one = ctypes.c_void_p(256)            # never dereferenced on the host
    ws_n = rk.restkv_workspace_bytes(p)
    # null pointers
    assert L.restkv_score(ctypes.byref(p), None, one, one, None, one, one, ws_n, None) == -1
    assert L.restkv_smooth(ctypes.byref(p), None, None, one, None, None, one, ws_n, None) == -1
    assert L.restkv_select(ctypes.byref(p), one, None, None, 0, None) == -1
    assert L.restkv_select(ctypes.byref(p), one, one, None, 0, None) == -3
    assert L.restkv_compact(ctypes.byref(p), one, one, None, one, one, None) == -1
    assert L.restkv_prepare_wo(ctypes.byref(p), None, 128, one, None) == -1
    # workspace: missing, too small, misaligned
    assert L.restkv_score(ctypes.byref(p), one, one, one, None, one, None, 0, None) == -3
    assert L.restkv_score(ctypes.byref(p), one, one, one, None, one, one, 256, None) == -3
    assert L.restkv_score_smooth(ctypes.byref(p), one, one, one, None, one, None, one, None, None, one, 256, None) == -3
    assert L.restkv_score_smooth(ctypes.byref(p), one, one, one, None, None, None, one, None, None, one, ws_n, None) == -1
    assert L.restkv_score(ctypes.byref(p), one, one, one, None, one, ctypes.c_void_p(264), ws_n, None) == -3
    assert L.restkv_smooth(ctypes.byref(p), one, None, one, None, None, one, 8, None) == -3
    # unsupported / invalid blocks
    assert L.restkv_score(ctypes.byref(good(rk, head_dim=96)), one, one, one, None, one, one, ws_n, None) == -2
    assert L.restkv_score(ctypes.byref(good(rk, dtype=7)), one, one, one, None, one, one, ws_n, None) == -2
    assert L.restkv_score(ctypes.byref(good(rk, budget=32)), one, one, one, None, one, one, ws_n, None) == -1
    assert L.restkv_select(ctypes.byref(good(rk, budget=1025)), one, one, None, 0, None) == -1
    bad_ld = good(rk, ld_score=100)
    assert L.restkv_smooth(ctypes.byref(bad_ld), one, None, one, None, None, one, 1 << 20, None) == -1
    # the streaming reference: null, odd sizes, misaligned pointers; nothing to move is not an error
    assert L.restkv_stream_reference(None, 32, one, 16, None) == -1
    assert L.restkv_stream_reference(one, 32, None, 16, None) == -1
    assert L.restkv_stream_reference(one, 24, one, 16, None) == -1
    assert L.restkv_stream_reference(one, 32, one, 20, None) == -1
    assert L.restkv_stream_reference(ctypes.c_void_p(264), 32, one, 16, None) == -1
    assert L.restkv_stream_reference(None, 0, None, 0, None) == 0
    for code in (0, -1, -2, -3, -4, -99):
        assert len(rk.strerror(code)) > 0


@pytest.mark.parametrize("Hq,Hkv", [(4, 1), (4, 2)])
@pytest.mark.parametrize("L", [1100, 2112, 4096, 8192, 16384, 32768])
@pytest.mark.parametrize("W", [4, 16, 32, 64])
def test_few_kv_heads_keep_all_key_splits_beside_the_value_gram_pass(rk, Hq, Hkv, L, W):
    """With one or two KV heads the key splits (64 at most) leave half of the units free, so the value-Gram pass beside
    them is no reason for longer ones: that made clustered contexts up to 19 % slower than one pass after the other."""
    splits, tiles, side, two = rk.restkv_debug_score_plan(good(rk, n_q_heads=Hq, n_kv_heads=Hkv, head_dim=128, seq_len=L, window=W,
                                                          budget=W + 64, dtype="bf16"))
    all_tiles = (L + 63) // 64
    assert (side, two) == (1, 0) and tiles == -(-all_tiles // min(64, all_tiles)) and splits == -(-all_tiles // tiles)


def test_score_plan_covers_the_context_and_both_launch_orders(rk):
    seen = set()
    for Hq, Hkv in [(4, 1), (4, 2), (8, 8), (16, 4), (28, 4), (32, 8), (64, 8), (1024, 256)]:
        for d in (64, 128):
            for L in (129, 1100, 2112, 9001, 32768, 131072):
                for W in (1, 33, 64):
                    p = good(rk, n_q_heads=Hq, n_kv_heads=Hkv, head_dim=d, seq_len=L, window=W, budget=W + 64, dtype="bf16")
                    splits, tiles, side, two = rk.restkv_debug_score_plan(p)
                    assert 1 <= splits <= 64 and (splits - 1) * tiles * 64 < L <= splits * tiles * 64
                    assert d == 128 or side == 0
                    assert side or not two
                    seen.add((d, side, two))
    assert seen == {(64, 0, 0), (128, 0, 0), (128, 1, 0), (128, 1, 1)}
    with pytest.raises(rk.RestkvError):
        rk.restkv_debug_score_plan(good(rk))               # float32
    assert rk.lib().restkv_debug_score_plan(ctypes.byref(good(rk)), None) == -1


@pytest.mark.parametrize("heads,d,L,W,plan", [
    ((4, 2), 64, 1024, 32, (32, 1, 2, 1)),             # the toy layer
    ((8, 2), 128, 16384, 16, (64, 1, 4, 0)),           # two wavefronts hold a head's rows: splits on half of the compute units ...
    ((16, 4), 128, 16384, 16, (64, 0, 4, 0)),          # ... and on all of them: two launches
    ((16, 4), 64, 16384, 16, (64, 1, 4, 0)),
    ((28, 4), 128, 4096, 32, (64, 1, 4, 1)), ((28, 4), 128, 4129, 32, (44, 1, 4, 0)),
    ((8, 8), 128, 2000, 16, (63, 0, 1, 0)),            # a group of one head
])
def test_fp32_plan_on_either_side_of_its_rules(rk, heads, d, L, W, plan):
    p = good(rk, n_q_heads=heads[0], n_kv_heads=heads[1], head_dim=d, seq_len=L, window=W, budget=W + 64)
    assert rk.restkv_debug_fp32_plan(p) == plan
    with pytest.raises(rk.RestkvError):
        rk.restkv_debug_fp32_plan(good(rk, dtype="bf16"))
    assert rk.lib().restkv_debug_fp32_plan(ctypes.byref(p), None) == -1


def test_binding_has_no_cpu_fallback(rk, monkeypatch):
    import paper_2605_08840_amd.binding as b
    monkeypatch.setattr(b, "_lib", None)
    monkeypatch.setattr(b, "LIB_PATH", "/nonexistent/librestkv.so")
    with pytest.raises(ImportError):
        b.lib()


def test_evict_checks_every_stage_before_it_enqueues(rk):
    L = rk.lib()
    p = good(rk)
    one = ctypes.c_void_p(256)            # never dereferenced on the host
    ws_n = rk.restkv_workspace_bytes(p)

    def call(p, at=None, ws=one, n=ws_n):
        # q, k, v, gram, score, ema, final, aws_info, aws_d, idx, k_out, v_out
        ptrs = [None if j == at else one for j in range(12)]
        return L.restkv_evict(ctypes.byref(p), *ptrs, ws, n, None)

    for at in (0, 1, 2, 4, 6, 9, 10, 11):
        assert call(p, at) == -1, at
    assert call(p, ws=None) == -3 and call(p, n=ws_n - 256) == -3 and call(p, ws=ctypes.c_void_p(264)) == -3
    assert call(good(rk, budget=32)) == -1 and call(good(rk, head_dim=96)) == -2


@pytest.mark.parametrize("fused,calls", [(False, ["restkv_evict"]),
                                         (True, ["restkv_score_smooth", "restkv_select", "restkv_compact"])])
def test_fused_switch_of_a_layer_reaches_the_fused_call(rk, monkeypatch, fused, calls):
    import types

    import paper_2605_08840_amd.binding as b
    p, seen = good(rk), []
    buf = rk.alloc_layer_buffers(p, torch.float32, "cpu")

    class Recorder:
        def __getattr__(self, name):
            return lambda *args: seen.append(name) or 0

    monkeypatch.setattr(b, "_lib", Recorder())
    q, k, v, gram = torch.empty(4, 32, 64), torch.empty(2, 1024, 64), torch.empty(2, 1024, 64), torch.empty(4, 64, 64)
    rk.evict_layer(p, q, k, v, gram, buf, stream=types.SimpleNamespace(cuda_stream=0), fused=fused)
    assert seen == calls
